// ae_noise.hip — the channel: per-sample power normalisation fused with additive
// white Gaussian noise drawn from Philox4x32-10, its backward, and the
// Monte-Carlo bookkeeping kernels (message bits, error counts).
//
// Counter layout: key = (seed_lo, seed_hi); counter = (sample_lo, sample_hi,
// quad, stream) with `sample` the global sample index, `quad` = element index / 4
// in (c,h,w) order, stream 0 = channel noise, 1 = message bits.  The u32 -> normal
// map is a fixed sequence of correctly rounded binary32 operations (explicit
// round-to-nearest intrinsics, never contracted), so the noise tensor is
// reproducible bit for bit.
#include "ae_device.h"
#include "ae_internal.h"
#include "ae_philox.h"

namespace ae {
namespace {

constexpr int NT = 256;

template <typename T> __device__ __forceinline__ void ld4(const T* p, float (&v)[4]);
template <> __device__ __forceinline__ void ld4<float>(const float* p, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
template <> __device__ __forceinline__ void ld4<bf16_t>(const bf16_t* p, float (&v)[4]) {
  const uint2 t = *reinterpret_cast<const uint2*>(p);
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xFFFF0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xFFFF0000u);
}
template <typename T> __device__ __forceinline__ void st4(T* p, const float (&v)[4]);
template <> __device__ __forceinline__ void st4<float>(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
template <> __device__ __forceinline__ void st4<bf16_t>(bf16_t* p, const float (&v)[4]) {
  uint2 t;
  t.x = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
  t.y = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
  *reinterpret_cast<uint2*>(p) = t;
}

// One wavefront per sample (TPS = 64) or, for small batches, workgroups of a sample (TPS = 256): gridDim.y of them, each of
// which forms the sample's sum of squares for itself and writes its share of the quads (24 samples of 20 x 18 x 30 in
// bfloat16: 23 us with one workgroup each, 7.7 with 21).  FLAT: the sample is a contiguous vector of n = C
// elements with n % 4 == 0 (16-byte / 8-byte vector access).  Otherwise the sample
// is stored [HW][C] and element i = c*HW + hw of the (c,h,w) order is gathered.
template <int TPS>
__device__ __forceinline__ float sample_sum(float v, float* sm) {
  if (TPS == 64) return wave_sum(v);
  return block_sum<NT>(v, sm);
}

// (z and y may be the same buffer: no __restrict__; every lane reads the elements it writes before it writes them)
template <typename T, bool FLAT, int TPS>
__global__ void k_pnorm_awgn(const T* z, T* y, int64_t batch, int C, int HW, int do_pnorm,
                             int do_awgn, float sigma, uint64_t seed, uint64_t first_sample, int vec) {
  __shared__ float sm[NT / 64 + 1];
  const int lane = threadIdx.x % TPS;
  const int64_t b = (int64_t)blockIdx.x * (NT / TPS) + (threadIdx.x / TPS);
  if (b >= batch) return;                        // whole wavefronts (TPS = 64) or never (TPS = 256: grid = batch)
  const int64_t n = (int64_t)C * HW;
  const T* zb = z + b * n;
  T* yb = y + b * n;
  const int64_t nquads = (n + 3) >> 2;
  const int64_t share = (nquads + gridDim.y - 1) / gridDim.y, q_lo = blockIdx.y * share, q_hi = q_lo + share < nquads ? q_lo + share : nquads;
  float scale = 1.0f;
  if (do_pnorm) {
    float ss = 0.0f;
    if (FLAT || vec) {                           // vec: whole aligned quads, the sum in storage order
#pragma unroll 4
      for (int64_t q = lane; q < nquads; q += TPS) {
        float v[4];
        ld4<T>(zb + 4 * q, v);
        ss = fmaf(v[0], v[0], ss); ss = fmaf(v[1], v[1], ss); ss = fmaf(v[2], v[2], ss); ss = fmaf(v[3], v[3], ss);
      }
    } else {
#pragma unroll 8
      for (int64_t i = lane; i < n; i += TPS) { float v = Store<T>::ld(zb + i); ss = fmaf(v, v, ss); }
    }
    ss = sample_sum<TPS>(ss, sm);
    const float ms = ss / (float)n;
    scale = ms > 0.0f ? 1.0f / sqrtf(ms) : 0.0f;
  }
  const uint64_t sample = first_sample + (uint64_t)b;
  for (int64_t q = q_lo + lane; q < q_hi; q += TPS) {
    float g[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (do_awgn) {
      normal_quad(seed, sample, (uint32_t)q, g);
#pragma unroll
      for (int j = 0; j < 4; ++j) g[j] = __fmul_rn(sigma, g[j]);
    }
    if (FLAT) {
      float v[4];
      ld4<T>(zb + 4 * q, v);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = __fadd_rn(__fmul_rn(v[j], scale), g[j]);
      st4<T>(yb + 4 * q, v);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t i = 4 * q + j;
        if (i < n) {
          const int64_t c = n <= 0x7FFFFFFF ? (int64_t)((unsigned)i / (unsigned)HW) : i / HW, hw = i - c * HW;
          const int64_t pos = (int64_t)hw * C + c;
          Store<T>::st(yb + pos, __fadd_rn(__fmul_rn(Store<T>::ld(zb + pos), scale), g[j]));
        }
      }
    }
  }
}

// Short flat latents (n = 4 L elements, L a power of two up to 32): L neighbouring lanes own one sample, one
// quad each, so a wavefront holds 64 / L samples and every lane of it loads, generates and stores; the sum
// of squares is reduced inside each group of L lanes with xor-shuffles (the same order for every sample,
// wherever it sits in the batch).  z and y may be the same buffer.
template <typename T, int L>
__global__ __launch_bounds__(NT) void k_pnorm_awgn_short(const T* z, T* y, int64_t batch, int do_pnorm, int do_awgn,
                                                         float sigma, uint64_t seed, uint64_t first_sample) {
  const int lane = threadIdx.x % L;
  const int64_t b = (int64_t)blockIdx.x * (NT / L) + (threadIdx.x / L);
  const bool valid = b < batch;                  // every lane stays for the shuffles
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (valid) ld4<T>(z + b * (4 * L) + 4 * lane, v);
  float scale = 1.0f;
  if (do_pnorm) {
    float ss = 0.0f;
    ss = fmaf(v[0], v[0], ss); ss = fmaf(v[1], v[1], ss); ss = fmaf(v[2], v[2], ss); ss = fmaf(v[3], v[3], ss);
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
    const float ms = ss / (float)(4 * L);
    scale = ms > 0.0f ? 1.0f / sqrtf(ms) : 0.0f;
  }
  float g[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (do_awgn) {
    normal_quad(seed, first_sample + (uint64_t)b, (uint32_t)lane, g);
#pragma unroll
    for (int j = 0; j < 4; ++j) g[j] = __fmul_rn(sigma, g[j]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = __fadd_rn(__fmul_rn(v[j], scale), g[j]);
  if (valid) st4<T>(y + b * (4 * L) + 4 * lane, v);
}

// x = z/r: dz = g/r - z * sum(g z) / (n r^3); elementwise in storage order
template <typename T, int TPS>
__global__ void k_pnorm_bwd(const T* __restrict__ z, const T* __restrict__ g, T* __restrict__ dz, int64_t batch,
                            int64_t n) {          // (gridDim.y workgroups per sample as in k_pnorm_awgn)
  __shared__ float sm[NT / 64 + 1];
  const int lane = threadIdx.x % TPS;
  const int64_t b = (int64_t)blockIdx.x * (NT / TPS) + (threadIdx.x / TPS);
  if (b >= batch) return;
  const T* zb = z + b * n;
  const T* gb = g + b * n;
  float szz = 0.0f, sgz = 0.0f;
#pragma unroll 8
  for (int64_t i = lane; i < n; i += TPS) {
    const float zv = Store<T>::ld(zb + i), gv = Store<T>::ld(gb + i);
    szz = fmaf(zv, zv, szz);
    sgz = fmaf(gv, zv, sgz);
  }
  szz = sample_sum<TPS>(szz, sm);
  sgz = sample_sum<TPS>(sgz, sm);
  const float ms = szz / (float)n;
  float inv_r = 0.0f, coef = 0.0f;
  if (ms > 0.0f) {
    inv_r = 1.0f / sqrtf(ms);
    coef = sgz / (float)n * inv_r * inv_r * inv_r;
  }
  const int64_t share = (n + gridDim.y - 1) / gridDim.y, i_hi = (blockIdx.y + 1) * share < n ? (blockIdx.y + 1) * share : n;
#pragma unroll 8
  for (int64_t i = blockIdx.y * share + lane; i < i_hi; i += TPS) {
    const float zv = Store<T>::ld(zb + i), gv = Store<T>::ld(gb + i);
    Store<T>::st(dz + b * n + i, gv * inv_r - zv * coef);
  }
}

__global__ void k_noise(uint64_t seed, uint64_t first_sample, int64_t batch, int64_t n, float* __restrict__ out) {
  const int64_t nquads = (n + 3) >> 2;
  const int64_t total = batch * nquads;
  for (int64_t it = (int64_t)blockIdx.x * NT + threadIdx.x; it < total; it += (int64_t)gridDim.x * NT) {
    const int64_t b = it / nquads, q = it % nquads;
    float g[4];
    normal_quad(seed, first_sample + (uint64_t)b, (uint32_t)q, g);
    for (int j = 0; j < 4; ++j)
      if (4 * q + j < n) out[b * n + 4 * q + j] = g[j];
  }
}

// Message bits: one Philox call yields the 128 bits of a unit (sample, group of 128 positions).  A workgroup generates
// GEN_UNITS units, one per thread, into LDS and then all its threads stream out the units' outputs, which are contiguous
// in x.  (One call per output, the earliest form, was bound by the generator's integer multiplies: 65 536 x 64 bits, 17 MB,
// 20.1 us; now 9.)  VEC: k % 4 == 0 and x on a 16-byte border: a quad never leaves its word.
template <int GEN_UNITS, bool VEC>
__global__ __launch_bounds__(NT) void k_gen_bits(uint64_t seed, uint64_t first_sample, int64_t batch, int k, float* __restrict__ x) {
  constexpr int W = VEC ? 4 : 1;
  __shared__ uint32_t words[GEN_UNITS * 4];
  const int64_t per_row = ((int64_t)k + 127) >> 7, units = batch * per_row;
  for (int64_t u0 = (int64_t)blockIdx.x * GEN_UNITS; u0 < units; u0 += (int64_t)gridDim.x * GEN_UNITS) {
    const int nu = units - u0 < GEN_UNITS ? (int)(units - u0) : GEN_UNITS;
    const int64_t b0 = u0 / per_row;
    const int g0 = (int)(u0 % per_row);
    __syncthreads();                               // the previous units have been read
    if ((int)threadIdx.x < nu) {
      const int64_t u = u0 + threadIdx.x, b = u / per_row;
      const uint64_t sample = first_sample + (uint64_t)b;
      const U4 w = philox4x32_10((uint32_t)sample, (uint32_t)(sample >> 32), (uint32_t)(u % per_row), 1u, (uint32_t)seed,
                                 (uint32_t)(seed >> 32));
      words[4 * threadIdx.x] = w.x; words[4 * threadIdx.x + 1] = w.y; words[4 * threadIdx.x + 2] = w.z; words[4 * threadIdx.x + 3] = w.w;
    }
    __syncthreads();
    // outputs [e0, e1) of x; j0: position of e0 in its row
    const int64_t ul = u0 + nu - 1, bl = ul / per_row;
    const int last = (int)(ul % per_row) * 128 + 128;
    const int64_t j0 = (int64_t)g0 * 128, e0 = b0 * k + j0, e1 = bl * k + (last < k ? last : k);
    const unsigned n = (unsigned)(e1 - e0);        // at most GEN_UNITS * 128
    for (unsigned r = threadIdx.x * W; r < n; r += NT * W) {
      const unsigned t = (unsigned)j0 + r;         // (below 2^31 + 2^13)
      const unsigned row = t / (unsigned)k, j = t - row * (unsigned)k;
      const unsigned unit = row * (unsigned)per_row + (j >> 7) - (unsigned)g0;
      const uint32_t word = words[4 * unit + ((j >> 5) & 3)] >> (j & 31);
      if constexpr (VEC)
        *reinterpret_cast<float4*>(x + e0 + r) = make_float4((word & 1u) ? 1.0f : -1.0f, (word & 2u) ? 1.0f : -1.0f,
                                                             (word & 4u) ? 1.0f : -1.0f, (word & 8u) ? 1.0f : -1.0f);
      else
        x[e0 + r] = (word & 1u) ? 1.0f : -1.0f;
    }
  }
}

// Rows of a few bits: a thread per row, which needs a part of one word.  (2^22 rows of 1 / 2 / 4 bits: 11.6 / 12.4 / 22.6 us, 25.7 /
// 28.4 / 26.8 through LDS, 13.7 / 24.1 / 43.9 with one generator call per output.)
__global__ __launch_bounds__(NT) void k_gen_bits_few(uint64_t seed, uint64_t first_sample, int64_t batch, int k, float* __restrict__ x) {
  for (int64_t b = (int64_t)blockIdx.x * NT + threadIdx.x; b < batch; b += (int64_t)gridDim.x * NT) {
    const uint64_t sample = first_sample + (uint64_t)b;
    const uint32_t word = philox4x32_10((uint32_t)sample, (uint32_t)(sample >> 32), 0u, 1u, (uint32_t)seed, (uint32_t)(seed >> 32)).x;
    for (int j = 0; j < k; ++j) x[b * k + j] = ((word >> j) & 1u) ? 1.0f : -1.0f;
  }
}

// Wrong decisions of a batch: L neighbouring lanes (a power of two) own a row, each reading 16 bytes (VEC) or one value
// of either tensor at a time, so a wavefront reads whole lines; the lanes of a row are combined by one ballot.  (One
// thread per row, the earlier form, read a line per lane and value: 65 536 x 64 decisions, 34 MB, 69.7 us; now 13.  512 workgroups: the same.)
template <bool VEC>
__global__ __launch_bounds__(NT) void k_count_errors(const float* __restrict__ y, const float* __restrict__ x, int64_t batch, int k, int log_l,
                                                     unsigned long long* bit_err, unsigned long long* blk_err) {
  constexpr int W = VEC ? 4 : 1;
  __shared__ unsigned long long sm[2][NT / 64];
  const int lane = threadIdx.x & 63, L = 1 << log_l;
  const int sub = lane & (L - 1);
  const uint64_t row_lanes = L == 64 ? ~0ull : ((1ull << L) - 1ull) << (lane & ~(L - 1));
  const int64_t rows_pass = (int64_t)gridDim.x * (NT >> log_l);
  unsigned long long bits = 0, rows = 0;
  // (the rows of a wavefront's lanes are neighbours: all its lanes make the same number of passes, a lane past the batch counts nothing)
  const int64_t r0 = ((int64_t)blockIdx.x * NT + (threadIdx.x & ~63)) >> log_l;
  for (int64_t rb = r0; rb < batch; rb += 4 * rows_pass) {
    const float *yr[4], *xr[4];
    int wrong[4] = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < 4; ++u) {                  // four rows at a time: their loads are in flight together
      int64_t b = rb + u * rows_pass + (lane >> log_l);
      b = b < batch ? b : batch - 1;
      yr[u] = y + b * k;
      xr[u] = x + b * k;
    }
    for (int j = sub * W; j < k; j += L * W) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if constexpr (VEC) {
          const float4 a = *reinterpret_cast<const float4*>(yr[u] + j), c = *reinterpret_cast<const float4*>(xr[u] + j);
          wrong[u] += ((a.x > 0.5f) != (c.x > 0.0f)) + ((a.y > 0.5f) != (c.y > 0.0f)) + ((a.z > 0.5f) != (c.z > 0.0f)) + ((a.w > 0.5f) != (c.w > 0.0f));
        } else {
          wrong[u] += (yr[u][j] > 0.5f) != (xr[u][j] > 0.0f);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (rb + u * rows_pass + (lane >> log_l) >= batch) wrong[u] = 0;
      bits += (unsigned)wrong[u];
      const uint64_t any = __ballot(wrong[u] != 0);
      if (sub == 0 && (any & row_lanes)) ++rows;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { bits += __shfl_xor(bits, off, 64); rows += __shfl_xor(rows, off, 64); }
  if (lane == 0) { sm[0][threadIdx.x >> 6] = bits; sm[1][threadIdx.x >> 6] = rows; }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned long long t = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) t += sm[threadIdx.x][i];
    if (t) atomicAdd(threadIdx.x ? blk_err : bit_err, t);
  }
}

constexpr int kCountBlocks = 256;

inline int grid_for(int64_t items, int cap) {
  int64_t g = (items + NT - 1) / NT;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

}  // namespace

// small batches of long vectors get a whole workgroup per sample
static bool block_per_sample(int64_t batch, int64_t n) { return batch < 1024 && n >= 1024; }
// workgroups per sample then: two per compute unit in all, at least 512 values (128 quads of noise) to a share.  Every share
// forms the whole sum for itself, which costs less than its noise saves at any length: binary32, one sample of 2^22 / 2^26 values 3.2 ->
// 0.53 / 68 -> 12 ms against one workgroup, 64 samples of 2^20 1.10 -> 0.40 ms, 1 024 to 4 096 values the same.
static unsigned shares_of_sample(int64_t batch, int64_t n) {
  int64_t s = 512 / batch;
  if (s > n / 512) s = n / 512;
  return (unsigned)(s < 1 ? 1 : s);
}

int launch_pnorm_awgn(const void* z, void* y, int64_t batch, int c, int hw, int dtype, int do_pnorm, int do_awgn,
                      float sigma, uint64_t seed, uint64_t first_sample, hipStream_t s) {
  // a flat vector is a tensor with hw == 1 (or c == 1: then (c,h,w) order is storage order too)
  int C = c, HW = hw;
  if (C == 1) { C = HW; HW = 1; }
  const bool flat = HW == 1 && (C % 4 == 0);
  if (flat && C <= 128 && (C & (C - 1)) == 0) {
    // short latents: several samples per wavefront
    const int L = C / 4;
    const int64_t blocks = (batch + NT / L - 1) / (NT / L);
    if (blocks > 0x7FFFFFFF) return fail(AE_EINVAL, "pnorm_awgn: batch too large");
#define LAUNCH_S(T, LV)                                                                                              \
  hipLaunchKernelGGL((k_pnorm_awgn_short<T, LV>), dim3((unsigned)blocks), dim3(NT), 0, s, (const T*)z, (T*)y, batch, \
                     do_pnorm, do_awgn, sigma, seed, first_sample)
#define LAUNCH_SL(T)                                                                                 \
  switch (L) {                                                                                       \
    case 1: LAUNCH_S(T, 1); break;   case 2: LAUNCH_S(T, 2); break;   case 4: LAUNCH_S(T, 4); break;  \
    case 8: LAUNCH_S(T, 8); break;   case 16: LAUNCH_S(T, 16); break; default: LAUNCH_S(T, 32); break; \
  }
    if (dtype == AE_BF16) { LAUNCH_SL(bf16_t) } else { LAUNCH_SL(float) }
#undef LAUNCH_SL
#undef LAUNCH_S
    return launch_status("pnorm_awgn_short");
  }
  const bool wide = block_per_sample(batch, (int64_t)C * HW);
  const int64_t blocks = wide ? batch : (batch + NT / 64 - 1) / (NT / 64);
  if (blocks > 0x7FFFFFFF) return fail(AE_EINVAL, "pnorm_awgn: batch too large");
  // (in place, a sample's sum has to be read before any of it is overwritten: one workgroup)
  const unsigned shares = wide && z != y ? shares_of_sample(batch, (int64_t)C * HW) : 1;
  const int vec = ((int64_t)C * HW) % 4 == 0 && ((uintptr_t)z & (dtype == AE_BF16 ? 7 : 15)) == 0;
#define LAUNCH(T, F, TPSV)                                                                                          \
  hipLaunchKernelGGL((k_pnorm_awgn<T, F, TPSV>), dim3((unsigned)blocks, shares), dim3(NT), 0, s, (const T*)z, (T*)y, batch, C, \
                     HW, do_pnorm, do_awgn, sigma, seed, first_sample, vec)
#define LAUNCH_F(T, F) do { if (wide) LAUNCH(T, F, 256); else LAUNCH(T, F, 64); } while (0)
  if (dtype == AE_BF16) { if (flat) LAUNCH_F(bf16_t, true); else LAUNCH_F(bf16_t, false); }
  else { if (flat) LAUNCH_F(float, true); else LAUNCH_F(float, false); }
#undef LAUNCH_F
#undef LAUNCH
  return launch_status("pnorm_awgn");
}

int launch_pnorm_bwd(const void* z, const void* g, void* dz, int64_t batch, int64_t n, int dtype, hipStream_t s) {
  const bool wide = block_per_sample(batch, n);
  const int64_t blocks = wide ? batch : (batch + NT / 64 - 1) / (NT / 64);
  const unsigned shares = wide ? shares_of_sample(batch, n) : 1;
#define LAUNCH(T, TPSV)                                                                                             \
  hipLaunchKernelGGL((k_pnorm_bwd<T, TPSV>), dim3((unsigned)blocks, shares), dim3(NT), 0, s, (const T*)z, (const T*)g, (T*)dz, \
                     batch, n)
  if (dtype == AE_BF16) { if (wide) LAUNCH(bf16_t, 256); else LAUNCH(bf16_t, 64); }
  else { if (wide) LAUNCH(float, 256); else LAUNCH(float, 64); }
#undef LAUNCH
  return launch_status("pnorm_bwd");
}

int launch_noise(uint64_t seed, uint64_t first_sample, int64_t batch, int64_t n, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_noise, dim3(grid_for(batch * ((n + 3) / 4), 1 << 20)), dim3(NT), 0, s, seed, first_sample, batch,
                     n, out);
  return launch_status("noise");
}

int launch_gen_bits(uint64_t seed, uint64_t first_sample, int64_t batch, int k, float* x, hipStream_t s) {
  if (k <= 4) {
    hipLaunchKernelGGL(k_gen_bits_few, dim3(grid_for(batch, 1 << 20)), dim3(NT), 0, s, seed, first_sample, batch, k, x);
    return launch_status("gen_bits");
  }
  const int64_t units = batch * (((int64_t)k + 127) >> 7);
  // A unit per thread while units are short, a wavefront of units beyond: 64 units leave three wavefronts idle while the first
  // calls the generator (2^20 rows of 5 / 16 / 32 bits 20.6 / 20.8 / 22.8 us, with 256 11.3 / 12.4 / 21.4), 256 make few workgroups of
  // large batches (65 536 x 63: 7.9 and 10.4 us; 4 096 x 4 099: 19.3 and 26.7).
  const bool vec = k % 4 == 0 && ((uintptr_t)x & 15) == 0, few = k <= 32;
  const int per_group = few ? 256 : 64;
  const int64_t groups = (units + per_group - 1) / per_group;
  const dim3 grid((unsigned)(groups < (1 << 20) ? groups : (1 << 20)));
#define GEN_BITS(U, V) hipLaunchKernelGGL((k_gen_bits<U, V>), grid, dim3(NT), 0, s, seed, first_sample, batch, k, x)
  if (few) { if (vec) GEN_BITS(256, true); else GEN_BITS(256, false); }
  else { if (vec) GEN_BITS(64, true); else GEN_BITS(64, false); }
#undef GEN_BITS
  return launch_status("gen_bits");
}

int launch_count_errors(const float* y, const float* x, int64_t batch, int k, uint64_t* bit_err, uint64_t* blk_err,
                        hipStream_t s) {
  if (k >= 65536) return fail(AE_EINVAL, "count_errors: k must be below 65536");
  const bool vec = k % 4 == 0 && (((uintptr_t)y | (uintptr_t)x) & 15) == 0;
  const int loads = vec ? k / 4 : k;
  int log_l = 0;                                   // as many lanes as a row has loads, up to a wavefront
  while (log_l < 6 && (2 << log_l) <= loads) ++log_l;
  // few workgroups: every one ends in two atomic adds on the same two counters
  const dim3 grid(grid_for(batch << log_l, kCountBlocks));
  if (vec)
    hipLaunchKernelGGL((k_count_errors<true>), grid, dim3(NT), 0, s, y, x, batch, k, log_l, (unsigned long long*)bit_err, (unsigned long long*)blk_err);
  else
    hipLaunchKernelGGL((k_count_errors<false>), grid, dim3(NT), 0, s, y, x, batch, k, log_l, (unsigned long long*)bit_err, (unsigned long long*)blk_err);
  return launch_status("count_errors");
}

}  // namespace ae
