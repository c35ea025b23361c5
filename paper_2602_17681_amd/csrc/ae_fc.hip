// ae_fc.hip — big fully-connected layers of bfloat16 models straight from the binary32 parameters.
//
// A layer of 32 M weights and a hundred rows is bound by reading its weights once: 134 MB in binary32, 25 us at 5.4 TB/s.
// Repacking them first (a bfloat16 copy for the forward pass, a transposed one for the input gradient) reads those 134 MB,
// writes 67 and reads 67 again.  Here the product reads the parameters itself and rounds them on their way into LDS, with
// the values a copy would hold:
//     forward          y [m][n] = sum_k a[m][k] w[n][k]     (w [n][k]: a row is contiguous in k)
//     input gradient   dx[m][n] = sum_k a[m][k] w[k][n]     (TRANS: a thread takes 8 rows x 4 columns and turns them in registers)
//
// A workgroup of four wavefronts computes 128 x 64 outputs over a range of K in slabs of 128: the next slab's loads are in
// flight (48 KiB per workgroup; a compute unit has room for three) while the present one is multiplied from LDS, which holds
// both operands in MFMA fragment order: octet o (8 of the slab's 128 k's) of row r at 16-byte slot (r % 32) ^ o of block
// (r / 32, o / 2), half o % 2, so that the 16 octets of a row that neighbouring lanes store fall into 16 different columns
// of the banks.  The matrix cores are a fifth busy: 64-column tiles and splits of K for bytes in flight, nothing else.
// Measured, 1 024 x 32 768 weights: 43 us per product at 128 rows, 3.1 TB/s, where conversion, transpose and the products on
// the copies took 50 + 31 us forward and 70 + 30 us backward (forward pass of two such layers 158 -> 97 us).
#include "ae_device.h"
#include "ae_internal.h"

namespace ae {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 64, BK = 128;

struct FcParams {
  const bf16_t* a; const float* w; const float* bias; bf16_t* y; float* part;
  int M, N, K, k_per_split, tiles_n, tiles_m, act;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4v to_bf16(const float4v& lo, const float4v& hi) {
  return uint4v{pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
}
// byte offset of octet o of row r in an operand's slab
__device__ __forceinline__ unsigned frag_slot(int r, int o) {
  return (unsigned)(((r >> 5) * (BK / 16) + (o >> 1)) * 1024 + (o & 1) * 512 + (((r & 31) ^ o) * 16));
}

template <bool TRANS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_fc(FcParams p) {
  __shared__ __attribute__((aligned(16))) char smem[(BM + BN) * BK * 2];
  char* const sA = smem;
  char* const sW = smem + BM * BK * 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // column tiles of one split are neighbours, a contiguous range of them on each of the eight dies: they share the rows of a
  const int per = (int)gridDim.x >> 3;
  const int lb = (int)blockIdx.x < (per << 3) ? ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
  const int tile_n = lb % p.tiles_n, t = lb / p.tiles_n, tile_m = t % p.tiles_m, split = t / p.tiles_m;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int k_lo = split * p.k_per_split, k_hi = min(p.K, k_lo + p.k_per_split);
  const int rows = min(BM, p.M - m0);            // (rows past M read zeros)
  const __amdgpu_buffer_rsrc_t rA = rsrc(p.a + (int64_t)m0 * p.K, (int64_t)rows * p.K * 2);
  const __amdgpu_buffer_rsrc_t rW = TRANS ? rsrc(p.w + (int64_t)k_lo * p.N + n0, ((int64_t)(k_hi - k_lo) * p.N - n0) * 4)
                                          : rsrc(p.w + (int64_t)n0 * p.K, (int64_t)BN * p.K * 4);
  const int o16 = tid & 15, r16 = tid >> 4;      // a (and w [n][k]): octet and first row;  w [k][n]: column quad and octet
  unsigned off_a = ((unsigned)r16 * (unsigned)p.K + (unsigned)(k_lo + o16 * 8)) * 2u;
  unsigned off_w = TRANS ? ((unsigned)(r16 * 8) * (unsigned)p.N + (unsigned)(o16 * 4)) * 4u
                         : ((unsigned)r16 * (unsigned)p.K + (unsigned)(k_lo + o16 * 8)) * 4u;
  uint4v ra[8], rw[8];
  auto load = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) rw[i] = TRANS ? __builtin_amdgcn_raw_buffer_load_b128(rW, off_w + (unsigned)i * (unsigned)p.N * 4u, 0, 0)
                                              : __builtin_amdgcn_raw_buffer_load_b128(rW, off_w + (unsigned)(i >> 1) * 16u * (unsigned)p.K * 4u + (unsigned)(i & 1) * 16u, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) ra[i] = __builtin_amdgcn_raw_buffer_load_b128(rA, off_a + (unsigned)i * 16u * (unsigned)p.K * 2u, 0, 0);
    off_a += BK * 2;
    off_w += TRANS ? (unsigned)p.N * (BK * 4u) : BK * 4u;
  };
  auto store = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<uint4v*>(sA + frag_slot(r16 + 16 * i, o16)) = ra[i];
    float4v f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = __builtin_bit_cast(float4v, rw[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (TRANS) {
        const float4v lo = {f[0][i], f[1][i], f[2][i], f[3][i]}, hi = {f[4][i], f[5][i], f[6][i], f[7][i]};
        *reinterpret_cast<uint4v*>(sW + frag_slot(o16 * 4 + i, r16)) = to_bf16(lo, hi);
      } else {
        *reinterpret_cast<uint4v*>(sW + frag_slot(r16 + 16 * i, o16)) = to_bf16(f[2 * i], f[2 * i + 1]);
      }
    }
  };
  const int wm = wave & 1, wn = wave >> 1;       // 64 rows x 32 columns per wavefront
  floatx16 acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.0f;
  load();
  for (int k = k_lo; k < k_hi; k += BK) {
    store();
    __syncthreads();
    if (k + BK < k_hi) load();
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
      const int o = 2 * s + (lane >> 5);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(sW + frag_slot(wn * 32 + (lane & 31), o));
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(sA + frag_slot(wm * 64 + i * 32 + (lane & 31), o));
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  const int col = n0 + wn * 32 + (lane & 31);
  const float bias = !p.part && p.bias ? p.bias[col] : 0.0f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = m0 + wm * 64 + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
      if (m >= p.M) continue;
      if (p.part) p.part[((int64_t)split * p.M + m) * p.N + col] = acc[i][e];
      else p.y[(int64_t)m * p.N + col] = f32_to_bf16(apply_act(round_to_storage<bf16_t>(acc[i][e] + bias), p.act));
    }
}

// y = act(round(sum of the splits + bias)), four columns per thread
__global__ __launch_bounds__(256) void k_fc_finish(const float4* __restrict__ part, int splits, int64_t quads, int quads_n,
                                                   const float* __restrict__ bias, int act, uint2* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= quads) return;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
  for (int s = 0; s < splits; ++s) {
    const float4 u = part[(int64_t)s * quads + i];
    v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
  }
  if (bias) {
    const float* b = bias + (int)(i % quads_n) * 4;          // (the parameter blob's vectors need not lie on 16-byte borders)
    v.x += b[0]; v.y += b[1]; v.z += b[2]; v.w += b[3];
  }
  const float f[4] = {apply_act(round_to_storage<bf16_t>(v.x), act), apply_act(round_to_storage<bf16_t>(v.y), act),
                      apply_act(round_to_storage<bf16_t>(v.z), act), apply_act(round_to_storage<bf16_t>(v.w), act)};
  y[i] = make_uint2(pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]));
}

}  // namespace

// Whole slabs and tiles in both directions, 32-bit byte offsets, at least 2^20 weights (is_big_fc), and few rows: every 128
// of them read the parameters again.  Two layers of 1 024 x 32 768, forward
// and forward + backward, against the packed copies: 1 row 67 and 254 us against 136 and 349, 128 rows 97 and 306 against 158 and 414,
// 512 rows 209 and 482 against 219 and 578; 2 048 x 512: 47 and 105 against 68 and 143, at 512 rows 50 and 122 against 77 and 155.
bool fc_direct_supported(int m, int cin, int cout) {
  return m <= 512 && cin % BK == 0 && cout % BK == 0 && (int64_t)cin * cout >= (1 << 20) && (int64_t)cin * cout < (1 << 29);
}

int launch_fc_direct(const FcArgs& a, hipStream_t s) {
  if (a.m < 1 || a.n % BN != 0 || a.k % BK != 0 || (int64_t)a.n * a.k >= (1 << 29) || (int64_t)BM * a.k * 2 > 0x7FFFFFFF)
    return fail(AE_EINVAL, "fc_direct: shape not supported");
  FcParams p;
  p.a = (const bf16_t*)a.a; p.w = a.w; p.bias = a.bias; p.y = (bf16_t*)a.y; p.act = a.act;
  p.M = a.m; p.N = a.n; p.K = a.k;
  p.tiles_n = a.n / BN; p.tiles_m = (a.m + BM - 1) / BM;
  // where K is split, at most 512 workgroups (two per compute unit), each over two slabs at least; more than that without a split only
  const int tiles = p.tiles_n * p.tiles_m, slabs = a.k / BK;
  int64_t splits = 512 / tiles;
  if (splits > slabs / 2) splits = slabs / 2;
  if (splits > a.splitk_floats / ((int64_t)a.m * a.n)) splits = a.splitk_floats / ((int64_t)a.m * a.n);
  if (splits < 1) splits = 1;
  const int per = (int)((slabs + splits - 1) / splits);
  p.k_per_split = per * BK;
  splits = (slabs + per - 1) / per;
  p.part = splits > 1 ? a.splitk_ws : nullptr;
  const dim3 grid((unsigned)(tiles * splits));
  if (a.trans) hipLaunchKernelGGL((k_fc<true>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((k_fc<false>), grid, dim3(256), 0, s, p);
  AE_TRY(launch_status("fc"));
  if (splits > 1) {
    const int64_t quads = (int64_t)a.m * a.n / 4;
    hipLaunchKernelGGL(k_fc_finish, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, (const float4*)p.part, (int)splits, quads, a.n / 4,
                       a.bias, a.act, (uint2*)a.y);
    AE_TRY(launch_status("fc_finish"));
  }
  return AE_OK;
}

}  // namespace ae
