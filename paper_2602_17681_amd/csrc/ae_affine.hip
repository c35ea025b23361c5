// ae_affine.hip — the LU parametrisation of a learnable invertible matrix (the paper's Section on learning
// affine transformations, Eq. 4):  A = P L (U + diag(s)),  L unit lower triangular, U strictly upper triangular,
// s = sign * exp(log_s) (the paper learns log|s| and keeps the signs), P a fixed permutation given as an index
// vector ((P M)[i] = M[perm[i]]); the gradients of the free parameters given dLoss/dA; and the volume regulariser
// in its practical form (sum_i log|s_i|)^2 (Eq. 6 and the paragraph after it).
//
// The three d x d x d products run on the matrix cores through the dense case of the implicit-GEMM kernel
// (y[m][n] = sum_k x[m][k] w[n][k], operands in the storage type, binary32 accumulation); small element-wise
// kernels materialise the triangular operands from the binary32 master parameters (transposed where the product
// needs it), apply the permutation to rows (of L (U + diag s) forward, of G backward), and cut the products back
// to the triangles the parameters live on.  Every product has a triangular operand and, backward, only a triangle
// of the result is wanted: the GEMM kernel walks only the K range of each tile that can hold non-zeros and skips
// the tiles nobody reads — a third of the multiply-adds of three dense products.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <mutex>
#include "ae_device.h"
#include "ae_internal.h"

namespace ae {
namespace {

struct LuSrc {
  const float* lp; const float* up; const float* log_s; const float* sign; const int* inv_perm; const void* g;
  int d;
};
enum { LU_L = 0, LU_UD = 1, LU_B = 2, LU_U = 3 };

// entry (r, c) of L, of U + diag(s), of B = P^T G (row r of B is row inv_perm[r] of G), or of U alone
template <typename T, int SRC>
__device__ __forceinline__ float lu_elem(const LuSrc& q, int r, int c) {
  if (SRC == LU_L) return c < r ? q.lp[(int64_t)r * q.d + c] : (c == r ? 1.0f : 0.0f);
  if (SRC == LU_UD) return r < c ? q.up[(int64_t)r * q.d + c] : (r == c ? q.sign[c] * expf(q.log_s[c]) : 0.0f);
  if (SRC == LU_U) return r < c ? q.up[(int64_t)r * q.d + c] : 0.0f;
  return Store<T>::ld(reinterpret_cast<const T*>(q.g) + (int64_t)q.inv_perm[r] * q.d + c);
}

// eight consecutive entries of one row, to and from the storage type
template <typename T> __device__ __forceinline__ void load8(const T* p, float (&v)[8]);
template <> __device__ __forceinline__ void load8<bf16_t>(const bf16_t* p, float (&v)[8]) { Store<bf16_t>::ldv(p, v); }
template <> __device__ __forceinline__ void load8<float>(const float* p, float (&v)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <typename T> __device__ __forceinline__ void store8(T* p, const float (&v)[8]);
template <> __device__ __forceinline__ void store8<bf16_t>(bf16_t* p, const float (&v)[8]) { Store<bf16_t>::stv(p, v); }
template <> __device__ __forceinline__ void store8<float>(float* p, const float (&v)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}

// out = the transpose of the matrix SRC in the storage type: 64 x 64 tiles through LDS, eight entries per lane on both
// sides; source chunks that lie wholly in the zero triangle read nothing.  d % 64 == 0.
template <typename T, int SRC>
__global__ __launch_bounds__(256) void k_lu_build_transposed(LuSrc q, T* __restrict__ out) {
  __shared__ float tile[64][65];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;           // output tile: rows r0.., columns c0..
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int chunk = threadIdx.x + 256 * j;
    const int sr = c0 + (chunk >> 3), sc0 = r0 + ((chunk & 7) << 3);   // source row (an output column), first source column
    float v[8];
    if (SRC == LU_B) {
      load8<T>(reinterpret_cast<const T*>(q.g) + (int64_t)q.inv_perm[sr] * q.d + sc0, v);
    } else if (SRC == LU_L ? sc0 + 7 < sr : sc0 > sr) {
      load8<float>((SRC == LU_L ? q.lp : q.up) + (int64_t)sr * q.d + sc0, v);
    } else if (SRC == LU_L ? sc0 > sr : sc0 + 7 < sr) {
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = 0.0f;
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = lu_elem<T, SRC>(q, sr, sc0 + t);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) tile[chunk >> 3][((chunk & 7) << 3) + t] = v[t];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int chunk = threadIdx.x + 256 * j;
    const int orow = chunk >> 3, oc0 = (chunk & 7) << 3;           // output row r0 + orow, columns c0 + oc0 ..
    float v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = tile[oc0 + t][orow];
    store8<T>(out + (int64_t)(r0 + orow) * q.d + c0 + oc0, v);
  }
}

// out = the matrix SRC (TR = false) or its transpose (TR = true), in the storage type; 32 x 32 tiles, d % 32 == 0
template <typename T, int SRC, bool TR>
__global__ __launch_bounds__(256) void k_lu_build(LuSrc q, T* __restrict__ out) {
  __shared__ float tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  if (!TR) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + ty + 8 * j;
      Store<T>::st(out + (int64_t)r * q.d + c0 + tx, lu_elem<T, SRC>(q, r, c0 + tx));
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) tile[ty + 8 * j][tx] = lu_elem<T, SRC>(q, c0 + ty + 8 * j, r0 + tx);   // source row c, column r
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) Store<T>::st(out + (int64_t)(r0 + ty + 8 * j) * q.d + c0 + tx, tile[tx][ty + 8 * j]);
  }
}

// out = the matrix SRC, row by row, eight entries per lane; chunks that lie wholly in the zero triangle read nothing
template <typename T, int SRC>
__global__ __launch_bounds__(256) void k_lu_build_rows(LuSrc q, T* __restrict__ out) {
  const int cpr = q.d >> 3;
  const int64_t n = (int64_t)q.d * cpr;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int r = (int)(i / cpr), c0 = (int)(i - (int64_t)r * cpr) << 3;
    float v[8];
    if (SRC == LU_B) {
      load8<T>(reinterpret_cast<const T*>(q.g) + (int64_t)q.inv_perm[r] * q.d + c0, v);
    } else if (SRC == LU_L ? c0 + 7 < r : c0 > r) {
      load8<float>((SRC == LU_L ? q.lp : q.up) + (int64_t)r * q.d + c0, v);       // wholly inside the used triangle
    } else if (SRC == LU_L ? c0 > r : c0 + 7 < r) {
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = 0.0f;
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = lu_elem<T, SRC>(q, r, c0 + t);           // the chunk that holds the diagonal
    }
    store8<T>(out + (int64_t)r * q.d + c0, v);
  }
}

// inv[i] = i, then inv[perm[i]] = i: entries of perm outside 0..d-1 are ignored, so every inv[r] stays inside 0..d-1 whatever
// perm holds.  One workgroup: d is at most 16 384, and a launch costs more.
__global__ __launch_bounds__(1024) void k_lu_invert_perm(const int* __restrict__ perm, int* __restrict__ inv, int d) {
  for (int i = threadIdx.x; i < d; i += 1024) inv[i] = i;
  __syncthreads();
#pragma unroll 4
  for (int i = threadIdx.x; i < d; i += 1024)
    if ((unsigned)perm[i] < (unsigned)d) inv[perm[i]] = i;
}

// A[i][:] = Y[perm[i]][:], 16 bytes per lane (row bytes are a multiple of 64)
__global__ __launch_bounds__(256) void k_lu_permute_rows(const uint4* __restrict__ y, const int* __restrict__ perm, int d,
                                                         int chunks_per_row, uint4* __restrict__ a) {
  const int64_t n = (int64_t)d * chunks_per_row;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int r = (int)(i / chunks_per_row), c = (int)(i - (int64_t)r * chunks_per_row);
    int src = perm[r];
    if ((unsigned)src >= (unsigned)d) src = r;                        // not a permutation: stay inside the arrays
    a[i] = y[(int64_t)src * chunks_per_row + c];
  }
}

// The same in binary32 with the diagonal's term of every entry: A[i][c] = Y[p][c] + L[p][c] s[c], p = perm[i], Y = L U.  That term is by
// far the largest of the results it enters, and the matrix cores round it at twice their last place: the largest deviation of
// A from float64 was 2.0e-6 of the root mean square at d = 256, 5.6e-6 at d = 1024 with it in the product (1.5e-6, 5.0e-6
// with the binary32 MFMA), 0.7e-6 and 2.2e-6 this way; the call took 52 and 368 us at d = 1024 and 4096, now 54 and 365.  Grid: 256 chunks of four columns by 16 rows.
// An entry that comes out as NaN is summed again over the triangles alone, up to the first NaN.
__global__ __launch_bounds__(256) void k_lu_permute_rows_diag(const float* __restrict__ y, const float* __restrict__ l, LuSrc q,
                                                              const int* __restrict__ perm, float* __restrict__ a) {
  const int c0 = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4, r0 = (int)blockIdx.y * 16, d = q.d;
  if (c0 >= d) return;
  float sv[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) sv[t] = q.sign[c0 + t] * expf(q.log_s[c0 + t]);
  for (int i = r0; i < min(r0 + 16, d); ++i) {
    int src = perm[i];
    if ((unsigned)src >= (unsigned)d) src = i;                        // not a permutation: stay inside the arrays
    const float4 w = *reinterpret_cast<const float4*>(y + (int64_t)src * d + c0);
    float v[4] = {w.x, w.y, w.z, w.w};
    if (c0 <= src) {                                                  // (L's zeros need not be read)
      const float4 x = *reinterpret_cast<const float4*>(l + (int64_t)src * d + c0);
      const float lv[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = c0 + t <= src ? fmaf(lv[t], sv[t], v[t]) : v[t];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (v[t] != v[t]) {
        const int c = c0 + t;
        v[t] = 0.0f;
        for (int k = 0; k < min(src + 1, c) && v[t] == v[t]; ++k) v[t] = fmaf(l[(int64_t)src * d + k], q.up[(int64_t)k * d + c], v[t]);
        if (c <= src) v[t] = fmaf(l[(int64_t)src * d + c], sv[t], v[t]);
      }
    *reinterpret_cast<float4*>(a + (int64_t)i * d + c0) = make_float4(v[0], v[1], v[2], v[3]);
  }
}

// d/dU = strictly upper part of L^T B, d/dlog_s = its diagonal times s  (tiles below the diagonal were never written:
// chunks wholly below it are not read)
template <typename T>
__global__ __launch_bounds__(256) void k_lu_grad_upper(const T* __restrict__ dud, const float* __restrict__ log_s,
                                                       const float* __restrict__ sign, int d, float* __restrict__ dup,
                                                       float* __restrict__ dlog_s) {
  const int cpr = d >> 3;
  const int64_t n = (int64_t)d * cpr;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int k = (int)(i / cpr), c0 = (int)(i - (int64_t)k * cpr) << 3;
    float v[8];
    if (c0 + 7 >= k) {
      load8<T>(dud + (int64_t)k * d + c0, v);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (c0 + t == k) dlog_s[k] = v[t] * (sign[k] * expf(log_s[k]));
        if (c0 + t <= k) v[t] = 0.0f;
      }
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = 0.0f;
    }
    store8<float>(dup + (int64_t)k * d + c0, v);
  }
}

// d/dL = strictly lower part of B (U + diag s)^T  (tiles above the diagonal were never written: not read)
template <typename T>
__global__ __launch_bounds__(256) void k_lu_grad_lower(const T* __restrict__ dl, int d, float* __restrict__ dlp) {
  const int cpr = d >> 3;
  const int64_t n = (int64_t)d * cpr;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int r = (int)(i / cpr), c0 = (int)(i - (int64_t)r * cpr) << 3;
    float v[8];
    if (c0 < r) {
      load8<T>(dl + (int64_t)r * d + c0, v);
#pragma unroll
      for (int t = 0; t < 8; ++t) if (c0 + t >= r) v[t] = 0.0f;
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = 0.0f;
    }
    store8<float>(dlp + (int64_t)r * d + c0, v);
  }
}

// (sum_i log|s_i|)^2 and its gradient 2 sum, one workgroup, fixed order
__global__ __launch_bounds__(256) void k_vol_penalty(const float* __restrict__ log_s, int d, float* __restrict__ value,
                                                     float* __restrict__ grad) {
  __shared__ double sm[256 / 64 + 1];
  __shared__ float total;
  double acc = 0.0;
#pragma unroll 16
  for (int i = threadIdx.x; i < d; i += 256) acc += (double)log_s[i];      // (sixteen loads in flight: 4 096 entries 8 -> 4.8 us)
  acc = block_sum<256>(acc, sm);
  if (threadIdx.x == 0) { total = (float)acc; *value = (float)(acc * acc); }
  __syncthreads();
  if (grad) for (int i = threadIdx.x; i < d; i += 256) grad[i] = 2.0f * total;
}

template <typename T, int SRC, bool TR>
void launch_build(const LuSrc& q, void* out, hipStream_t s) {
  hipLaunchKernelGGL((k_lu_build<T, SRC, TR>), dim3(q.d / 32, q.d / 32), dim3(256), 0, s, q, reinterpret_cast<T*>(out));
}

// ---- inverse of the parametrised matrix ---------------------------------------------------------------------
// A^-1 = (U + diag s)^-1 L^-1 P^T.  Both triangular inverses are blocked recursions: 128 x 128 diagonal blocks are inverted by
// substitution, then neighbouring inverses X11, X22 of blocks of size b merge into the inverse of the 2b x 2b block,
//     L:  [[X11, 0], [-X22 L21 X11, X22]],      U:  [[X11, -X11 U12 X22], [0, X22]].
// X and X^T live as full d x d binary32 matrices whose diagonal blocks come first and which fill level by level (the other
// triangle is never written and never read: every product starts or ends its K range at the tile's own rows).  The product kernel
// computes x w^T, and the parameters themselves are what it wants as w, so that a level is two launches over ALL pairs of both factors:
//     L:  T = X11^T L21^T = (L21 X11)^T,  X21 = -X22 T^T;      U:  T = X22^T U12^T = (U12 X22)^T,  X12 = -X11 T^T;
// the second writes its block into X and the transpose into X^T.

// ---- many small matrices at once (the per-block transformations: one d x d parameter set per transformer block, d the
// head dimension) --------------------------------------------------------------------------------------------------
// For d <= 128 a matrix fits into LDS, and the full-size path above would be a dozen launch-bound kernels per matrix; one
// launch covers `count` of them.  A product of 128 x 128 matrices is microseconds of the binary32 MFMA, so what counts is
// that a handful of matrices (32 blocks of a model) still spreads over the chip and that no thread waits for one load at a
// time: a workgroup of eight wavefronts owns 32 rows of one product (four workgroups per matrix composing, eight backward), a
// wavefront two 16 x 16 tiles of them, and all loads of its operands, of 16 bytes, are in flight at once.  Code that runs once per
// launch is paid for by the KiB, so what only odd alignments, infinities or NaN reach is kept in rolled loops.  Measured for
// 32 (512) matrices of 128, bfloat16 in and out: four wavefronts of one 32 x 32 tile, operands one after the other, 11.1 (88) us composing
// and 13.9 (240) backward; this way 10.7 (66) and 11.3 (168).
// LDS rows are 132 floats: the 16-byte fragment reads of 16 rows and the 4-byte ones of two rows fall into different banks.
constexpr int kSmallLd = 132;

__device__ __forceinline__ LuSrc small_src(const float* lp, const float* up, const float* log_s, const float* sign_s, int d, int m) {
  const int64_t mo = (int64_t)m * d * d, vo = (int64_t)m * d;
  return LuSrc{lp + mo, up + mo, log_s + vo, sign_s + vo, nullptr, nullptr, d};
}
__device__ __forceinline__ int small_perm(const int* perm, int d, int i) {       // an entry out of range is treated as i
  const int p = perm[i];
  return (unsigned)p < (unsigned)d ? p : i;
}

// four consecutive entries of row r (c0 % 4 == 0), zeros past column d; vec: the rows allow one wide load
template <typename T>
__device__ __forceinline__ float4 small_load4(const T* m, int d, int r, int c0, bool vec) {
  const T* p = m + (int64_t)r * d + c0;
  if (vec) {
    if constexpr (sizeof(T) == 4) return *reinterpret_cast<const float4*>(p);
    const uint2 w = *reinterpret_cast<const uint2*>(p);
    return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u));
  }
  return make_float4(Store<T>::ld(p), c0 + 1 < d ? Store<T>::ld(p + 1) : 0.0f, c0 + 2 < d ? Store<T>::ld(p + 2) : 0.0f, c0 + 3 < d ? Store<T>::ld(p + 3) : 0.0f);
}
template <typename T> __device__ __forceinline__ bool small_vec(const T* p, int d) { return d % 4 == 0 && ((uintptr_t)p % (4 * sizeof(T))) == 0; }

// dst[i][c] for i < rows, c < cols (both multiples of 4), dst rows of kSmallLd: entry (src_row(i), c0 + c) of src, passed through
// fix(value, i, c); a negative row, or one past the matrix, reads zeros.  All threads of the workgroup, N loads of 16 bytes each;
// load() and store() apart, so that the loads of all operands are in flight together (rows that allow no wide loads: all in store()).
template <typename T, int N>
struct SmallStage {
  const T* src;
  int rows, q, d, c0;
  bool vec;
  float4 v[N];
  __device__ __forceinline__ SmallStage(const T* src_, int rows_, int cols, int d_, int c0_) : src(src_), rows(rows_), q(cols >> 2), d(d_), c0(c0_), vec(small_vec(src_, d_)) {}
  template <typename ROW>
  __device__ __forceinline__ float4 get(int e, ROW src_row, bool wide) const {
    const int i = e / q, c = (e - i * q) * 4, r = e < rows * q ? src_row(i) : -1;
    return r >= 0 && r < d && c0 + c < d ? small_load4<T>(src, d, r, c0 + c, wide) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
  template <typename FIX>
  __device__ __forceinline__ void put(float* dst, int e, const float4& w, FIX fix) const {
    const int i = e / q, c = (e - i * q) * 4;
    if (e < rows * q) *reinterpret_cast<float4*>(dst + i * kSmallLd + c) = make_float4(fix(w.x, i, c), fix(w.y, i, c + 1), fix(w.z, i, c + 2), fix(w.w, i, c + 3));
  }
  template <typename ROW>
  __device__ __forceinline__ void load(ROW src_row) {
    if (!vec) return;
#pragma unroll
    for (int t = 0; t < N; ++t) v[t] = get((int)threadIdx.x + t * 512, src_row, true);
  }
  template <typename ROW, typename FIX>
  __device__ __forceinline__ void store(float* dst, ROW src_row, FIX fix) const {
    if (vec) {
#pragma unroll
      for (int t = 0; t < N; ++t) put(dst, (int)threadIdx.x + t * 512, v[t], fix);
    } else {
#pragma unroll 1
      for (int e = threadIdx.x; e < rows * q; e += 512) put(dst, e, get(e, src_row, false), fix);
    }
  }
};

// c += the product over k = k0 .. k1 - 1 on tiles of 16 x 16, two of them side by side (columns lane % 16 and 16 on): a(k, v), b(k, h, v) give this lane's operands for
// the k's k + 8 (lane / 16) + 0 .. 7 (element e of a lane: row 4 (lane / 16) + e); k0 and k1 are multiples of 32.
typedef float floatx4 __attribute__((ext_vector_type(4)));
template <typename A, typename B>
__device__ __forceinline__ void small_mma16(floatx4 (&c)[2], int k0, int k1, A a, B b) {
  floatx4 s[4][2] = {};                                  // four partial sums (errors of 32 x 128^2 composed: 5.39e-8 with two, 4.81e-8 with four)
#pragma unroll 1
  for (int k = k0; k < k1; k += 32) {
    float av[8], bv[2][8];
    a(k, av);
    b(k, 0, bv[0]);
    b(k, 1, bv[1]);
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) s[t & 3][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t], bv[h][t], s[t & 3][h], 0, 0, 0);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) c[h] += (s[0][h] + s[1][h]) + (s[2][h] + s[3][h]);
}
// sums that are NaN replaced by value(e): a zero of a triangle meets an infinity in a tile's K range, where the sum over the
// triangle alone need not be NaN (nothing but infinities and NaN gets there; one fused multiply-add per sum otherwise)
template <typename V, typename VALUE>
__device__ __forceinline__ void small_resum_nan(V& c, VALUE value) {
  constexpr int N = (int)(sizeof(V) / sizeof(float));
  float z = 0.0f;
#pragma unroll
  for (int e = 0; e < N; ++e) z = fmaf(c[e], 0.0f, z);
  if (z == 0.0f) return;
  unsigned bits = 0;
#pragma unroll
  for (int e = 0; e < N; ++e) bits |= (unsigned)(c[e] != c[e]) << e;
  while (bits != 0) {
    const int t = __ffs(bits) - 1;
    bits &= bits - 1;
    const float v = value(t);
#pragma unroll
    for (int e = 0; e < N; ++e) c[e] = e == t ? v : c[e];
  }
}
// operands in LDS: eight k's of one row, or one column of eight rows
__device__ __forceinline__ void small_row8(const float* p, float (&v)[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float4 f = *reinterpret_cast<const float4*>(p + 4 * h);
    v[4 * h] = f.x; v[4 * h + 1] = f.y; v[4 * h + 2] = f.z; v[4 * h + 3] = f.w;
  }
}
__device__ __forceinline__ void small_col8(const float* p, float (&v)[8]) {
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] = p[t * kSmallLd];
}

// out[r][j] = sum_k L[perm[r]][k] (U + diag s)[k][j]: workgroup (m, rb) has rows 32 rb .. of matrix m, wavefront w 16 of them (w / 4)
// and columns 32 (w % 4) ..
template <typename T>
__global__ __launch_bounds__(512) void k_lu_small_compose(const float* __restrict__ lp, const float* __restrict__ up, const float* __restrict__ log_s,
                                                          const float* __restrict__ sign_s, const int* __restrict__ perm, int d, T* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) float lm[32 * kSmallLd];
  __shared__ __attribute__((aligned(16))) float um[128 * kSmallLd];
  __shared__ int pr[32];
  __shared__ float dg[128];
  const int nb = (d + 31) >> 5, dp = nb * 32, m = blockIdx.x / nb, rb = blockIdx.x - m * nb, tid = threadIdx.x;
  const LuSrc q = small_src(lp, up, log_s, sign_s, d, m);
  SmallStage<float, 8> su(q.up, dp, dp, d, 0);
  SmallStage<float, 2> sl(q.lp, 32, dp, d, 0);
  auto row_u = [](int i) { return i; };
  auto row_l = [&](int i) { return pr[i]; };
  if (tid < 32) pr[tid] = rb * 32 + tid < d ? small_perm(perm + (int64_t)m * d, d, rb * 32 + tid) : -1;
  if (tid < 128) dg[tid] = tid < d ? q.sign[tid] * expf(q.log_s[tid]) : 0.0f;
  su.load(row_u);
  __syncthreads();
  sl.load(row_l);
  su.store(um, row_u, [](float v, int i, int c) { return c > i ? v : 0.0f; });
  sl.store(lm, row_l, [&](float v, int i, int c) { return c < pr[i] ? v : (c == pr[i] ? 1.0f : 0.0f); });
  __syncthreads();
  const int wave = tid >> 6, lane = tid & 63, j = wave & 3, r0 = (wave >> 2) * 16, lc = lane & 15, g = lane >> 4, col = j * 32 + lc;
  if (j >= nb) return;
  const float* const lrow = lm + (r0 + 4 * g) * kSmallLd;          // of this lane's four rows of results
  floatx4 acc[2] = {};
  // (below 64 the few terms of a sum come out closer to float64 when they are added one by one with fused multiply-adds:
  // 2-norm 3.9e-8 against 4.3e-8 at d = 24, but 6.1e-8 against 5.6e-8 at d = 128)
  if (d < 64) {
    for (int k = 0; k < 32 * (j + 1); ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float b = um[k * kSmallLd + col + 16 * h];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[h][e] = fmaf(lrow[e * kSmallLd + k], b, acc[h][e]);
      }
  } else
    small_mma16(acc, 0, 32 * (j + 1), [&](int k, float (&v)[8]) { small_row8(lm + (r0 + lc) * kSmallLd + k + 8 * g, v); },
                [&](int k, int h, float (&v)[8]) { small_col8(um + (k + 8 * g) * kSmallLd + col + 16 * h, v); });
  // The term with the diagonal of U + diag s, by far the largest of a result of which it is one, last and in a fused multiply-add: the
  // binary32 MFMA rounds at twice the last place (largest deviation over 24 matrices of 128: 1.6e-6 of the root mean square with it
  // in the product, 0.8e-6 this way, 1.0e-6 one by one; 2-norm 5.3e-8, 4.7e-8, 5.7e-8)
  T* const o = out + (int64_t)m * d * d;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = col + 16 * h;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[h][e] = fmaf(lrow[e * kSmallLd + c], dg[c], acc[h][e]);
    small_resum_nan(acc[h], [&](int e) {
      const float* const l = lrow + e * kSmallLd;
      const int p = pr[r0 + 4 * g + e];
      float v = 0.0f;
      for (int t = 0; t <= p && t < c; ++t) v = fmaf(l[t], um[t * kSmallLd + c], v);
      return c <= p ? fmaf(l[c], dg[c], v) : v;
    });
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = rb * 32 + r0 + 4 * g + e;
      if (r < d && c < d) Store<T>::st(o + (int64_t)r * d + c, acc[h][e]);
    }
  }
}

// B = P^T G (B[perm[i]] = G[i], zero rows where perm names none);  d_up = strictly upper part of L^T B, d_log_s = its diagonal
// times s, d_lp = strictly lower part of B (U + diag s)^T.  Workgroup (m, w): w < nb rows 32 w .. of the first product, else rows
// 32 (w - nb) .. of the second; wavefronts as in k_lu_small_compose
template <typename T>
__global__ __launch_bounds__(512) void k_lu_small_backward(const T* __restrict__ g, const float* __restrict__ lp, const float* __restrict__ up,
                                                           const float* __restrict__ log_s, const float* __restrict__ sign_s, const int* __restrict__ perm,
                                                           int d, float* __restrict__ d_lp, float* __restrict__ d_up, float* __restrict__ d_log_s) {
  __shared__ __attribute__((aligned(16))) float thin[128 * kSmallLd];   // 32 columns of L, or 32 rows of B
  __shared__ __attribute__((aligned(16))) float wide[128 * kSmallLd];   // B, or U + diag s
  __shared__ int inv[128];
  __shared__ float dg[128];
  const int nb = (d + 31) >> 5, dp = nb * 32, m = blockIdx.x / (2 * nb), w = blockIdx.x - m * 2 * nb, tid = threadIdx.x;
  const int64_t mo = (int64_t)m * d * d, vo = (int64_t)m * d;
  const LuSrc q = small_src(lp, up, log_s, sign_s, d, m);
  const bool first = w < nb;
  const int r0 = (first ? w : w - nb) * 32;
  // (the operand that needs no permutation is asked for before the permutation is)
  SmallStage<float, 8> sp(first ? q.lp : q.up, first ? dp - r0 : r0 + 32, first ? 32 : dp, d, first ? r0 : 0);
  SmallStage<T, 8> sb(g + mo, first ? dp - r0 : 32, first ? dp - r0 : dp, d, first ? r0 : 0);
  auto row_p = [&](int i) { return first ? r0 + i : i; };
  auto row_b = [&](int i) { return r0 + i < d ? inv[r0 + i] : -1; };
  sp.load(row_p);
  if (tid < 128) inv[tid] = -1;
  if (tid < d) dg[tid] = q.sign[tid] * expf(q.log_s[tid]);
  const int pv = tid < d ? small_perm(perm + vo, d, tid) : 0;
  __syncthreads();
  if (tid < d) inv[pv] = tid;
  __syncthreads();
  sb.load(row_b);
  if (first)
    sp.store(thin, row_p, [&](float v, int i, int c) { return c < i ? v : (c == i && r0 + i < d ? 1.0f : 0.0f); });
  else
    sp.store(wide, row_p, [&](float v, int i, int c) { return c > i ? v : (c == i && i < d ? dg[i] : 0.0f); });
  sb.store(first ? wide : thin, row_b, [](float v, int, int) { return v; });
  __syncthreads();
  const int wave = tid >> 6, lane = tid & 63, j = wave & 3, rw = (wave >> 2) * 16, lc = lane & 15, g8 = (lane >> 4) * 8, col = j * 32 + lc;
  if (j >= nb) return;
  floatx4 acc[2] = {};
  if (first) {                                           // (L^T B)[k][n] = sum over i >= k of L[i][k] B[i][n], n >= k
    if (j >= w)
      small_mma16(acc, 0, dp - r0, [&](int k, float (&v)[8]) { small_col8(thin + (k + g8) * kSmallLd + rw + lc, v); },
                  [&](int k, int h, float (&v)[8]) { small_col8(wide + (k + g8) * kSmallLd + col - r0 + 16 * h, v); });
  } else if (j * 32 <= r0) {                             // (B (U + diag s)^T)[r][k] = sum over n >= k of B[r][n] (U + diag s)[k][n], k < r
    small_mma16(acc, j * 32, dp, [&](int k, float (&v)[8]) { small_row8(thin + (rw + lc) * kSmallLd + k + g8, v); },
                [&](int k, int h, float (&v)[8]) { small_row8(wide + (col + 16 * h) * kSmallLd + k + g8, v); });
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = r0 + rw + 4 * (lane >> 4) + e, c = col + 16 * h;
      if (r >= d || c >= d) continue;
      if (first) {
        d_up[mo + (int64_t)r * d + c] = c > r ? acc[h][e] : 0.0f;
        if (c == r) d_log_s[vo + r] = acc[h][e] * dg[r];
      } else {
        d_lp[mo + (int64_t)r * d + c] = c < r ? acc[h][e] : 0.0f;
      }
    }
}

// Both triangular factors of one matrix in LDS at once, inverted in place by four wavefronts each: entry (i, j), j <= i, of L is
// p[129 i + j], of (U + diag s)^T p[129 j + i + 1] — U as it lies in memory, one column to the right.
struct SmallTri {
  float* p;
  int si, sj;                     // strides of i and j
  __device__ __forceinline__ float& at(int i, int j) const { return p[i * si + j * sj]; }
};

// the 16 x 16 diagonal blocks by substitution: thread tid < 128 has column tid, in registers; all 256 threads of the factor call
__device__ __forceinline__ void small_tri_diag(const SmallTri& x, int tid) {
  float col[16];
  const int b0 = tid & ~15, jj = tid & 15;
  if (tid < 128) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float acc = 0.0f;                                // (from row jj on: a zero above it may meet an infinity)
#pragma unroll
      for (int k = 0; k < i; ++k) { const float t = fmaf(x.at(b0 + i, b0 + k), col[k], acc); acc = k >= jj ? t : acc; }
      col[i] = (i == jj ? 1.0f : -acc) / x.at(b0 + i, b0 + i);
      if (i < jj) col[i] = 0.0f;
    }
  }
  __syncthreads();
  if (tid < 128) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i >= jj) x.at(b0 + i, b0 + jj) = col[i];
  }
  __syncthreads();
}

// one merge level of one factor in place, all pairs of neighbouring B x B diagonal blocks: X21 = -X22 (M21 X11) over M21; 256
// threads (tid), tb: 64 * 68 floats.  Blocks of 16 on the vector ALUs; blocks of 32 and 64 on the matrix cores, a wavefront per 32 x 32 tile.
__device__ __forceinline__ void small_tri_merge16(const SmallTri& x, float* tb, int tid) {
  const int pr = tid >> 6, t = tid & 63, tr = t >> 3, tc = t & 7, o0 = 32 * pr, o1 = o0 + 16;
  float* tp = tb + pr * 256;
  float acc[2][2] = {};
  if (tid >= 256) {                                    // (whole wavefronts, where one factor has 512 threads)
    __syncthreads();
    __syncthreads();
    return;
  }
#pragma unroll
  for (int k = 0; k < 16; ++k)                         // T = M21 X11:  X11[k][c] = 0 for k < c
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float v = k >= tc + 8 * j ? x.at(o0 + k, o0 + tc + 8 * j) : 0.0f;
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i][j] = fmaf(x.at(o1 + tr + 8 * i, o0 + k), v, acc[i][j]);
    }
  // (as small_resum_nan: a zero of a triangle may have met an infinity)
  auto odd = [&]() { return fmaf(acc[0][0], 0.0f, fmaf(acc[0][1], 0.0f, fmaf(acc[1][0], 0.0f, acc[1][1] * 0.0f))) != 0.0f; };
  if (odd()) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        acc[i][j] = 0.0f;
        for (int k = tc + 8 * j; k < 16; ++k) acc[i][j] = fmaf(x.at(o1 + tr + 8 * i, o0 + k), x.at(o0 + k, o0 + tc + 8 * j), acc[i][j]);
      }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      tp[(tr + 8 * i) * 16 + tc + 8 * j] = acc[i][j];
      acc[i][j] = 0.0f;
    }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k)                         // X21 = -X22 T:  X22[r][k] = 0 for k > r
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float a = k <= tr + 8 * i ? x.at(o1 + tr + 8 * i, o1 + k) : 0.0f;
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = fmaf(a, tp[k * 16 + tc + 8 * j], acc[i][j]);
    }
  if (odd()) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        acc[i][j] = 0.0f;
        for (int k = 0; k <= tr + 8 * i; ++k) acc[i][j] = fmaf(x.at(o1 + tr + 8 * i, o1 + k), tp[k * 16 + tc + 8 * j], acc[i][j]);
      }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) x.at(o1 + tr + 8 * i, o0 + tc + 8 * j) = -acc[i][j];   // (M21 was last read before the barrier)
  __syncthreads();
}
// (eight wavefronts: one or two 16 x 16 tiles each, as small_mma16)
template <int B>
__device__ __forceinline__ void small_tri_merge(const SmallTri& x, float* tb, int tid) {
  constexpr int NT = B / 32, LT = B + 4, COLS = B / (16 * NT), TASKS = B / 16 * COLS;   // tiles per wavefront; row length of T; wavefronts per row of tiles, per pair
  static_assert(TASKS * (64 / B) == 8, "one task each");
  const int w = tid >> 6, lane = tid & 63, lc = lane & 15, g8 = (lane >> 4) * 8, pr = w / TASKS, t = w % TASKS;
  const int o0 = 2 * pr * B, o1 = o0 + B, r0 = t / COLS * 16, c0 = t % COLS * 16 * NT;
  float* const tp = tb + pr * (B * LT);
  auto product = [&](floatx4 (&c)[NT], int k0, int k1, auto a, auto b) {
    floatx4 s[4][NT] = {};
#pragma unroll 1
    for (int k = k0; k < k1; k += 32) {
      float av[8], bv[NT][8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        av[u] = a(k + g8 + u);
#pragma unroll
        for (int h = 0; h < NT; ++h) bv[h][u] = b(k + g8 + u, c0 + 16 * h + lc);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int h = 0; h < NT; ++h) s[u & 3][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[h][u], s[u & 3][h], 0, 0, 0);
    }
#pragma unroll
    for (int h = 0; h < NT; ++h) c[h] = (s[0][h] + s[1][h]) + (s[2][h] + s[3][h]);
  };
  floatx4 acc[NT];
  product(acc, c0 & ~31, B, [&](int k) { return x.at(o1 + r0 + lc, o0 + k); },   // T = M21 X11:  X11[k][c] = 0 for k < c
          [&](int k, int c) { const float u = x.at(o0 + k, o0 + c); return k >= c ? u : 0.0f; });
#pragma unroll
  for (int h = 0; h < NT; ++h) {
    const int c = c0 + 16 * h + lc;
    small_resum_nan(acc[h], [&](int e) {
      float v = 0.0f;
      for (int k = c; k < B; ++k) v = fmaf(x.at(o1 + r0 + 4 * (lane >> 4) + e, o0 + k), x.at(o0 + k, o0 + c), v);
      return v;
    });
#pragma unroll
    for (int e = 0; e < 4; ++e) tp[(r0 + 4 * (lane >> 4) + e) * LT + c] = acc[h][e];
  }
  __syncthreads();
  product(acc, 0, (r0 & ~31) + 32, [&](int k) { const float u = x.at(o1 + r0 + lc, o1 + k); return k <= r0 + lc ? u : 0.0f; },   // X21 = -X22 T:  X22[r][k] = 0 for k > r
          [&](int k, int c) { return tp[k * LT + c]; });
#pragma unroll
  for (int h = 0; h < NT; ++h) {
    const int c = c0 + 16 * h + lc;
    small_resum_nan(acc[h], [&](int e) {
      const int row = r0 + 4 * (lane >> 4) + e;
      float v = 0.0f;
      for (int k = 0; k <= row; ++k) v = fmaf(x.at(o1 + row, o1 + k), tp[k * LT + c], v);
      return v;
    });
#pragma unroll
    for (int e = 0; e < 4; ++e) x.at(o1 + r0 + 4 * (lane >> 4) + e, o0 + c) = -acc[h][e];   // (M21 was last read before the barrier)
  }
  __syncthreads();
}

// The same, NC x 32 columns of one matrix per workgroup: out[:, c] = (U + diag s)^-1 L^-1 e_perm[c] by block substitution.  What bounds
// the call for a few matrices is the chain of dependent steps of one workgroup on a chip that is nearly empty; the columns of a
// result are independent, and substitution needs the inverses of the 32 x 32 diagonal blocks only, which every workgroup forms for
// itself (16 x 16 blocks, one merge).  Per block two steps of one 32 x 32 x 32 product each on 16 x 16 tiles, a wavefront per tile:
// the block's inverse times its rows, then the rows of the blocks behind.  32 matrices of 128 in bf16: 30.8 us with both triangles inverted
// and multiplied in one workgroup per matrix, 17.9 this way; 512 of them 64 and 59.  2-norm error against float64 1.75e-7 and 1.40e-7.
template <typename T, int NC>
__global__ __launch_bounds__(512) void k_lu_small_solve(const float* __restrict__ lp, const float* __restrict__ up, const float* __restrict__ log_s,
                                                        const float* __restrict__ sign_s, const int* __restrict__ perm, int d, T* __restrict__ out) {
  constexpr int LY = 32 * NC + 2;                        // (eight rows on, sixteen banks on: the four lane groups of a read do not meet)
  __shared__ float pk[128 * 129];
  // right-hand sides and solution of the one factor, in turn; four blocks of columns have room for one of them: a wavefront then has
  // all rows of its columns, and its reads lie before its writes
  constexpr int RT = NC == 4 ? 2 : 1;                    // row tiles per wavefront where the block's inverse is applied
  __shared__ float y[128 * LY], zs[NC == 4 ? 2048 : 128 * LY];
  float* const z = NC == 4 ? y : zs;
  __shared__ int pc[32 * NC];
  const int nb = (d + 31) >> 5, parts = (nb + NC - 1) / NC, m = blockIdx.x / parts, c0 = (blockIdx.x - m * parts) * 32 * NC, tid = threadIdx.x;
  const LuSrc q = small_src(lp, up, log_s, sign_s, d, m);
  const bool vl = small_vec(q.lp, d), vu = small_vec(q.up, d);
  auto put = [&](int i, int c, const float4& l, const float4& u) {
    const float lv[4] = {l.x, l.y, l.z, l.w}, uv[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (c + s != i) pk[i * 129 + c + s + (c + s > i)] = c + s < i ? lv[s] : uv[s];
  };
  const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float4 l[8], u[8];                                     // 128 x 32 chunks of four columns: eight per thread and factor, all in flight
  if (vl && vu) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = tid + t * 512, i = e >> 5, c = (e & 31) * 4;
      const bool in = i < d && c < d;
      l[t] = in && c < i ? small_load4<float>(q.lp, d, i, c, true) : zero;
      u[t] = in && c + 3 > i ? small_load4<float>(q.up, d, i, c, true) : zero;
    }
  }
  const float dv = tid < d ? q.sign[tid] * expf(q.log_s[tid]) : 1.0f;
  if (tid < 32 * NC) pc[tid] = c0 + tid < d ? small_perm(perm + (int64_t)m * d, d, c0 + tid) : -1;
  for (int e = tid; e < 128 * LY; e += 512) y[e] = 0.0f;
  if (vl && vu) {
#pragma unroll
    for (int t = 0; t < 8; ++t) put((tid + t * 512) >> 5, (tid & 31) * 4, l[t], u[t]);
  } else {
#pragma unroll 1
    for (int e = tid; e < 4096; e += 512) {
      const int i = e >> 5, c = (e & 31) * 4;
      const bool in = i < d && c < d;
      put(i, c, in && c < i ? small_load4<float>(q.lp, d, i, c, false) : zero, in && c + 3 > i ? small_load4<float>(q.up, d, i, c, false) : zero);
    }
  }
  if (tid < 128) {
    pk[tid * 129 + tid] = 1.0f;
    pk[tid * 129 + tid + 1] = dv;
  }
  __syncthreads();
  if (tid < 32 * NC && pc[tid] >= 0) y[pc[tid] * LY + tid] = 1.0f;
  const int f = tid >> 8, ft = tid & 255;
  const SmallTri x = f == 0 ? SmallTri{pk, 129, 1} : SmallTri{pk + 1, 1, 129};
  small_tri_diag(x, ft);                                 // (barriers inside)
  if (d > 16) small_tri_merge16(x, zs + f * 1024, ft);
  const int wave = tid >> 6, lane = tid & 63, lc = lane & 15, g8 = (lane >> 4) * 8;
  // a 16 x 16 tile of the product of 32 columns k of a (entry (row, k)) and rows k of b, b's columns from cc on (rows_of): element e of
  // a lane is row 4 (lane / 16) + e, column lane % 16
  float bv[8];
  auto rows_of = [&](const float* b, int cc) {           // the rows' part of this wavefront
#pragma unroll
    for (int t = 0; t < 8; ++t) bv[t] = b[(g8 + t) * LY + cc + lc];
  };
  auto product = [&](auto a) {
    float av[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) av[t] = a(lc, g8 + t);
    floatx4 c = {}, c2 = {};                             // (two partial sums)
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t], bv[t], c, 0, 0, 0);
      c2 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t + 1], bv[t + 1], c2, 0, 0, 0);
    }
    return c + c2;
  };
  constexpr int G = 4 / NC;                              // wavefronts per 16 columns; one alone waits for nobody, ...
  const int cc = wave / G * 16, g = wave % G;
  // ... but its lanes read what others of them have written: LDS serves a wavefront in order, and this keeps the compiler to it
  auto wave_sync = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto sync = [&]() { if constexpr (G > 1) __syncthreads(); else wave_sync(); };
  auto sync_same = [&]() { if constexpr (NC == 4) wave_sync(); };  // where y is z: rows that all lanes have read are overwritten
  // (a zero outside a triangle, or above the one of a column, may have met an infinity: NaN is summed again over k = first .. last(row))
  auto resum = [&](floatx4& c, auto a, const float* b, auto first, auto last) {
    if (fmaf(c[0], 0.0f, fmaf(c[1], 0.0f, fmaf(c[2], 0.0f, c[3] * 0.0f))) == 0.0f) return;
#pragma unroll 1
    for (int e = 0; e < 4; ++e) {
      const int row = 4 * (lane >> 4) + e;
      const float w = e < 2 ? (e == 0 ? c[0] : c[1]) : (e == 2 ? c[2] : c[3]);
      float v = 0.0f;
      if (w == w) continue;
      for (int k = first(row); k <= last(row); ++k) v = fmaf(a(row, k), b[k * LY + cc + lc], v);
      c[0] = e == 0 ? v : c[0]; c[1] = e == 1 ? v : c[1]; c[2] = e == 2 ? v : c[2]; c[3] = e == 3 ? v : c[3];
    }
  };
  for (int i = 0; i < nb; ++i) {                         // L z = y
    const int o = i * 32;
    if (g < 2) {
      floatx4 c[RT];
      rows_of(y + o * LY, cc);
#pragma unroll
      for (int h = 0; h < RT; ++h) {
        const int r = 16 * (g + h);
        auto a = [&](int row, int k) { const float v = pk[(o + r + row) * 129 + o + k]; return k <= r + row ? v : 0.0f; };
        c[h] = product(a);
        resum(c[h], a, y + o * LY, [&](int) { return max(pc[cc + lc] - o, 0); }, [&](int row) { return r + row; });
      }
      sync_same();
#pragma unroll
      for (int h = 0; h < RT; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) z[(o + 16 * (g + h) + 4 * (lane >> 4) + e) * LY + cc + lc] = c[h][e];
    }
    sync();
    rows_of(z + o * LY, cc);
#pragma unroll 2
    for (int t = g; t < (nb - 1 - i) * 2; t += G) {
      const int r = o + 32 + t * 16;
      auto a = [&](int row, int k) { return pk[(r + row) * 129 + o + k]; };
      floatx4 c = product(a);
      resum(c, a, z + o * LY, [&](int) { return max(pc[cc + lc] - o, 0); }, [](int) { return 31; });
#pragma unroll
      for (int e = 0; e < 4; ++e) y[(r + 4 * (lane >> 4) + e) * LY + cc + lc] -= c[e];
    }
    sync();
  }
  T* const om = out + (int64_t)m * d * d;
  for (int i = nb - 1; i >= 0; --i) {                    // (U + diag s) y = z
    const int o = i * 32;
    if (g < 2) {
      floatx4 c[RT];
      rows_of(z + o * LY, cc);
#pragma unroll
      for (int h = 0; h < RT; ++h) {
        const int r = 16 * (g + h);
        auto a = [&](int row, int k) { const float v = pk[(o + r + row) * 129 + o + k + 1]; return k >= r + row ? v : 0.0f; };
        c[h] = product(a);
        resum(c[h], a, z + o * LY, [&](int row) { return r + row; }, [](int) { return 31; });
      }
      sync_same();
#pragma unroll
      for (int h = 0; h < RT; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = o + 16 * (g + h) + 4 * (lane >> 4) + e, col = c0 + cc + lc;
          y[row * LY + cc + lc] = c[h][e];
          if (row < d && col < d) Store<T>::st(om + (int64_t)row * d + col, c[h][e]);
        }
    }
    sync();
    rows_of(y + o * LY, cc);
#pragma unroll 2
    for (int t = g; t < i * 2; t += G) {
      const int r = t * 16;
      const floatx4 c = product([&](int row, int k) { return pk[(r + row) * 129 + o + k + 1]; });
#pragma unroll
      for (int e = 0; e < 4; ++e) z[(r + 4 * (lane >> 4) + e) * LY + cc + lc] -= c[e];
    }
    sync();
  }
}

// X_bb = M_bb^-1 for every 128 x 128 diagonal block b of M = L (which 0) or (U + diag s)^T (1) (one workgroup of 512 threads
// each; blockIdx.y + first: which), inverted in place in LDS as above; the block and its transpose are written into the full
// matrices lo (lower triangular) and hi of the factor.
struct TriOut { float* lo; float* hi; };
__global__ __launch_bounds__(512) void k_tri_diag_inverse(LuSrc q, int dp, int first, TriOut l, TriOut u) {
  __shared__ float pk[128 * 129];
  __shared__ float tb[64 * 68];
  const int tid = threadIdx.x, o = blockIdx.x * 128, which = first + (int)blockIdx.y;
  const float* src = which == 0 ? q.lp : q.up;
  const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  auto get = [&](int e, bool wide) {                     // 128 x 32 chunks of four columns
    const int i = e >> 5, c = (e & 31) * 4;
    const bool in = o + i < q.d && o + c < q.d && (which == 0 ? c < i : c + 3 > i);
    return in ? small_load4<float>(src, q.d, o + i, o + c, wide) : zero;
  };
  auto put = [&](int e, const float4& v) {
    const int i = e >> 5, c = (e & 31) * 4;
    const float w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (c + s != i) pk[i * 129 + c + s] = w[s];
  };
  if (small_vec(src, q.d)) {
    float4 v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = get(tid + t * 512, true);
#pragma unroll
    for (int t = 0; t < 8; ++t) put(tid + t * 512, v[t]);
  } else {
#pragma unroll 1
    for (int e = tid; e < 4096; e += 512) put(e, get(e, false));
  }
  if (tid < 128) pk[tid * 129 + tid] = which == 0 || o + tid >= q.d ? 1.0f : q.sign[o + tid] * expf(q.log_s[o + tid]);
  __syncthreads();
  const SmallTri m = which == 0 ? SmallTri{pk, 129, 1} : SmallTri{pk, 1, 129};
  small_tri_diag(m, tid);
  small_tri_merge16(m, tb, tid);
  small_tri_merge<32>(m, tb, tid);
  small_tri_merge<64>(m, tb, tid);
  const TriOut out = which == 0 ? l : u;
#pragma unroll 4
  for (int e = tid; e < 128 * 128; e += 512) {
    const int i = e >> 7, j = e & 127;
    out.lo[(int64_t)(o + i) * dp + o + j] = j <= i ? m.at(i, j) : 0.0f;
    out.hi[(int64_t)(o + i) * dp + o + j] = i <= j ? m.at(j, i) : 0.0f;
    if (blockIdx.x & 1) out.hi[(int64_t)(o + i) * dp + o - 128 + j] = 0.0f;   // 256 x 256 diagonal blocks hold zeros below the diagonal (launch_tri_last)
  }
}

// out[r][c] = z[r][perm[c]] in the storage type (z P^T), z + z2 in rows and columns below `split`; z is d x d, d % 8 == 0.  A row goes through LDS, so that global memory sees
// whole rows on both sides (gathered straight from memory, d = 4096 took 81 us; this way 18).
template <typename T>
__global__ __launch_bounds__(256) void k_lu_inverse_out(const float* __restrict__ z, const float* __restrict__ z2, int split, const int* __restrict__ perm, int d, T* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) float row[];
  for (int r = blockIdx.x; r < d; r += gridDim.x) {
    for (int c = 4 * threadIdx.x; c < d; c += 1024) {
      float4 v = *reinterpret_cast<const float4*>(z + (int64_t)r * d + c);
      if (r < split && c < split) {
        const float4 w = *reinterpret_cast<const float4*>(z2 + (int64_t)r * d + c);
        v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
      }
      *reinterpret_cast<float4*>(row + c) = v;
    }
    __syncthreads();
    for (int c0 = 8 * threadIdx.x; c0 < d; c0 += 2048) {
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int src = perm[c0 + t];
        v[t] = row[(unsigned)src < (unsigned)d ? src : c0 + t];      // not a permutation: stay inside the row
      }
      T* o = out + (int64_t)r * d + c0;
#pragma unroll
      for (int t = 0; t < 8; ++t) Store<T>::st(o + t, v[t]);
    }
    __syncthreads();
  }
}

// dst [d][d] = the leading d x d part of src, whose rows hold dp entries (both multiples of 128: 16-byte vectors)
__global__ __launch_bounds__(256) void k_tri_compact(const float* __restrict__ src, int dp, int d, float* __restrict__ dst) {
  const int64_t n4 = (int64_t)d * (d / 4);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    const int r = (int)(i / (d / 4)), c4 = (int)(i - (int64_t)r * (d / 4));
    reinterpret_cast<float4*>(dst)[i] = *reinterpret_cast<const float4*>(src + (int64_t)r * dp + 4 * c4);
  }
}

template <typename T, int SRC>
void launch_build_transposed(const LuSrc& q, void* out, hipStream_t s) {
  if (q.d % 64 == 0) hipLaunchKernelGGL((k_lu_build_transposed<T, SRC>), dim3(q.d / 64, q.d / 64), dim3(256), 0, s, q, reinterpret_cast<T*>(out));
  else launch_build<T, SRC, true>(q, out, s);
}

template <typename T, int SRC>
void launch_build_rows(const LuSrc& q, void* out, hipStream_t s) {
  const int64_t g = ((int64_t)q.d * (q.d / 8) + 255) / 256;
  hipLaunchKernelGGL((k_lu_build_rows<T, SRC>), dim3((unsigned)(g < 8192 ? g : 8192)), dim3(256), 0, s, q, reinterpret_cast<T*>(out));
}

// measurement aid (model_lu_timing): HIP events around every matrix-core product, waited for at once
bool g_timing = false;
double g_timing_ms = 0.0;
int64_t g_timing_launches = 0;
hipEvent_t g_ev0 = nullptr, g_ev1 = nullptr;

// one stream of the library's own (default priority, created on first use, kept until the process ends) for work that
// runs beside the caller's stream; null if it cannot be created (the callers then stay on one stream)
hipStream_t lu_side_stream() {
  static std::once_flag once;
  static hipStream_t side = nullptr;
  std::call_once(once, [] {
    if (hipStreamCreateWithFlags(&side, hipStreamNonBlocking) != hipSuccess) side = nullptr;
  });
  return side;
}

// A second branch of work beside the caller's stream: begin() forks the library's stream from `main`, end() joins it
// back — also after an error, so that `main` always covers both branches.  The two events are created once per host
// thread and reused by every call (a wait enqueued on a stream refers to the record that preceded it, so recording
// the event again for the next call does not disturb waits already enqueued); calls from several host threads only
// share the stream.  Disabled (or no stream / events to be had): side == main, everything stays in order.
struct SideBranch {
  hipStream_t main = nullptr, side = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  static bool events(hipEvent_t* f, hipEvent_t* j) {
    static thread_local hipEvent_t ev[2] = {nullptr, nullptr};
    static thread_local bool tried = false;
    if (!tried) {
      tried = true;
      if (hipEventCreateWithFlags(&ev[0], hipEventDisableTiming) != hipSuccess) ev[0] = nullptr;
      if (ev[0] && hipEventCreateWithFlags(&ev[1], hipEventDisableTiming) != hipSuccess) {
        (void)hipEventDestroy(ev[0]);
        ev[0] = ev[1] = nullptr;
      }
    }
    *f = ev[0];
    *j = ev[1];
    return ev[0] != nullptr;
  }
  int begin(hipStream_t s, bool enable, const char* who) {
    main = side = s;
    hipStream_t s2 = enable ? lu_side_stream() : nullptr;
    hipEvent_t f = nullptr, j = nullptr;
    if (!s2 || !events(&f, &j)) return AE_OK;
    if (hipEventRecord(f, s) != hipSuccess || hipStreamWaitEvent(s2, f, 0) != hipSuccess)
      return fail(AE_EHIP, "%s: cannot fork the side stream", who);
    fork = f;
    join = j;
    side = s2;
    return AE_OK;
  }
  int end(int rc, const char* who) {
    if (!fork) return rc;
    const bool joined = hipEventRecord(join, side) == hipSuccess && hipStreamWaitEvent(main, join, 0) == hipSuccess;
    fork = join = nullptr;
    if (!joined && rc == AE_OK) rc = fail(AE_EHIP, "%s: cannot join the side stream", who);
    return rc;
  }
};

// launch(), between two events while model_lu_timing is on
template <typename LAUNCH>
int timed_product(hipStream_t s, LAUNCH launch) {
  if (!g_timing) return launch();
  AE_HIP(hipEventRecord(g_ev0, s));
  AE_TRY(launch());
  AE_HIP(hipEventRecord(g_ev1, s));
  AE_HIP(hipEventSynchronize(g_ev1));
  float ms = 0.0f;
  AE_HIP(hipEventElapsedTime(&ms, g_ev0, g_ev1));
  g_timing_ms += ms;
  ++g_timing_launches;
  return AE_OK;
}

// y[m][n] = sum_k x[m][k] w[n][k], all d x d in the storage type; tri: which operand is triangular (CONV_TRI_*)
int dense_product(const void* x, const void* w, void* y, int d, int dtype, int tri, hipStream_t s) {
  ConvArgs a;
  memset(&a, 0, sizeof(a));
  a.x = x; a.w = w; a.bias = nullptr; a.y = y;
  a.n = d; a.hc = a.wc = 1; a.cin = a.cout = d; a.k = 1; a.up = 0; a.act = ACT_NONE; a.dtype = dtype;
  a.tri = tri;
  // Products of matrices close to the identity (the exponential and its squarings) and those of the QR calls with a triangle keep the binary32 MFMA up to d = 480: a bf16 dot of 16 products is rounded at its largest one, a bias of 1.6e-7 at the
  // diagonal that five squarings carry along coherently, while the binary32 MFMA's error grows with d.  A after compose, 2-norm
  // against float64: d = 256 4.0e-6 by parts against 3.6e-6, d = 1024 4.2e-6 against 1.4e-5, d = 2048 4.6e-6 against 3.7e-5;
  // dG 3.5e-6 against 2.5e-6, 3.4e-6 against 1.1e-5, 3.5e-6 against 3.1e-5.
  a.f32_mfma = (tri == CONV_TRI_NONE || tri == CONV_TRI_LOWER_W_FULL || tri == CONV_TRI_UPPER_W_FULL) && d < 512;
  return timed_product(s, [&]() { return launch_conv_mfma(a, s); });
}

int64_t lu_mat_bytes(int64_t d, int dtype) { return d * d * (int64_t)dtype_size(dtype); }
unsigned lu_grid(int64_t items) {
  const int64_t g = (items + 256 * 8 - 1) / (256 * 8);
  return (unsigned)(g < 4096 ? (g < 1 ? 1 : g) : 4096);
}

// 128 times the smallest power of two that reaches d: the working size of the recursion
int64_t tri_padded_size(int64_t d) {
  int64_t dp = 128;
  while (dp < d) dp *= 2;
  return dp;
}

// The recursion above for L (first 0, count 2 for both) or U + diag s alone (first 1), padded with an identity block to the working size
// dp (128 times a power of two, at least q.d): lo and hi of a factor are its inverse and the inverse's transpose, whichever is
// lower and upper triangular; tt is scratch; all [dp][dp] binary32.
struct TriWork { float* lo; float* hi; float* tt; };
int tri_inverse(const LuSrc& q, int dp, int first, int count, const TriWork& l, const TriWork& u, hipStream_t s) {
  hipLaunchKernelGGL(k_tri_diag_inverse, dim3(dp / 128, count), dim3(512), 0, s, q, dp, first, TriOut{l.lo, l.hi}, TriOut{u.lo, u.hi});
  AE_TRY(launch_status("tri_diag_inverse"));
  for (int b = 128; b < dp; b *= 2) {
    const TriProduct t[2] = {{l.hi, q.lp, q.d, l.tt, nullptr, false}, {u.lo, q.up, q.d, u.tt, nullptr, true}};
    const TriProduct x[2] = {{l.lo, l.tt, dp, l.lo, l.hi, true}, {u.hi, u.tt, dp, u.hi, u.lo, false}};   // (reads diagonal blocks, writes beside them)
    AE_TRY(launch_tri_pairs(t + first, count, dp, b, q.d, false, s));
    AE_TRY(launch_tri_pairs(x + first, count, dp, b, q.d, true, s));
  }
  return AE_OK;
}

// ---- QR parametrisation (Eq. 5):  Q = exp((G - G^T) / 2),  A = Q (R + diag s) ------------------------------------
// The exponential is scaling and squaring: X = S / 2^J, the Taylor polynomial of order 8, then J squarings — all
// binary32 products on the matrix cores.  The polynomial is evaluated in powers of Y = X^3 (four products instead of
// the seven of Horner's rule in X):
//     X2 = X X,  Y = X2 X,   B0 = I + X + X2/2,  B1 = I/3! + X/4! + X2/5!,  B2 = I/6! + X/7! + X2/8!,
//     U = B1 + B2 Y,   Q_0 = B0 + U Y.
// The product kernel computes y = x w^T; X is exactly skew-symmetric, so X^T = -X, X2^T = X2, Y^T = -Y and none of
// these factors needs a transposed copy (x X = -(x X^T)); -X2 is what is stored, as the product leaves it.  The backward pass is the
// adjoint of this chain, step by step, with the stored X, -X2, Y, U, U^T, B2, B2^T and Q_i, Q_i^T (seven products for the
// polynomial, where the two of X2 = X X are one for the skew part that is asked for; two per squaring); few element-wise passes
// form sums, scalings and transposes.  The three products with a triangle: the two whose zeros bound K walk half of it (0.66 ->
// 0.35 ms at d = 4096).  d = 4096: 30 products and 33 passes 21.2 ms, 29 and 23 now 19.7; d = 1024 1.23 and 1.14, d = 2048 3.48 and 3.26.
constexpr int kQrOrder = 8;

// Element-wise passes of the exponential and its adjoint: 32 x 32 tiles, sums of up to three matrices, read once, and the result's
// transpose through LDS.  Bound by HBM.

// out = ident I + c[0] a0 + c[1] a1 + c[2] a2, out_t = out^T.  Absent matrices are null; so may be out or out_t.
struct QrSum { const float* a[3]; float c[3]; float ident; };
template <typename T>
__global__ __launch_bounds__(256) void k_qr_combine(QrSum q, const T* __restrict__ first, int d, float* __restrict__ out, float* __restrict__ out_t) {
  __shared__ float tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = r0 + ty + 8 * j, c = c0 + tx;
    const int64_t i = (int64_t)r * d + c;
    float v = q.c[0] * Store<T>::ld(first + i) + (r == c ? q.ident : 0.0f);
#pragma unroll
    for (int t = 1; t < 3; ++t)
      if (q.a[t]) v += q.c[t] * q.a[t][i];
    if (out) out[i] = v;
    tile[ty + 8 * j][tx] = v;
  }
  __syncthreads();
  if (out_t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) out_t[(int64_t)(c0 + ty + 8 * j) * d + r0 + tx] = tile[tx][ty + 8 * j];
  }
}

// out = scale (s + sign s^T), s = a + b - c (b, c may be null): the skew (sign -1) and symmetric parts
__global__ __launch_bounds__(256) void k_qr_skew(const float* __restrict__ a, const float* __restrict__ b, const float* __restrict__ c, float scale, float sign,
                                                 int d, float* __restrict__ out) {
  __shared__ float tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  auto at = [&](int r, int col) {
    const int64_t i = (int64_t)r * d + col;
    float v = a[i];
    if (b) v += b[i];
    if (c) v -= c[i];
    return v;
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) tile[ty + 8 * j][tx] = at(c0 + ty + 8 * j, r0 + tx);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = r0 + ty + 8 * j, col = c0 + tx;
    out[(int64_t)r * d + col] = scale * (at(r, col) + sign * tile[tx][ty + 8 * j]);
  }
}

// x = a + b/4! + c/7!,  x2 = a/2 + b/5! + c/8!: the gradients of X and X2 through B0, B1 and B2 (16-byte vectors)
__global__ __launch_bounds__(256) void k_qr_powers_grad(const float4* __restrict__ a, const float4* __restrict__ b, const float4* __restrict__ c, int64_t n4,
                                                        float4* __restrict__ x, float4* __restrict__ x2) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    const float4 p = a[i], q = b[i], r = c[i];
    auto s = [](float u, float v, float w, float cu, float cv, float cw) { return cu * u + cv * v + cw * w; };
    constexpr float f4 = 1.0f / 24.0f, f5 = 1.0f / 120.0f, f7 = 1.0f / 5040.0f, f8 = 1.0f / 40320.0f;
    x[i] = make_float4(s(p.x, q.x, r.x, 1.0f, f4, f7), s(p.y, q.y, r.y, 1.0f, f4, f7), s(p.z, q.z, r.z, 1.0f, f4, f7), s(p.w, q.w, r.w, 1.0f, f4, f7));
    x2[i] = make_float4(s(p.x, q.x, r.x, 0.5f, f5, f8), s(p.y, q.y, r.y, 0.5f, f5, f8), s(p.z, q.z, r.z, 0.5f, f5, f8), s(p.w, q.w, r.w, 0.5f, f5, f8));
  }
}

// rowsum[i] = sum_j |m[i][j]|: one wavefront per row, fixed order
__global__ __launch_bounds__(256) void k_row_abs_sum(const float* __restrict__ m, int d, float* __restrict__ rowsum) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= d) return;
  float acc = 0.0f;
  for (int j = lane; j < d; j += 64) acc += fabsf(m[(int64_t)row * d + j]);
  acc = wave_sum(acc);
  if (lane == 0) rowsum[row] = acc;
}
// out[0] = max_i v[i] (one workgroup; NaN propagates as +inf so that the caller refuses it)
__global__ __launch_bounds__(256) void k_vec_max(const float* __restrict__ v, int d, float* __restrict__ out) {
  __shared__ float sm[256];
  float mx = 0.0f;
  for (int i = threadIdx.x; i < d; i += 256) { const float x = v[i]; mx = (x == x) ? fmaxf(mx, x) : INFINITY; }
  sm[threadIdx.x] = mx;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) sm[threadIdx.x] = fmaxf(sm[threadIdx.x], sm[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sm[0];
}

// binary32 -> storage type
template <typename T>
__global__ __launch_bounds__(256) void k_from_f32(const float* __restrict__ in, T* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) Store<T>::st(out + i, in[i]);
}

void qr_combine(const QrSum& q, int d, float* out, float* out_t, hipStream_t s) {
  hipLaunchKernelGGL((k_qr_combine<float>), dim3(d / 32, d / 32), dim3(256), 0, s, q, q.a[0], d, out, out_t);
}
void qr_transpose(const float* y, int d, float* out_t, hipStream_t s) { qr_combine(QrSum{{y, nullptr, nullptr}, {1.0f, 0.0f, 0.0f}, 0.0f}, d, nullptr, out_t, s); }
void qr_skew(const float* a, const float* b, const float* c, float scale, float sign, int d, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_qr_skew, dim3(d / 32, d / 32), dim3(256), 0, s, a, b, c, scale, sign, d, out);
}

// workspace of the QR calls: binary32 d x d matrices
struct QrSlots {
  float* base; int64_t dd; int J;
  float* x() const { return base; }                                  // S / 2^J
  float* h(int k) const { return base + (int64_t)(k - 1) * dd; }     // slots 1 .. kQrOrder-1 (k = 2 .. kQrOrder):
  float* nx2() const { return h(2); }                                //   -X X (symmetric)
  float* y3() const { return h(3); }                                 //   X^3 (skew-symmetric)
  float* u() const { return h(4); }                                  //   U = B1 + B2 Y
  float* ut() const { return h(5); }
  float* b2() const { return h(6); }                                 //   B2 = I/6! + X/7! + X2/8!
  float* b2t() const { return h(7); }
  float* spare() const { return h(8); }                              //   a seventh temporary of the backward pass
  float* q(int i) const { return base + (int64_t)(kQrOrder + i) * dd; }              // Q_i, i = 0 .. J
  float* qt(int i) const { return base + (int64_t)(kQrOrder + J + 1 + i) * dd; }     // Q_i^T
  float* tmp(int t) const { return base + (int64_t)(kQrOrder + 2 * (J + 1) + t) * dd; }   // six temporaries
  static int64_t count(int J) { return kQrOrder + 2 * (J + 1) + 6; }
};

int check_qr_args(const char* who, int64_t d, int dtype, int squarings) {
  if (dtype != AE_F32 && dtype != AE_BF16) return fail(AE_EINVAL, "%s: bad dtype", who);
  if (d < 32 || d % 32 != 0 || d > 16384) return fail(AE_EINVAL, "%s: d must be a multiple of 32 between 32 and 16384", who);
  if (squarings < 0 || squarings > 16) return fail(AE_EINVAL, "%s: squarings must be 0 .. 16", who);
  return AE_OK;
}

int check_lu_size(const char* who, int64_t d, int dtype) {
  if (dtype != AE_F32 && dtype != AE_BF16) return fail(AE_EINVAL, "%s: bad dtype", who);
  if (d < 32 || d % 32 != 0 || d > 16384) return fail(AE_EINVAL, "%s: d must be a multiple of 32 between 32 and 16384", who);
  return AE_OK;
}

int check_small_batch(const char* who, int64_t count, int64_t d, int dtype) {
  if (dtype != AE_F32 && dtype != AE_BF16) return fail(AE_EINVAL, "%s: bad dtype", who);
  if (d < 1 || d > 128) return fail(AE_EINVAL, "%s: d must be 1 .. 128 (larger matrices take the full-size calls)", who);
  if (count < 1 || count > (1 << 20)) return fail(AE_EINVAL, "%s: count must be 1 .. 2^20", who);
  return AE_OK;
}

}  // namespace
}  // namespace ae

extern "C" int model_lu_compose_batch(const float* lp, const float* up, const float* log_s, const float* sign_s, const int* perm,
                                      int64_t count, int64_t d, int dtype, void* a_out, void* stream) {
  using namespace ae;
  if (!lp || !up || !log_s || !sign_s || !perm || !a_out) return fail(AE_EINVAL, "model_lu_compose_batch: null argument");
  AE_TRY(check_small_batch("model_lu_compose_batch", count, d, dtype));
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid((unsigned)(count * ((d + 31) / 32)));
  if (dtype == AE_BF16) hipLaunchKernelGGL((k_lu_small_compose<bf16_t>), grid, dim3(512), 0, s, lp, up, log_s, sign_s, perm, (int)d, (bf16_t*)a_out);
  else hipLaunchKernelGGL((k_lu_small_compose<float>), grid, dim3(512), 0, s, lp, up, log_s, sign_s, perm, (int)d, (float*)a_out);
  return launch_status("lu_small_compose");
}

extern "C" int model_lu_backward_batch(const void* g, const float* lp, const float* up, const float* log_s, const float* sign_s,
                                       const int* perm, int64_t count, int64_t d, int dtype, float* d_lp, float* d_up,
                                       float* d_log_s, void* stream) {
  using namespace ae;
  if (!g || !lp || !up || !log_s || !sign_s || !perm || !d_lp || !d_up || !d_log_s) return fail(AE_EINVAL, "model_lu_backward_batch: null argument");
  AE_TRY(check_small_batch("model_lu_backward_batch", count, d, dtype));
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid((unsigned)(count * 2 * ((d + 31) / 32)));
  if (dtype == AE_BF16) hipLaunchKernelGGL((k_lu_small_backward<bf16_t>), grid, dim3(512), 0, s, (const bf16_t*)g, lp, up, log_s, sign_s, perm, (int)d, d_lp, d_up, d_log_s);
  else hipLaunchKernelGGL((k_lu_small_backward<float>), grid, dim3(512), 0, s, (const float*)g, lp, up, log_s, sign_s, perm, (int)d, d_lp, d_up, d_log_s);
  return launch_status("lu_small_backward");
}

extern "C" int model_lu_inverse_batch(const float* lp, const float* up, const float* log_s, const float* sign_s, const int* perm,
                                      int64_t count, int64_t d, int dtype, void* a_inv_out, void* stream) {
  using namespace ae;
  if (!lp || !up || !log_s || !sign_s || !perm || !a_inv_out) return fail(AE_EINVAL, "model_lu_inverse_batch: null argument");
  AE_TRY(check_small_batch("model_lu_inverse_batch", count, d, dtype));
  hipStream_t s = (hipStream_t)stream;
  const int nb = (int)(d + 31) / 32;
  // blocks of 32 columns per workgroup: as few as keep the launch at one workgroup per compute unit (a workgroup's LDS leaves no room
  // for another), or all.  us with 1 / 2 / 4, bf16, matrices x d: 32 x 128 17.9 / 20.0 / 26.5; 128 x 128 39.0 / 21.0 / 27.6; 256 x 128 74.6 / 43.5 /
  // 29.0; 128 x 96 29.1 / 17.1 / 21.2; 512 x 96 88 / 65 / 42; 64 x 64 12.8 / 13.1; 512 x 64 47.7 / 26.2
  int nc = 1;
  while (nc < 4 && nc < nb && count * ((nb + nc - 1) / nc) > 256) nc *= 2;
  const dim3 grid((unsigned)(count * ((nb + nc - 1) / nc)));
#define SOLVE(NC)                                                                                                                                     \
  do {                                                                                                                                                \
    if (dtype == AE_BF16) hipLaunchKernelGGL((k_lu_small_solve<bf16_t, NC>), grid, dim3(512), 0, s, lp, up, log_s, sign_s, perm, (int)d, (bf16_t*)a_inv_out); \
    else hipLaunchKernelGGL((k_lu_small_solve<float, NC>), grid, dim3(512), 0, s, lp, up, log_s, sign_s, perm, (int)d, (float*)a_inv_out);              \
  } while (0)
  if (nc == 1) SOLVE(1);
  else if (nc == 2) SOLVE(2);
  else SOLVE(4);
#undef SOLVE
  return launch_status("lu_small_inverse");
}

extern "C" int model_lu_workspace(int64_t d, int dtype, int64_t* bytes) {
  using namespace ae;
  if (!bytes) return fail(AE_EINVAL, "model_lu_workspace: null argument");
  AE_TRY(check_lu_size("model_lu_workspace", d, dtype));
  *bytes = 6 * lu_mat_bytes(d, dtype) + ((d * 4 + 255) / 256) * 256;
  return AE_OK;
}

extern "C" int model_lu_compose(const float* lp, const float* up, const float* log_s, const float* sign_s, const int* perm,
                                int64_t d, int dtype, void* a_out, void* workspace, void* stream) {
  using namespace ae;
  if (!lp || !up || !log_s || !sign_s || !perm || !a_out || !workspace) return fail(AE_EINVAL, "model_lu_compose: null argument");
  AE_TRY(check_lu_size("model_lu_compose", d, dtype));
  if (((reinterpret_cast<uintptr_t>(a_out) | reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(lp) |
        reinterpret_cast<uintptr_t>(up)) & 15) != 0)
    return fail(AE_EINVAL, "model_lu_compose: the matrices and the workspace must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int64_t mat = lu_mat_bytes(d, dtype);
  char* ws = reinterpret_cast<char*>(workspace);
  void* l = ws;                 // L                 [i][k]
  void* udt = ws + mat;         // (U + diag s)^T    [n][k]   (binary32: U^T, the diagonal follows in k_lu_permute_rows_diag; kn: U + diag s [k][n])
  void* y = ws + 2 * mat;       // L (U + diag s)    [i][n]
  LuSrc q{lp, up, log_s, sign_s, nullptr, nullptr, (int)d};
  const bool kn = dtype == AE_BF16 && dense_kn_supported(d, d, d, d);     // w as it lies: [k][n]
  if (dtype == AE_BF16) {
    launch_build_rows<bf16_t, LU_L>(q, l, s);
    if (kn) launch_build_rows<bf16_t, LU_UD>(q, udt, s);
    else launch_build_transposed<bf16_t, LU_UD>(q, udt, s);
  } else { launch_build_rows<float, LU_L>(q, l, s); launch_build_transposed<float, LU_U>(q, udt, s); }
  AE_TRY(launch_status("lu_build"));
  if (kn) AE_TRY(timed_product(s, [&]() { return launch_dense_kn(l, udt, y, d, d, d, d, s, CONV_TRI_LOWER_UPPER); }));
  else AE_TRY(dense_product(l, udt, y, (int)d, dtype, CONV_TRI_LOWER_UPPER, s));
  if (dtype == AE_F32) {
    const dim3 grid((unsigned)((d + 1023) / 1024), (unsigned)((d + 15) / 16));
    hipLaunchKernelGGL(k_lu_permute_rows_diag, grid, dim3(256), 0, s, (const float*)y, (const float*)l, q, perm, (float*)a_out);
    return launch_status("lu_permute_rows_diag");
  }
  const int cpr = (int)(d * (int64_t)dtype_size(dtype) / 16);
  hipLaunchKernelGGL(k_lu_permute_rows, dim3(lu_grid(d * cpr)), dim3(256), 0, s, (const uint4*)y, perm, (int)d, cpr, (uint4*)a_out);
  return launch_status("lu_permute_rows");
}

extern "C" int model_lu_backward(const void* g, const float* lp, const float* up, const float* log_s, const float* sign_s,
                                 const int* perm, int64_t d, int dtype, float* d_lp, float* d_up, float* d_log_s,
                                 void* workspace, void* stream) {
  using namespace ae;
  if (!g || !lp || !up || !log_s || !sign_s || !perm || !d_lp || !d_up || !d_log_s || !workspace)
    return fail(AE_EINVAL, "model_lu_backward: null argument");
  AE_TRY(check_lu_size("model_lu_backward", d, dtype));
  if (((reinterpret_cast<uintptr_t>(g) | reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(lp) |
        reinterpret_cast<uintptr_t>(up) | reinterpret_cast<uintptr_t>(d_lp) | reinterpret_cast<uintptr_t>(d_up)) & 15) != 0)
    return fail(AE_EINVAL, "model_lu_backward: the matrices and the workspace must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int64_t mat = lu_mat_bytes(d, dtype);
  char* ws = reinterpret_cast<char*>(workspace);
  void* lt = ws;                // L^T               [k][i]
  void* bt = ws + mat;          // B^T = (P^T G)^T   [n][i]
  void* ud = ws + 2 * mat;      // U + diag s        [k][n]
  void* b = ws + 3 * mat;       // B = P^T G         [r][n]
  void* dud = ws + 4 * mat;     // L^T B             [k][n]  (on and above the diagonal)
  void* dl = ws + 5 * mat;      // B (U + diag s)^T  [r][k]  (below the diagonal)
  int* inv = reinterpret_cast<int*>(ws + 6 * mat);
  hipLaunchKernelGGL(k_lu_invert_perm, dim3(1), dim3(1024), 0, s, perm, inv, (int)d);
  LuSrc q{lp, up, log_s, sign_s, inv, g, (int)d};
  // The two gradient branches share nothing but their inputs, and a product with triangular K ranges ends on a few long
  // tiles that leave most of the chip idle: the lower-triangle branch runs on a stream of the library's own beside the
  // upper-triangle branch (not while model_lu_timing brackets every product with events on one stream).
  SideBranch br;
  // (Smaller matrices stay on one stream, where the kernels are shorter than the fork and the join: us of the call with and without it, bf16 d = 256
  // 75 / 33, 1 024 74 / 46, 1 536 69 / 63, 2 048 74 / 73, 3 072 116 / 133, 4 096 212 / 257; binary32 256 75 / 42, 1 024 84 / 99.)
  const bool kn = dtype == AE_BF16 && dense_kn_supported(d, d, d, d);     // both products read B as it lies: [k][n] and [m][k]
  if (kn) launch_build_rows<bf16_t, LU_B>(q, b, s);
  AE_TRY(br.begin(s, !g_timing && d >= (dtype == AE_BF16 ? 2048 : 1024), "model_lu_backward"));
  hipStream_t s2 = br.side;
  int rc = AE_OK;
  const unsigned grid = lu_grid(d * d / 8 * 4);
  if (dtype == AE_BF16) {
    launch_build_transposed<bf16_t, LU_L>(q, lt, s);
    launch_build_rows<bf16_t, LU_UD>(q, ud, s2);
    if (!kn) { launch_build_transposed<bf16_t, LU_B>(q, bt, s); launch_build_rows<bf16_t, LU_B>(q, b, s2); }
  } else {
    launch_build_transposed<float, LU_L>(q, lt, s); launch_build_transposed<float, LU_B>(q, bt, s);
    launch_build_rows<float, LU_UD>(q, ud, s2); launch_build_rows<float, LU_B>(q, b, s2);
  }
  rc = launch_status("lu_build");
  if (rc == AE_OK) rc = kn ? timed_product(s, [&]() { return launch_dense_kn(lt, b, dud, d, d, d, d, s, CONV_TRI_UPPER_X); }) : dense_product(lt, bt, dud, (int)d, dtype, CONV_TRI_UPPER_X, s);
  if (rc == AE_OK) rc = dense_product(b, ud, dl, (int)d, dtype, CONV_TRI_UPPER_W, s2);
  if (rc == AE_OK) {
    if (dtype == AE_BF16) {
      hipLaunchKernelGGL((k_lu_grad_upper<bf16_t>), dim3(grid), dim3(256), 0, s, (const bf16_t*)dud, log_s, sign_s, (int)d, d_up, d_log_s);
      hipLaunchKernelGGL((k_lu_grad_lower<bf16_t>), dim3(grid), dim3(256), 0, s2, (const bf16_t*)dl, (int)d, d_lp);
    } else {
      hipLaunchKernelGGL((k_lu_grad_upper<float>), dim3(grid), dim3(256), 0, s, (const float*)dud, log_s, sign_s, (int)d, d_up, d_log_s);
      hipLaunchKernelGGL((k_lu_grad_lower<float>), dim3(grid), dim3(256), 0, s2, (const float*)dl, (int)d, d_lp);
    }
    rc = launch_status("lu_backward");
  }
  return br.end(rc, "model_lu_backward");
}

extern "C" int model_qr_workspace(int64_t d, int squarings, int64_t* bytes) {
  using namespace ae;
  if (!bytes) return fail(AE_EINVAL, "model_qr_workspace: null argument");
  AE_TRY(check_qr_args("model_qr_workspace", d, AE_F32, squarings));
  *bytes = QrSlots::count(squarings) * d * d * 4 + 1024;
  return AE_OK;
}

extern "C" int model_qr_squarings(const float* g, int64_t d, void* workspace, int* squarings, void* stream) {
  using namespace ae;
  if (!g || !workspace || !squarings) return fail(AE_EINVAL, "model_qr_squarings: null argument");
  AE_TRY(check_qr_args("model_qr_squarings", d, AE_F32, 0));
  if ((reinterpret_cast<uintptr_t>(workspace) & 15) != 0) return fail(AE_EINVAL, "model_qr_squarings: the workspace must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int n = (int)d;
  float* skew = reinterpret_cast<float*>(workspace);          // S = (G - G^T) / 2
  float* rowsum = skew + d * d;                               // then d row sums and the maximum
  qr_skew(g, nullptr, nullptr, 0.5f, -1.0f, n, skew, s);
  hipLaunchKernelGGL(k_row_abs_sum, dim3((n + 3) / 4), dim3(256), 0, s, (const float*)skew, n, rowsum);
  hipLaunchKernelGGL(k_vec_max, dim3(1), dim3(256), 0, s, (const float*)rowsum, n, rowsum + d);
  AE_TRY(launch_status("qr_squarings"));
  float norm = 0.0f;
  AE_HIP(hipMemcpyAsync(&norm, rowsum + d, sizeof(float), hipMemcpyDeviceToHost, s));
  AE_HIP(hipStreamSynchronize(s));
  if (!(norm < INFINITY)) return fail(AE_EINVAL, "model_qr_squarings: the generator holds a NaN or an infinity");
  int j = 0;
  while (j <= 16 && ldexpf(1.0f, j) < 2.0f * norm) ++j;       // ||S||_2 <= ||S||_inf for a skew-symmetric S
  if (j > 16) return fail(AE_EINVAL, "model_qr_squarings: ||(G - G^T)/2|| = %g needs more than 16 squarings", (double)norm);
  *squarings = j;
  return AE_OK;
}

extern "C" int model_qr_compose(const float* g, const float* rp, const float* log_s, const float* sign_s, int64_t d, int dtype,
                                int squarings, void* a_out, void* workspace, void* stream) {
  using namespace ae;
  if (!g || !rp || !log_s || !sign_s || !a_out || !workspace) return fail(AE_EINVAL, "model_qr_compose: null argument");
  AE_TRY(check_qr_args("model_qr_compose", d, dtype, squarings));
  if (((reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(a_out) | reinterpret_cast<uintptr_t>(rp)) & 15) != 0)
    return fail(AE_EINVAL, "model_qr_compose: the matrices and the workspace must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int n = (int)d, J = squarings;
  const QrSlots w{reinterpret_cast<float*>(workspace), d * d, J};
  qr_skew(g, nullptr, nullptr, 0.5f / (float)(1 << J), -1.0f, n, w.x(), s);
  float* y = w.tmp(1);
  // (dense_product(x, w, out) = x w^T; with w skew-symmetric that is -(x w))
  AE_TRY(dense_product(w.x(), w.x(), w.nx2(), n, AE_F32, CONV_TRI_NONE, s));                // X X^T = -X2
  AE_TRY(dense_product(w.nx2(), w.x(), w.y3(), n, AE_F32, CONV_TRI_NONE, s));               // -X2 X^T = Y
  qr_combine(QrSum{{w.x(), w.nx2(), nullptr}, {1.0f / 5040.0f, -1.0f / 40320.0f, 0.0f}, 1.0f / 720.0f}, n, w.b2(), w.b2t(), s);
  AE_TRY(launch_status("qr_powers"));
  AE_TRY(dense_product(w.b2(), w.y3(), y, n, AE_F32, CONV_TRI_NONE, s));                    // B2 Y^T = -B2 Y
  qr_combine(QrSum{{w.x(), w.nx2(), y}, {1.0f / 24.0f, -1.0f / 120.0f, -1.0f}, 1.0f / 6.0f}, n, w.u(), w.ut(), s);       // U = B1 + B2 Y
  AE_TRY(launch_status("qr_u"));
  AE_TRY(dense_product(w.u(), w.y3(), y, n, AE_F32, CONV_TRI_NONE, s));                     // U Y^T = -U Y
  qr_combine(QrSum{{w.x(), w.nx2(), y}, {1.0f, -0.5f, -1.0f}, 1.0f}, n, w.q(0), w.qt(0), s);   // Q_0 = B0 + U Y
  AE_TRY(launch_status("qr_polynomial"));
  for (int i = 0; i < J; ++i) {
    AE_TRY(dense_product(w.q(i), w.qt(i), w.q(i + 1), n, AE_F32, CONV_TRI_NONE, s));        // Q_{i+1} = Q_i Q_i
    qr_transpose(w.q(i + 1), n, w.qt(i + 1), s);
    AE_TRY(launch_status("qr_square"));
  }
  float* rdt = w.tmp(2);                                                                     // (R + diag s)^T
  LuSrc q{nullptr, rp, log_s, sign_s, nullptr, nullptr, n};
  launch_build_transposed<float, LU_UD>(q, rdt, s);
  AE_TRY(launch_status("qr_build"));
  if (dtype == AE_F32) return dense_product(w.q(J), rdt, a_out, n, AE_F32, CONV_TRI_LOWER_W_FULL, s);
  AE_TRY(dense_product(w.q(J), rdt, y, n, AE_F32, CONV_TRI_LOWER_W_FULL, s));
  hipLaunchKernelGGL((k_from_f32<bf16_t>), dim3(lu_grid(d * d)), dim3(256), 0, s, (const float*)y, (bf16_t*)a_out, d * d);
  return launch_status("qr_compose");
}

extern "C" int model_qr_backward(const void* g_a, const float* rp, const float* log_s, const float* sign_s, int64_t d, int dtype,
                                 int squarings, float* d_g, float* d_rp, float* d_log_s, void* workspace, void* stream) {
  using namespace ae;
  if (!g_a || !rp || !log_s || !sign_s || !d_g || !d_rp || !d_log_s || !workspace) return fail(AE_EINVAL, "model_qr_backward: null argument");
  AE_TRY(check_qr_args("model_qr_backward", d, dtype, squarings));
  if (((reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(g_a) | reinterpret_cast<uintptr_t>(rp) |
        reinterpret_cast<uintptr_t>(d_rp)) & 15) != 0)
    return fail(AE_EINVAL, "model_qr_backward: the matrices and the workspace must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int n = (int)d, J = squarings;
  const int64_t dd = d * d;
  const QrSlots w{reinterpret_cast<float*>(workspace), dd, J};
  float *t0 = w.tmp(0), *t1 = w.tmp(1), *t2 = w.tmp(2), *t3 = w.tmp(3), *t4 = w.tmp(4), *t5 = w.tmp(5);
  // dA in binary32 (t0) and its transpose (t1)
  const QrSum one{{nullptr, nullptr, nullptr}, {1.0f, 0.0f, 0.0f}, 0.0f};
  const dim3 tgrid(n / 32, n / 32);
  if (dtype == AE_BF16) hipLaunchKernelGGL((k_qr_combine<bf16_t>), tgrid, dim3(256), 0, s, one, (const bf16_t*)g_a, n, t0, t1);
  else hipLaunchKernelGGL((k_qr_combine<float>), tgrid, dim3(256), 0, s, one, (const float*)g_a, n, t0, t1);
  AE_TRY(launch_status("qr_backward_in"));
  // d(R + diag s) = Q^T dA: strictly upper part and diagonal
  AE_TRY(dense_product(w.qt(J), t1, t2, n, AE_F32, CONV_TRI_NONE, s));
  hipLaunchKernelGGL((k_lu_grad_upper<float>), dim3(lu_grid(dd / 8 * 4)), dim3(256), 0, s, (const float*)t2, log_s, sign_s, n, d_rp, d_log_s);
  // dQ_J = dA (R + diag s)^T  -> cur (t3), cur^T (t4)
  LuSrc q{nullptr, rp, log_s, sign_s, nullptr, nullptr, n};
  launch_build_rows<float, LU_UD>(q, t2, s);
  AE_TRY(launch_status("qr_build"));
  AE_TRY(dense_product(t0, t2, t3, n, AE_F32, CONV_TRI_UPPER_W_FULL, s));
  qr_transpose(t3, n, t4, s);
  float *cur = t3, *cur_t = t4;
  // squarings in reverse: dQ_i = dQ_{i+1} Q_i^T + Q_i^T dQ_{i+1}
  for (int i = J - 1; i >= 0; --i) {
    AE_TRY(dense_product(cur, w.q(i), t0, n, AE_F32, CONV_TRI_NONE, s));
    AE_TRY(dense_product(w.qt(i), cur_t, t1, n, AE_F32, CONV_TRI_NONE, s));
    qr_combine(QrSum{{t0, t1, nullptr}, {1.0f, 1.0f, 0.0f}, 0.0f}, n, cur, cur_t, s);
    AE_TRY(launch_status("qr_backward_square"));
  }
  // the polynomial in reverse; A = dQ_0, B = its transpose, C .. G free
  float *A = cur, *B = cur_t, *C = t0, *D = t1, *E = t2, *F = w.spare(), *G = t5;
  AE_TRY(dense_product(A, w.y3(), C, n, AE_F32, CONV_TRI_NONE, s));                         // dU = dQ_0 Y^T
  qr_transpose(C, n, D, s);                                                                 // dU^T
  AE_TRY(dense_product(w.ut(), B, E, n, AE_F32, CONV_TRI_NONE, s));                         // U^T dQ_0        (Q_0 = B0 + U Y)
  AE_TRY(dense_product(w.b2t(), D, F, n, AE_F32, CONV_TRI_NONE, s));                        // B2^T dU         (U = B1 + B2 Y)
  qr_combine(QrSum{{E, F, nullptr}, {1.0f, 1.0f, 0.0f}, 0.0f}, n, E, D, s);                 // dY = their sum (E) and dY^T (D)
  AE_TRY(launch_status("qr_backward_dy"));
  AE_TRY(dense_product(C, w.y3(), F, n, AE_F32, CONV_TRI_NONE, s));                         // dB2 = dU Y^T
  // dX  = dB0 + dB1/4! + dB2/7!  + ...,   dX2 = dB0/2 + dB1/5! + dB2/8! + ...   with dB0 = dQ_0, dB1 = dU
  hipLaunchKernelGGL(k_qr_powers_grad, dim3(lu_grid(dd)), dim3(256), 0, s, (const float4*)A, (const float4*)C, (const float4*)F, dd / 4, (float4*)G, (float4*)B);
  AE_TRY(launch_status("qr_backward_db"));
  AE_TRY(dense_product(E, w.x(), A, n, AE_F32, CONV_TRI_NONE, s));                          // Y = X2 X:  dX2 += dY X^T
  AE_TRY(dense_product(w.nx2(), D, C, n, AE_F32, CONV_TRI_NONE, s));                        //            dX  += X2^T dY = X2 dY = -C
  // X2 = X X:  dX += dX2 X^T + X^T dX2.  Only the skew part of dX is asked for, and that of these two terms is the skew part of
  // (dX2 + dX2^T) X^T:  X^T = -X, so the transpose of the second is -dX2^T X^T, and skew parts of a matrix and of its negative transpose agree
  qr_skew(B, A, nullptr, 1.0f, 1.0f, n, F, s);
  AE_TRY(launch_status("qr_backward_dx2"));
  AE_TRY(dense_product(F, w.x(), A, n, AE_F32, CONV_TRI_NONE, s));
  // X = (G - G^T) / (2 * 2^J):  dG = (dX - dX^T) / (2 * 2^J)
  qr_skew(G, A, C, 0.5f / (float)(1 << J), -1.0f, n, d_g, s);
  return launch_status("qr_backward");
}

extern "C" int model_qr_inverse(const float* rp, const float* log_s, const float* sign_s, int64_t d, int dtype, int squarings,
                                const void* qr_workspace, void* a_inv_out, void* workspace, void* stream) {
  using namespace ae;
  if (!rp || !log_s || !sign_s || !qr_workspace || !a_inv_out || !workspace) return fail(AE_EINVAL, "model_qr_inverse: null argument");
  AE_TRY(check_qr_args("model_qr_inverse", d, dtype, squarings));
  if (d < 128 || d % 128 != 0) return fail(AE_EINVAL, "model_qr_inverse: d must be a multiple of 128, at most 16384");
  if (((reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(qr_workspace) | reinterpret_cast<uintptr_t>(a_inv_out)) & 15) != 0)
    return fail(AE_EINVAL, "model_qr_inverse: the matrices and the workspaces must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int64_t dd = d * d, dp = tri_padded_size(d), pp = dp * dp;
  const QrSlots w{const_cast<float*>(reinterpret_cast<const float*>(qr_workspace)), dd, squarings};
  float* f = reinterpret_cast<float*>(workspace);
  float *compact = f, *tt = f + pp, *rdinv_t = f + 2 * pp, *rdinv = f + 3 * pp, *z = f + 4 * pp;
  LuSrc q{nullptr, rp, log_s, sign_s, nullptr, nullptr, (int)d};
  AE_TRY(tri_inverse(q, (int)dp, 1, 1, TriWork{}, TriWork{rdinv_t, rdinv, tt}, s));
  if (dp != d) {                                                          // drop the identity padding
    hipLaunchKernelGGL(k_tri_compact, dim3(lu_grid(dd)), dim3(256), 0, s, (const float*)rdinv, (int)dp, (int)d, compact);
    AE_TRY(launch_status("tri_compact"));
    rdinv = compact;
  }
  // A^-1 = (R + diag s)^-1 Q^T = x w^T with w = Q, x upper triangular (its lower triangle is not written)
  if (dtype == AE_F32) return dense_product(rdinv, w.q(squarings), a_inv_out, (int)d, AE_F32, CONV_TRI_UPPER_X_FULL, s);
  AE_TRY(dense_product(rdinv, w.q(squarings), z, (int)d, AE_F32, CONV_TRI_UPPER_X_FULL, s));
  hipLaunchKernelGGL((k_from_f32<bf16_t>), dim3(lu_grid(dd)), dim3(256), 0, s, (const float*)z, (bf16_t*)a_inv_out, dd);
  return launch_status("qr_inverse");
}

extern "C" int model_lu_inverse_workspace(int64_t d, int64_t* bytes) {
  using namespace ae;
  if (!bytes) return fail(AE_EINVAL, "model_lu_inverse_workspace: null argument");
  if (d < 128 || d > 16384 || d % 128 != 0) return fail(AE_EINVAL, "model_lu_inverse_workspace: d must be a multiple of 128, at most 16384");
  const int64_t dp = tri_padded_size(d);
  *bytes = 8 * dp * dp * 4 + 1024;
  return AE_OK;
}

extern "C" int model_lu_inverse(const float* lp, const float* up, const float* log_s, const float* sign_s, const int* perm,
                                int64_t d, int dtype, void* a_inv_out, void* workspace, void* stream) {
  using namespace ae;
  if (!lp || !up || !log_s || !sign_s || !perm || !a_inv_out || !workspace) return fail(AE_EINVAL, "model_lu_inverse: null argument");
  if (dtype != AE_F32 && dtype != AE_BF16) return fail(AE_EINVAL, "model_lu_inverse: bad dtype");
  if (d < 128 || d > 16384 || d % 128 != 0) return fail(AE_EINVAL, "model_lu_inverse: d must be a multiple of 128, at most 16384");
  if ((reinterpret_cast<uintptr_t>(workspace) & 15) != 0) return fail(AE_EINVAL, "model_lu_inverse: the workspace must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int64_t dp = tri_padded_size(d), pp = dp * dp;
  float* f = reinterpret_cast<float*>(workspace);
  const TriWork l{f, f + pp, f + 4 * pp};                  // L^-1 and its transpose
  const TriWork u{f + 2 * pp, f + 3 * pp, f + 5 * pp};     // the transpose of (U + diag s)^-1 and itself
  float *z = f + 6 * pp, *z2 = f + 7 * pp;                 // (U + diag s)^-1 L^-1, the second halves of its long sums
  LuSrc q{lp, up, log_s, sign_s, nullptr, nullptr, (int)d};
  AE_TRY(tri_inverse(q, (int)dp, 0, 2, l, u, s));
  AE_TRY(timed_product(s, [&]() { return launch_tri_last(u.hi, l.hi, (int)dp, z, z2, (int)d, s); }));
  const int split = tri_last_split((int)d);
  const dim3 og((unsigned)(d < 2048 ? d : 2048));
  if (dtype == AE_BF16) hipLaunchKernelGGL((k_lu_inverse_out<bf16_t>), og, dim3(256), (size_t)d * 4, s, (const float*)z, (const float*)z2, split, perm, (int)d, (bf16_t*)a_inv_out);
  else hipLaunchKernelGGL((k_lu_inverse_out<float>), og, dim3(256), (size_t)d * 4, s, (const float*)z, (const float*)z2, split, perm, (int)d, (float*)a_inv_out);
  return launch_status("lu_inverse_out");
}

extern "C" int model_lu_timing(int enable, double* gemm_ms, int64_t* launches) {
  using namespace ae;
  if (gemm_ms) *gemm_ms = g_timing_ms;
  if (launches) *launches = g_timing_launches;
  if (enable && !g_ev0) {
    AE_HIP(hipEventCreate(&g_ev0));
    AE_HIP(hipEventCreate(&g_ev1));
  }
  g_timing = enable != 0;
  g_timing_ms = 0.0;
  g_timing_launches = 0;
  return AE_OK;
}

extern "C" int model_vol_penalty(const float* log_s, int64_t d, float* value, float* d_log_s, void* stream) {
  using namespace ae;
  if (!log_s || !value) return fail(AE_EINVAL, "model_vol_penalty: null argument");
  if (d < 1 || d > (1 << 24)) return fail(AE_EINVAL, "model_vol_penalty: bad size");
  hipLaunchKernelGGL(k_vol_penalty, dim3(1), dim3(256), 0, (hipStream_t)stream, log_s, (int)d, value, d_log_s);
  return launch_status("vol_penalty");
}
