// ae_conv_mfma.hip — convolution / fully-connected layers as implicit GEMM on the
// CDNA4 matrix cores.
//
//   C[M][N] = A[M][K] * B[N][K]^T,  M = batch*H*W output pixels, N = C_out,
//   K = k*k*C_in ordered (r, s, ci).
// A is never materialised: row m is pixel (n,h,w) and the K-slab [kt*BK, kt*BK+BK)
// lies inside one filter tap (r,s) because C_in is a multiple of BK, so the slab is
// BK contiguous channels of input pixel (h+r-p, w+s-p) (zero outside the image; read
// through a x2 nearest upsample when `up`).  B is the packed weight [C_out][k][k][C_in].
//
// One workgroup of 256 threads (4 wavefronts) computes a BM x BN tile with
// v_mfma_f32_32x32x16_bf16 (bf16) or v_mfma_f32_32x32x2_f32 (fp32).  Kernels in this file:
//   k_conv3_patch  3x3 convolutions of 16/32/64-wide images (wider ones by column strips): the input patch
//                  of a tile lives in LDS and all nine taps are read from it (one global read per input
//                  element); the weights, packed in MFMA fragment order, go straight into registers
//   k_igemm        every other shape: per-tap slabs through a three-stage global-to-LDS ring,
//                  optionally split over K; also the two cheaper forms of a 3x3 convolution behind
//                  a x2 upsample (four 2x2 phase convolutions forward, one 4x4 stride-2
//                  convolution for the input gradient; see IgemmParams)
//                  and, with CHUNKS, any channel counts (a 16-byte chunk of K belongs to one tap; see there)
//   k_wgrad_row3   weight gradient, three taps per workgroup from one input patch (bf16)
//   k_wgrad_rows, k_wgrad   weight gradient, one tap per workgroup (1x1, odd shapes)
//   k_wgrad_chunks          weight gradient of any channel counts, columns (tap, ci) walked across tap borders; binary32: k_wgrad_split
//   k_dense                 dense bf16 products in check-free tiles
//   k_gemm_split            binary32 products and convolutions by bf16 parts
// The shared epilogue adds the bias, rounds to the storage type, optionally reduces per-channel
// sum / sum of squares of the tile (batch-norm statistics), applies the activation and stores [M][N].
#include <algorithm>
#include <type_traits>

#include "ae_device.h"
#include "ae_internal.h"

namespace ae {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

struct IgemmParams {
  const void* x; const void* w; const float* bias; void* y; float* y_aux; float* partial;
  int64_t M;
  int N, K;             // C_out, k*k*C_in
  int Hc, Wc, Cin, ksz, up;
  int act;
  int tiles_n;
  unsigned x_bytes, w_bytes;   // sizes of the two operand tensors (buffer range checks)
  // split-K (layers with too few output tiles to fill the chip): workgroup (split, tile) works on
  // K slabs [split*slabs_per_split, ...) and writes its fp32 tile to split_out[split][M][N];
  // k_splitk_finish sums the splits and applies bias / rounding / activation
  int tiles_mn, slabs_per_split;
  float* split_out;
  // Source geometry.  GEMM row m is pixel (n, i, j) of an Hc x Wc grid; tap (r, s) of that row
  // reads source position (i*stride + r - pad_h, j*stride + s - pad_w) of an Hv x Wv image
  // (stored at (Hv>>up) x (Wv>>up): nearest-neighbour upsampling folded into the read), zero
  // outside.  Plain convolution: Hv = Hc, Wv = Wc, stride 1, pad = (ksz-1)/2.
  int Hv, Wv, stride, pad;
  // phases = 4: the convolution behind a x2 upsample, written as four 2x2 convolutions of the
  // stored input (one per output parity (a, b) = (phase>>1, phase&1), pads 1-a and 1-b, weights
  // w + phase*N*K); row (n, i, j) of phase (a, b) is output pixel (2i+a, 2j+b) of a 2Hc x 2Wc image
  int phases;
  // k_dense with its second operand [k][n] (KN): output rows are groups of kn_group, each a product of its own with the x of
  // kn_group rows and K rows of w (group g: rows K g .. of w)
  int kn_group = 0;
  // epilogue variants of the dense-GEMM use (EPI template parameter of k_dense, k_igemm and k_gemm_split):
  //   1: the stored output is MX block-quantised (blocks of mx_block output columns: a power of two from one 16-byte
  //      chunk up to the 64 columns of a wave tile; FP4 E2M1 elements);
  //   2: nothing is stored; the epilogue forms resid[m][n] - (acc + bias) and leaves per-tile column sums of it
  //      and of its square in `partial` (resid: [M][N] in the storage type)
  const void* resid;
  int mx_block, mx_elem;       // block size and element format (MX_FP4 / MX_INT4 / MX_FP8) of epilogue 1
  // Square dense products (M = N = K) with triangular operands: K range per tile, and tiles nobody wants skipped.
  //   1: x[m][k] = 0 for k > m and w[n][k] = 0 for k > n (lower times upper): K ends at min(last row, last column) + 1
  //   2: x[m][k] = 0 for k < m, wanted outputs n >= m: K starts at the tile's first row; tiles below the diagonal return
  //   3: w[n][k] = 0 for k < n, wanted outputs n < m: K starts at the tile's first column; tiles above the diagonal return
  //   4: x[m][k] = 0 for k < m: K starts at the tile's first row
  //   5: w[n][k] = 0 for k > n: K ends at the tile's last column
  //   6: w[n][k] = 0 for k < n: K starts at the tile's first column
  int tri;
  // k_gemm_split<..., TRI_PAIRS>: one product of one level of the blocked triangular inverse, for all pairs of neighbouring tri_b x tri_b diagonal
  // blocks (r even, r + 1) of one or two matrices in one launch: only the tiles of one off-diagonal block per pair, K the block of their rows
  //   upper: rows in block r, columns in block r + 1, x upper triangular: K from the tile's first row on;
  //   lower: rows in block r + 1, columns in block r, x lower triangular: K up to the tile's last row
  // tri_d: the matrices are an identity block beyond row and column tri_d; tiles of the odd block that lie wholly beyond it return
  // (their outputs are zero and stay unwritten) and K ranges over the odd block end there.  negate: -(x w^T), and its transpose into yt.
  // TRI_LAST: x upper, w^T lower triangular: K starts at max(first row, first column); 128 x 128 outputs whose K range is longer than half of K are two
  // workgroups, of which the second leaves its sums in the other matrix's y.
  // Row lengths ldx and ldw (elements) of the operands, N of the outputs.
  struct Tri { const void* x; const void* w; void* y; float* yt; bool lower; } tm[2];
  int tri_b, tri_d, tri_pairs, ldx, ldw;
  bool negate;
  // k_conv3_patch on images wider than its tile: a tile is TH rows x Wt columns of one of `strips` column strips
  // of the image (Wt = Wc / strips, TH = 256 / Wt); GEMM row m = tile * 256 + th * Wt + tw then is pixel
  // (row block * TH + th, strip * Wt + tw) of its image.  1: a tile spans the image width and rows are pixels in order.
  int strips = 1;
  int chunks = 0;              // CHUNKS kernels: 16-byte chunks of one tap (= Cin / elements per chunk)
  int log_wt = 6;              // log2 of the strip width Wc / strips
  int log_w = -1, log_h = -1;  // log2 of Wc and Hc when both are powers of two (the four-phase output mapping), else -1
  // Companion tensor of the output's shape and layout (interior tiles only): the saved activation a of the layer whose
  // output gradient this launch computes.  With dyv = (a > 0 ? value : 0) per stored value:
  //   1: dyv is stored instead of the value (ReLU backward); partial receives per-tile column sums of dyv (the bias gradient);
  //   2: the value is stored unchanged; partial receives per-tile column sums of dyv and of dyv * xhat, with
  //      xhat = a * invstd/scale - (shift/scale + mean) * invstd from comp_bn = [scale | shift | mean | invstd] (the sums
  //      of a batch-norm backward behind ReLU and max-pooling; columns with scale = 0 get a zero second sum).
  const void* comp = nullptr;
  int comp_mode = 0;
  const float* comp_bn = nullptr;
};

// output row (pixel index in y) of GEMM row m.  Column strips: the part that depends on the 256-row tile alone
// (image, row block, strip) is igemm_strip_base, taken once per tile by the caller; the strip width is a power of two.
__device__ __forceinline__ int64_t igemm_strip_base(const IgemmParams& p, int64_t m_tile) {
  const unsigned tile = (unsigned)(m_tile >> 8), wt = 1u << p.log_wt, th_n = 256u >> p.log_wt;
  const unsigned strip = tile % (unsigned)p.strips, t2 = tile / (unsigned)p.strips;
  const unsigned blocks = (unsigned)p.Hc / th_n;
  const unsigned rb = t2 % blocks, img = t2 / blocks;
  return ((int64_t)img * p.Hc + rb * th_n) * p.Wc + strip * wt;
}
__device__ __forceinline__ int64_t igemm_out_row(const IgemmParams& p, int64_t m, int phase, int64_t strip_base) {
  if (p.strips > 1) {
    const unsigned ml = (unsigned)m & 255u;
    return strip_base + (int64_t)((ml >> p.log_wt) * (unsigned)p.Wc + (ml & ((1u << p.log_wt) - 1u)));
  }
  if (p.phases == 1) return m;
  const unsigned mu = (unsigned)m;
  unsigned j, i, n;
  if (p.log_w >= 0) {        // power-of-two images: no divisions
    j = mu & ((unsigned)p.Wc - 1u);
    const unsigned t = mu >> p.log_w;
    i = t & ((unsigned)p.Hc - 1u); n = t >> p.log_h;
  } else {
    j = mu % (unsigned)p.Wc;
    const unsigned t = mu / (unsigned)p.Wc;
    i = t % (unsigned)p.Hc; n = t / (unsigned)p.Hc;
  }
  return ((int64_t)n * (2 * p.Hc) + 2 * i + (phase >> 1)) * (2 * p.Wc) + 2 * j + (phase & 1);
}

// ---------------------------------------------------------------------------
// The kernel, for T = bf16 (v_mfma_f32_32x32x16_bf16) or T = float (v_mfma_f32_32x32x2_f32).
// A slab row is BKB = 64 or 128 bytes of K = CPR 16-byte chunks.  LDS rows are not
// padded; chunk c of row r is stored in slot c ^ f(r) with f(r) = (r>>2)&3 (64-byte rows)
// or (r>>1)&7 (128-byte rows): the LDS has 64 banks and serves 16 lanes of a 16-byte
// access per pass, and with this swizzle the 16 rows of a pass fall into 16 different
// 16-byte columns for the loader's stores and for the MFMA fragment reads alike.
// A fragment read fetches 16 bytes per lane: lanes 0-31 chunk 2*ks, lanes 32-63 chunk
// 2*ks+1 of their row.  For bf16 that is exactly the operand of one K=16 MFMA; for fp32
// the four floats feed four K=2 MFMAs (component j of the low lanes is paired with
// component j of the high lanes — any pairing works as long as A and B use the same).
// Global loads are buffer loads: the hardware range check returns zero for the offsets
// that the loader marks invalid (zero padding of the image, rows past M or N), so no
// select or clamp is needed, and addresses are 32-bit byte offsets that only change when
// the filter tap changes.
// ---------------------------------------------------------------------------
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
constexpr unsigned kOob = 0x80000000u;         // beyond any tensor (tensors are < 2 GiB): reads as zero

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// Workgroups are handed to the 8 accelerator dies (XCDs, each with its own L2) round-robin by
// workgroup id.  This maps the hardware id to a logical one such that each XCD works on one
// contiguous range of logical ids, so that workgroups which share operand rows (neighbouring
// tiles, the taps of one tile) hit in the same L2.
__device__ __forceinline__ int xcd_logical_block(int b, int nb) {
  const int per = nb >> 3;                       // full rounds of 8
  return b < (per << 3) ? (b & 7) * per + (b >> 3) : b;
}

template <typename T> __device__ __forceinline__ void mma_step(const uint4v& a, const uint4v& b, floatx16& c);
template <> __device__ __forceinline__ void mma_step<bf16_t>(const uint4v& a, const uint4v& b, floatx16& c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ void mma_step<float>(const uint4v& a, const uint4v& b, floatx16& c) {
  const float4v fa = __builtin_bit_cast(float4v, a), fb = __builtin_bit_cast(float4v, b);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[0], fb[0], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[1], fb[1], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[2], fb[2], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[3], fb[3], c, 0, 0, 0);
}

// Smallest magnitude seen, zeros aside, as twice its bits less one (a zero wraps to the largest number).  The parts of a
// binary32 value are exact while its last place is one of a bfloat16 denormal, 2^-133: from 2^-110 on.
__device__ __forceinline__ void track_smallest(unsigned& lo, const uint4v& v) {
  lo = min(min(lo, v[0] * 2u - 1u), v[1] * 2u - 1u);
  lo = min(min(lo, v[2] * 2u - 1u), v[3] * 2u - 1u);
}
__device__ __forceinline__ bool parts_inexact(unsigned lo) { return lo < 2u * ((127u - 110u) << 23) - 1u; }

// acc += low; true if a sum is then no finite number
template <int MI, int NJ>
__device__ __forceinline__ bool add_not_finite(floatx16 (&acc)[MI][NJ], const floatx16 (&low)[MI][NJ]) {
  float z = 0.0f;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[i][j][e] += low[i][j][e];
        z = fmaf(acc[i][j][e], 0.0f, z);         // NaN from the first infinity or NaN on
      }
  return z != 0.0f;
}

typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) void lds_void_t;
// 16 bytes per lane from a buffer straight into LDS: lane l writes lds_wave_base + 16*l
// (offsets past the buffer's range deliver zeros like any buffer load)
__device__ __forceinline__ void dma_load16(__amdgpu_buffer_rsrc_t rsrc, char* lds_wave_base, unsigned voffset) {
  typedef __attribute__((address_space(3))) void lds_void;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)lds_wave_base, 16, voffset, 0, 0, 0);
}
// the same with a scalar (uniform) byte offset added to every lane's offset
__device__ __forceinline__ void dma_load16s(__amdgpu_buffer_rsrc_t rsrc, char* lds_wave_base, unsigned voffset, unsigned soffset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_t*)lds_wave_base, 16, voffset, soffset, 0, 0);
}
constexpr int vm_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }   // s_waitcnt vmcnt(n) only

// Epilogue of a tile that lies wholly inside the output (no bounds checks): bias, rounding to the
// storage type, optional column statistics of the stored value, optional ReLU, then 16-byte
// row stores staged through this wave's LDS area.
// the 16/sizeof(T) values of a 16-byte chunk held in registers
template <typename T> __device__ __forceinline__ void unpack_chunk(const uint4v& w, float (&v)[16 / (int)sizeof(T)]);
template <> __device__ __forceinline__ void unpack_chunk<bf16_t>(const uint4v& w, float (&v)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float((uint32_t)w[i] << 16);
    v[2 * i + 1] = __uint_as_float((uint32_t)w[i] & 0xFFFF0000u);
  }
}
template <> __device__ __forceinline__ void unpack_chunk<float>(const uint4v& w, float (&v)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __uint_as_float((uint32_t)w[i]);
}

// Per-lane state of the companion-tensor epilogues (IgemmParams::comp): a lane stores the same 16-byte column chunk of
// every row it handles, so it keeps that chunk's column sums (and the two coefficients of xhat per column).
template <int EPC> struct CompSums { float s1[EPC], s2[EPC], p1[EPC], p0[EPC]; };

template <typename T, int MI, int NJ, int WN, int SW, bool STATS, bool RELU, int MXF = -1, int COMP = 0>   // MXF: element format of the quantising epilogue, or -1
__device__ __forceinline__ void igemm_store_interior(const floatx16 (&acc)[MI][NJ], const float (&bias)[NJ], T* stage,
                                                     T* yrow, int N, int lane, float (&s1)[NJ], float (&s2)[NJ],
                                                     const IgemmParams& p, int64_t mrow0, int phase, T* ycol,
                                                     CompSums<16 / (int)sizeof(T)>* cs = nullptr) {
  constexpr int ES = (int)sizeof(T);
  constexpr int EPC = 16 / ES;               // elements per 16-byte chunk
  constexpr int CPRO = WN / EPC;             // chunks per staged row
  const int col_lane = lane & 31, row_lane = (lane >> 5) * 4;
  const int64_t sbase = p.strips > 1 ? igemm_strip_base(p, mrow0) : 0;   // (a wave's rows lie in one 256-row tile)
  // companion tensor: all of this wave's chunks are requested before the first row is staged, so that their
  // latency runs behind the conversion and the stores of the rows before them
  constexpr int NCH = (32 * CPRO) / 64;
  uint4v cmp[COMP != 0 ? MI : 1][COMP != 0 ? NCH : 1];
  if constexpr (COMP != 0) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int idx = c * 64 + lane;
        const int lr = idx / CPRO, ch = idx % CPRO;
        const T* dst = (p.phases == 1 && p.strips == 1) ? yrow + (int64_t)(i * 32 + lr) * N + ch * EPC
                                                        : ycol + igemm_out_row(p, mrow0 + i * 32 + lr, phase, sbase) * N + ch * EPC;
        cmp[i][c] = *reinterpret_cast<const uint4v*>(reinterpret_cast<const T*>(p.comp) + (dst - reinterpret_cast<T*>(p.y)));
      }
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int lr = (e >> 2) * 8 + row_lane + (e & 3);
        float v = acc[i][j][e] + bias[j];
        if (STATS) {   // statistics of the stored value, taken about the channel's bias (see k_bn_finalize)
          v = round_to_storage<T>(v);
          const float d = v - bias[j];
          s1[j] += d;
          s2[j] = fmaf(d, d, s2[j]);
        }
        if (RELU) v = fmaxf(v, 0.0f);          // rounding is monotonic and keeps 0: same as ReLU of the rounded value
        Store<T>::st(&stage[lr * SW + j * 32 + col_lane], v);
      }
    }
#pragma unroll
    for (int c = 0; c < (32 * CPRO) / 64; ++c) {
      const int idx = c * 64 + lane;
      const int lr = idx / CPRO, ch = idx % CPRO;
      T* dst = (p.phases == 1 && p.strips == 1) ? yrow + (int64_t)(i * 32 + lr) * N + ch * EPC
                                                : ycol + igemm_out_row(p, mrow0 + i * 32 + lr, phase, sbase) * N + ch * EPC;
      if constexpr (MXF >= 0) {
        // MX block quantisation of the stored row: a block of mx_block columns is mx_block/EPC neighbouring lanes of this
        // pass (a staged row is CPRO >= mx_block/EPC consecutive lanes, blocks do not straddle rows)
        float f[EPC];
        Store<T>::ldv(&stage[lr * SW + ch * EPC], f);
        float amax = 0.0f;
#pragma unroll
        for (int t = 0; t < EPC; ++t) amax = fmaxf(amax, fabsf(f[t]));
        for (int off = 1; off < p.mx_block / EPC; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
        if (amax > 0.0f) {
          const int k = mx_scale_exp(amax, MxFormat<MXF>::r_max);
          const float sc = mx_pow2(k), inv_sc = mx_pow2(-k);
#pragma unroll
          for (int t = 0; t < EPC; ++t) f[t] = MxFormat<MXF>::quant(f[t], inv_sc, sc);
        }
        Store<T>::stv(dst, f);
      } else if constexpr (COMP != 0) {
        float f[EPC], a[EPC];
        Store<T>::ldv(&stage[lr * SW + ch * EPC], f);
        unpack_chunk<T>(cmp[i][c], a);
#pragma unroll
        for (int t = 0; t < EPC; ++t) {
          const float dyv = a[t] > 0.0f ? f[t] : 0.0f;
          cs->s1[t] += dyv;
          if (COMP == 2) cs->s2[t] = fmaf(dyv, fmaf(a[t], cs->p1[t], cs->p0[t]), cs->s2[t]);
          else f[t] = dyv;
        }
        if (COMP == 1) Store<T>::stv(dst, f);
        else *reinterpret_cast<uint4v*>(dst) = *reinterpret_cast<const uint4v*>(&stage[lr * SW + ch * EPC]);
      } else {
        *reinterpret_cast<uint4v*>(dst) = *reinterpret_cast<const uint4v*>(&stage[lr * SW + ch * EPC]);
      }
    }
  }
}

// Epilogue variant 2: column sums of resid - (acc + bias) and of its square over the tile's rows; nothing stored.
template <typename T, int MI, int NJ>
__device__ __forceinline__ void igemm_resid_stats(const floatx16 (&acc)[MI][NJ], const float (&bias)[NJ], const T* rrow, int N,
                                                  int lane, float (&s1)[NJ], float (&s2)[NJ]) {
  const int col_lane = lane & 31, row_lane = (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int lr = (e >> 2) * 8 + row_lane + (e & 3);
        const float dv = Store<T>::ld(rrow + (int64_t)(i * 32 + lr) * N + j * 32 + col_lane) - (acc[i][j][e] + bias[j]);
        s1[j] += dv;
        s2[j] = fmaf(dv, dv, s2[j]);
      }
}

// Epilogue shared by the implicit-GEMM kernels.  Accumulator element e of lane l in tile (i,j):
//     row = wm*WM + i*32 + (e/4)*8 + (l/32)*4 + e%4,  column = wn*WN + j*32 + l%32
// Results go through a wave-private LDS staging area (the operand buffers are free: the K loop
// ended on a barrier) so that global stores are 16 bytes wide and each instruction covers
// whole row segments.  smem: at least 4*32*(WN + 16/sizeof(T))*sizeof(T) bytes; sRed: [WGM][2][BN].
// PHASED: a checked tile may belong to an output parity of an upsampled convolution (interior tiles always may).
// RESID_LDS: smem holds the whole tile in the storage type.  DIRECT: the checked tiles of direct_stores.
template <typename T, int BM, int BN, int WGM, int WGN, bool INTERIOR, int EPI = 0, bool PHASED = false, bool RESID_LDS = false, bool DIRECT = false>
__device__ __forceinline__ void igemm_epilogue(floatx16 (&acc)[BM / WGM / 32][BN / WGN / 32], const IgemmParams& p,
                                               char* smem, float (*sRed)[2][BN], int64_t m0, int n0, int64_t tile_m,
                                               int phase = 0) {
  constexpr int ES = (int)sizeof(T);
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int MI = WM / 32, NJ = WN / 32;
  constexpr int SW = WN + 16 / ES;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  T* __restrict__ Y = (T*)p.y;
  const int col_lane = lane & 31, row_lane = (lane >> 5) * 4;
  const bool wide_store = ((p.N * ES) % 16 == 0) && !p.y_aux;
  T* stage = reinterpret_cast<T*>(smem) + wave * (32 * SW);
  float s1[NJ], s2[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) { s1[j] = 0.0f; s2[j] = 0.0f; }
  if constexpr (INTERIOR) {
    float bias[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) bias[j] = p.bias ? p.bias[n0 + wn * WN + j * 32 + col_lane] : 0.0f;
    T* yrow = Y + (m0 + wm * WM) * p.N + n0 + wn * WN;
    T* ycol = Y + n0 + wn * WN;
    const int64_t mrow0 = m0 + wm * WM;
    if constexpr (EPI == 1)
      // (one copy per format: with the format looked up per value the compiler evaluates all three and selects)
      switch (p.mx_elem) {
        case MX_FP8: igemm_store_interior<T, MI, NJ, WN, SW, false, false, MX_FP8>(acc, bias, stage, yrow, p.N, lane, s1, s2, p, mrow0, phase, ycol); break;
        case MX_INT4: igemm_store_interior<T, MI, NJ, WN, SW, false, false, MX_INT4>(acc, bias, stage, yrow, p.N, lane, s1, s2, p, mrow0, phase, ycol); break;
        default: igemm_store_interior<T, MI, NJ, WN, SW, false, false, MX_FP4>(acc, bias, stage, yrow, p.N, lane, s1, s2, p, mrow0, phase, ycol); break;
      }
    else if constexpr (EPI == 2) {
      const T* const resid = (const T*)p.resid + (m0 + wm * WM) * p.N + n0 + wn * WN;
      if constexpr (RESID_LDS) {
        // the wave's part of resid comes through the operand buffers, 16 bytes a lane at once (rows of WN values, lane order)
        constexpr int CPRO = WN * ES / 16, ROWS = 64 / CPRO;
        static_assert(WM % ROWS == 0, "whole passes");
        char* const area = smem + __builtin_amdgcn_readfirstlane(wave) * (WM * WN * ES);
        const unsigned row_bytes = (unsigned)p.N * (unsigned)ES;
        const __amdgpu_buffer_rsrc_t rR = make_rsrc(resid, (WM - 1) * row_bytes + WN * ES);
        const unsigned off = (unsigned)(lane / CPRO) * row_bytes + (unsigned)(lane % CPRO) * 16u;
#pragma unroll
        for (int r = 0; r < WM / ROWS; ++r) dma_load16s(rR, area + r * 1024, off, (unsigned)(r * ROWS) * row_bytes);
        __builtin_amdgcn_s_waitcnt(vm_imm(0));
        igemm_resid_stats<T, MI, NJ>(acc, bias, reinterpret_cast<const T*>(area), WN, lane, s1, s2);
      } else {
        igemm_resid_stats<T, MI, NJ>(acc, bias, resid, p.N, lane, s1, s2);
      }
    }
    else if constexpr (EPI == 3 || EPI == 4) {
      // companion-tensor sums (EPI 3: IgemmParams::comp_mode 1, EPI 4: comp_mode 2): this lane's chunk of columns is the same in every row it stores (CPRO divides 64)
      constexpr int EPC = 16 / ES, CPRO = WN / EPC;
      static_assert(64 % CPRO == 0, "a lane keeps one column chunk");
      CompSums<EPC> cs;
      const int colc = n0 + wn * WN + (lane % CPRO) * EPC;
#pragma unroll
      for (int t = 0; t < EPC; ++t) {
        cs.s1[t] = 0.0f; cs.s2[t] = 0.0f; cs.p1[t] = 0.0f; cs.p0[t] = 0.0f;
        if (EPI == 4) {
          const float sc = p.comp_bn[colc + t], sh = p.comp_bn[p.N + colc + t];
          const float mu = p.comp_bn[2 * p.N + colc + t], is = p.comp_bn[3 * p.N + colc + t];
          if (sc != 0.0f) {
            const float inv = 1.0f / sc;
            cs.p1[t] = is * inv;
            cs.p0[t] = -(sh * inv + mu) * is;
          }
        }
      }
      igemm_store_interior<T, MI, NJ, WN, SW, false, false, -1, EPI - 2>(acc, bias, stage, yrow, p.N, lane, s1, s2, p, mrow0, phase, ycol, &cs);
#pragma unroll
      for (int t = 0; t < EPC; ++t) {
        for (int off = CPRO; off < 64; off <<= 1) {
          cs.s1[t] += __shfl_xor(cs.s1[t], off, 64);
          cs.s2[t] += __shfl_xor(cs.s2[t], off, 64);
        }
        if (lane < CPRO) {
          sRed[wm][0][wn * WN + lane * EPC + t] = cs.s1[t];
          sRed[wm][1][wn * WN + lane * EPC + t] = cs.s2[t];
        }
      }
    }
    else if (p.partial) igemm_store_interior<T, MI, NJ, WN, SW, true, false>(acc, bias, stage, yrow, p.N, lane, s1, s2, p, mrow0, phase, ycol);
    else if (p.act == ACT_RELU) igemm_store_interior<T, MI, NJ, WN, SW, false, true>(acc, bias, stage, yrow, p.N, lane, s1, s2, p, mrow0, phase, ycol);
    else igemm_store_interior<T, MI, NJ, WN, SW, false, false>(acc, bias, stage, yrow, p.N, lane, s1, s2, p, mrow0, phase, ycol);
  } else if constexpr (DIRECT) {
    // Checked tiles of rows of no whole 16 bytes, most of the columns inside: from the accumulators to memory.  The buffer's range
    // drops the rows past M, an offset past it the columns past N, so a store is one instruction.  (The loop below costs such
    // rows two LDS accesses per value: bf16, 16 x 96 x 96 pixels, 100 -> 99 channels, 3x3: 84 us, with all the checks formed per
    // accumulator 77, so 64; 36 -> 99, 1x1: 38, 37, 14.  A kernel of its own: in the same one the others pay up to 2 % for the code.)
    const int uw = __builtin_amdgcn_readfirstlane(wave), row_bytes = p.N * ES;
    const int64_t um = m0 + uw / WGN * WM;
    const int un = n0 + uw % WGN * WN, cols = min(WN, p.N - un), inside = (int)min((int64_t)WM, p.M - um);
    const __amdgpu_buffer_rsrc_t rY = make_rsrc(Y + um * p.N + un, inside > 0 && cols > 0 ? (inside - 1) * row_bytes + cols * ES : 0);
    unsigned off[NJ];
    float bias[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const bool ok = j * 32 + col_lane < cols;
      off[j] = ok ? (unsigned)(row_lane * row_bytes + (j * 32 + col_lane) * ES) : kOob;
      bias[j] = p.bias && ok ? p.bias[un + j * 32 + col_lane] : 0.0f;
    }
    const bool relu = p.act == ACT_RELU;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int lr = i * 32 + (e >> 2) * 8 + (e & 3);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const float v = round_to_storage<T>(acc[i][j][e] + bias[j]);   // the stored conv result
          if (p.partial) {                       // (columns past N are not stored)
            const float d = lr + row_lane < inside ? v - bias[j] : 0.0f;
            s1[j] += d;
            s2[j] = fmaf(d, d, s2[j]);
          }
          __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(relu ? apply_act(v, ACT_RELU) : v), rY, off[j] + (unsigned)(lr * row_bytes), 0, 0);
        }
      }
  } else {
    // Checked tiles: the conv results are rounded and staged without looking at M, N or the activation; a rolled loop then
    // applies the activation and stores what lies inside.  (With the checks, the activation and the output row formed per
    // accumulator this was 30 to 40 KiB of straight-line code that every workgroup of a launch of a few slabs fetched once: bf16, 24 x
    // 72 x 120 pixels, 3 -> 48 channels 35 -> 30 us, 48 -> 80 at half the side 26 -> 21, 48 -> 3 behind an upsample 27 -> 16.)
    constexpr int EPC = 16 / ES;                 // elements per 16-byte chunk
    constexpr int CPRO = WN / EPC;               // chunks per staged row
    const int cols = min(WN, p.N - (n0 + wn * WN));       // of this wave's part, those inside (may be negative)
    const int64_t mw = m0 + wm * WM;
    float bias[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) bias[j] = p.bias && j * 32 + col_lane < cols ? p.bias[n0 + wn * WN + j * 32 + col_lane] : 0.0f;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int rows = (int)min((int64_t)32, p.M - (mw + i * 32));
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int lr = (e >> 2) * 8 + row_lane + (e & 3);
          const float v = round_to_storage<T>(acc[i][j][e] + bias[j]);   // the stored conv result
          if (p.partial) {                       // (columns past N are not stored)
            const float d = lr < rows ? v - bias[j] : 0.0f;
            s1[j] += d;
            s2[j] = fmaf(d, d, s2[j]);
          }
          Store<T>::st(&stage[lr * SW + j * 32 + col_lane], v);
        }
      auto out_row = [&](int lr) {               // (column strips: interior tiles only)
        const int64_t m = mw + i * 32 + lr;
        return PHASED ? igemm_out_row(p, m, phase, 0) : m;
      };
      if (wide_store) {
#pragma unroll 1
        for (int idx = lane; idx < 32 * CPRO; idx += 64) {
          const int lr = idx / CPRO, ch = idx % CPRO;
          if (lr >= rows || ch * EPC >= cols) continue;
          float f[EPC];
          Store<T>::ldv(&stage[lr * SW + ch * EPC], f);
#pragma unroll
          for (int t = 0; t < EPC; ++t) f[t] = apply_act(f[t], p.act);
          Store<T>::stv(Y + out_row(lr) * p.N + n0 + wn * WN + ch * EPC, f);
        }
      } else if (cols > 0) {
#pragma unroll 1
        for (int idx = lane; idx < rows * cols; idx += 64) {
          const int lr = (int)((unsigned)idx / (unsigned)cols), c = idx - lr * cols;
          const int64_t o = out_row(lr) * p.N + n0 + wn * WN + c;
          const float a = apply_act(Store<T>::ld(&stage[lr * SW + c]), p.act);
          Store<T>::st(&Y[o], a);
          if (p.y_aux) p.y_aux[o] = a;
        }
      }
    }
  }
  if (p.partial && EPI != 3 && EPI != 4) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      float t1 = s1[j] + __shfl_xor(s1[j], 32, 64);
      float t2 = s2[j] + __shfl_xor(s2[j], 32, 64);
      if (lane < 32) {
        sRed[wm][0][wn * WN + j * 32 + col_lane] = t1;
        sRed[wm][1][wn * WN + j * 32 + col_lane] = t2;
      }
    }
  }
  if (p.partial) {
    __syncthreads();
    for (int i = tid; i < 2 * BN; i += WGM * WGN * 64) {
      const int q = i / BN, c = i - q * BN;
      float t = 0.0f;
#pragma unroll
      for (int g = 0; g < WGM; ++g) t += sRed[g][q][c];
      if (n0 + c < p.N) p.partial[(tile_m * 2 + q) * p.N + n0 + c] = t;
    }
  }
}

// ---- hand-scheduled LDS fragment reads of the DMA pipeline -------------------------------
// The compiler orders an LDS read after EVERY outstanding global-to-LDS load (it cannot tell
// the stages apart), which would serialise the pipeline; these reads are therefore issued as
// inline assembly, and the waits on them (lgkmcnt) are placed by hand: LDS reads of a wave
// return in order, so "at most n outstanding" identifies which fragments have arrived.  An
// empty asm with the fragment as in/out operand keeps the MFMAs after the wait.
template <int I, int E, int STRIDE>              // fragments I .. E - 1
struct LdsReadFrags {
  template <int N>
  static __device__ __forceinline__ void run(uint4v (&f)[N], unsigned addr) {
#if defined(__HIP_DEVICE_COMPILE__)             // the host pass only needs the kernel's stub
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f[I]) : "v"(addr), "n"(I * STRIDE));
#endif
    LdsReadFrags<I + 1, E, STRIDE>::run(f, addr);
  }
};
template <int E, int STRIDE>
struct LdsReadFrags<E, E, STRIDE> {
  template <int N>
  static __device__ __forceinline__ void run(uint4v (&)[N], unsigned) {}
};
// f(0), f(1), ... f(N - 1) with the index as a constant
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unroll(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll<N, I + 1>(f);
  }
}
template <int I, int N>
struct TieFrags {
  static __device__ __forceinline__ void run(uint4v (&f)[N]) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(f[I]));
#endif
    TieFrags<I + 1, N>::run(f);
  }
};
template <int N>
struct TieFrags<N, N> {
  static __device__ __forceinline__ void run(uint4v (&)[N]) {}
};
// wait until at most N LDS reads are outstanding, then hand the fragments to the compiler
template <int N, int MI>
__device__ __forceinline__ void lds_wait_tie_a(uint4v (&a)[MI]) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N));
#endif
  TieFrags<0, MI>::run(a);
}
// MFMAs of K-steps K .. KS-1 of one slab; fragments of step k arrived once at most
// (KS-1-k)*(MI+NJ) reads are outstanding
template <typename T, int KS, int K, int MI, int NJ>
struct SlabSteps {
  static __device__ __forceinline__ void run(uint4v (&a)[KS][MI], uint4v (&b)[KS][NJ], floatx16 (&acc)[MI][NJ]) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"((KS - 1 - K) * (MI + NJ)));
#endif
    TieFrags<0, MI>::run(a[K]);
    TieFrags<0, NJ>::run(b[K]);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) mma_step<T>(a[K][i], b[K][j], acc[i][j]);
    __builtin_amdgcn_sched_barrier(0);           // keep these MFMAs ahead of the next step's wait
    SlabSteps<T, KS, K + 1, MI, NJ>::run(a, b, acc);
  }
};
template <typename T, int KS, int MI, int NJ>
struct SlabSteps<T, KS, KS, MI, NJ> {
  static __device__ __forceinline__ void run(uint4v (&)[KS][MI], uint4v (&)[KS][NJ], floatx16 (&)[MI][NJ]) {}
};
template <int K, int KS, int MI, int NJ, int BKB>
struct SlabReads {
  static __device__ __forceinline__ void run(uint4v (&a)[KS][MI], uint4v (&b)[KS][NJ], unsigned addr_a, unsigned addr_b,
                                             const int (&lane_off)[KS]) {
    LdsReadFrags<0, NJ, 32 * BKB>::run(b[K], addr_b + (unsigned)lane_off[K]);
    LdsReadFrags<0, MI, 32 * BKB>::run(a[K], addr_a + (unsigned)lane_off[K]);
    SlabReads<K + 1, KS, MI, NJ, BKB>::run(a, b, addr_a, addr_b, lane_off);
  }
};
template <int KS, int MI, int NJ, int BKB>
struct SlabReads<KS, KS, MI, NJ, BKB> {
  static __device__ __forceinline__ void run(uint4v (&)[KS][MI], uint4v (&)[KS][NJ], unsigned, unsigned, const int (&)[KS]) {}
};

// Which tile a workgroup computes, in what order (ONE_SPLIT: the launch does not split K; TRI: a triangular K range, p.tri).
// The modes are decided at run time, but in instances of their own: every workgroup would pay for them before its first load
// (Monte-Carlo estimates with the modes in every instance and without: batch 5 783 439 -> 427 us, 12 716 576 -> 566, 65 536 1 524 -> 1 516).
struct IgemmTileId { int64_t m; int n, split, phase; };
template <int BM, int BN, bool ONE_SPLIT, bool TRI>
__device__ __forceinline__ IgemmTileId igemm_tile_id(const IgemmParams& p) {
  IgemmTileId t;
  int lb0 = xcd_logical_block((int)blockIdx.x, (int)gridDim.x);
  // triangular products: tile rows differ in work by an order of magnitude, so neighbouring tiles go to different
  // XCDs (the hardware's own round-robin) instead of one contiguous range per XCD, the longest K ranges first
  if (TRI) lb0 = p.tri == 1 ? (int)gridDim.x - 1 - (int)blockIdx.x : (int)blockIdx.x;
  t.phase = 0;
  if (p.phases == 4) { t.phase = lb0 & 3; lb0 >>= 2; }   // the four phases of a tile run side by side: they read the same input
  t.split = ONE_SPLIT ? 0 : lb0 / p.tiles_mn;
  const int lb = ONE_SPLIT ? lb0 : lb0 - t.split * p.tiles_mn;
  // tile order: groups of kGroupM tile rows are walked column by column, so the workgroups in flight on an XCD
  // cover a squarish patch of the output (few distinct operand rows per K slab in its L2) instead of a wide strip
  constexpr int kGroupM = 4;
  const int gsz = kGroupM * p.tiles_n, grp = lb / gsz, in_grp = lb - grp * gsz;
  const int gm = min(p.tiles_mn / p.tiles_n - grp * kGroupM, kGroupM);
  t.n = in_grp / gm;
  t.m = grp * kGroupM + in_grp % gm;
  if (TRI && (p.tri == 3 || p.tri >= 5)) {      // K range [column, K) or [0, column]: walk column by column, the longest first
    const int tiles_m = p.tiles_mn / p.tiles_n;
    t.n = lb / tiles_m;
    t.m = lb - t.n * tiles_m;
    if (p.tri == 5) t.n = p.tiles_n - 1 - t.n;
  }
  return t;
}
// its K range (triangular operands: see IgemmParams::tri); false: no output of the tile is wanted
template <int BM, int BN, bool TRI>
__device__ __forceinline__ bool igemm_k_range(const IgemmParams& p, int64_t m0, int n0, int& k_lo, int& k_hi) {
  k_lo = 0; k_hi = p.K;
  if (!TRI) return true;
  if (p.tri == 1) k_hi = (int)min((int64_t)p.K, min(m0 + BM, (int64_t)n0 + BN));
  else if (p.tri == 2) { if ((int64_t)n0 + BN <= m0) return false; k_lo = (int)m0; }
  else if (p.tri == 3) { if ((int64_t)n0 >= m0 + BM) return false; k_lo = n0; }
  else if (p.tri == 4) k_lo = (int)m0;
  else if (p.tri == 5) k_hi = min(p.K, n0 + BN);
  else if (p.tri == 6) k_lo = n0;
  return true;
}

// Tiles and K ranges of the triangular inverse's products (IgemmParams::tm); TRI_RANGE: those of IgemmParams::tri
enum { TRI_NO = 0, TRI_PAIRS = 1, TRI_LAST = 2, TRI_RANGE = 3 };
struct TriTile { int which, m0, n0, k_lo, k_hi; bool second; };      // matrix; second half of a K range
template <int BM, int BN>
__device__ __forceinline__ bool tri_pair_tile(const IgemmParams& p, TriTile& t) {
  const int tbm = p.tri_b / BM, tbn = p.tri_b / BN;
  int tr, col;                                  // rank of the tile's row in its block, longest K first; column among those of all pairs
  if (gridDim.x > 256) {
    // Several workgroups per compute unit: rows of equal K range together, the longest first, their columns spread over
    // the XCDs.  (With a contiguous range of tiles each, one XCD gets the longest rows alone: two merges of 2048-blocks
    // side by side, LU step of d = 4096, 1.23 against 1.15 ms.)
    const int per_row = (int)gridDim.x / tbm;
    tr = (int)blockIdx.x / per_row;
    col = xcd_logical_block((int)blockIdx.x - tr * per_row, per_row);
    // Two each at most, all resident at once: the second half the other way round, so that a long range shares its compute unit with a short one
    if (gridDim.x <= 512 && tr >= tbm / 2) tr = tbm / 2 + tbm - 1 - tr;
  } else {
    // one each: the longest K range decides, so neighbours share an L2 (d = 2048, 1536: 0.5 to 0.8 % of the step)
    const int lb = xcd_logical_block((int)blockIdx.x, (int)gridDim.x), pair = lb / (tbm * tbn), in_pair = lb - pair * (tbm * tbn);
    tr = in_pair / tbn;
    col = pair * tbn + in_pair - tr * tbn;
  }
  int pair = col / tbn;
  const int tc = col - pair * tbn;
  t.which = pair >= p.tri_pairs ? 1 : 0;
  pair -= t.which * p.tri_pairs;
  const bool lower = t.which ? p.tm[1].lower : p.tm[0].lower;
  const int even = 2 * pair * p.tri_b, odd = even + p.tri_b;
  t.m0 = lower ? odd + (tbm - 1 - tr) * BM : even + tr * BM;
  t.n0 = (lower ? even : odd) + tc * BN;
  t.k_lo = lower ? odd : t.m0;
  t.k_hi = lower ? min(t.m0 + BM, p.tri_d) : odd;
  t.second = false;
  return (lower ? t.m0 : t.n0) < p.tri_d;
}
// The L-shaped shells max(row, column) = 0, 1, ... of BM x BM outputs (two tiles where BN is half of it): those whose range [max, K) is longer than half, two halves each, then
// the others, so that the ranges of either kind are dispatched longest first and the hardware's in-order dispatch balances the rest
template <int BM, int BN>
__device__ __forceinline__ bool tri_last_tile(const IgemmParams& p, TriTile& t) {
  const int sub = BN < BM ? (int)blockIdx.x & 1 : 0, lb = BN < BM ? (int)blockIdx.x >> 1 : (int)blockIdx.x;
  const int half = p.K / BM / 2, n2 = 2 * half * half;
  const bool two = lb < n2;
  const int i = two ? lb >> 1 : lb - n2 / 2;
  int sh = (int)sqrtf((float)i);
  while (sh * sh > i) --sh;
  while ((sh + 1) * (sh + 1) <= i) ++sh;
  const int r = i - sh * sh;                    // 0 .. 2 sh
  t.m0 = (r <= sh ? r : sh) * BM;
  t.n0 = (r <= sh ? sh : r - sh - 1) * BM + sub * BN;
  t.which = two && (lb & 1) ? 1 : 0;
  t.second = t.which == 1;
  const int lo = sh * BM, mid = two ? lo + (p.K - lo) / 64 * 32 : p.K;
  t.k_lo = t.second ? mid : lo;
  t.k_hi = t.second ? p.K : mid;
  return true;
}

// Accumulators that are NaN, as bits (element e of tile (i, j): bit 16 (i NJ + j) + e); 0 after one fused multiply-add per
// accumulator where all are finite.
template <int MI, int NJ>
__device__ __forceinline__ uint64_t nan_bits(const floatx16 (&acc)[MI][NJ]) {
  static_assert(MI * NJ <= 4, "64 bits");
  float z = 0.0f;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) z = fmaf(acc[i][j][e], 0.0f, z);
  uint64_t bits = 0;
  if (z != 0.0f) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) bits |= (uint64_t)(acc[i][j][e] != acc[i][j][e]) << (16 * (i * NJ + j) + e);
  }
  return bits;
}
// those accumulators replaced by value(i, j, e)
template <int MI, int NJ, typename VALUE>
__device__ __forceinline__ void replace_bits(floatx16 (&acc)[MI][NJ], uint64_t bits, VALUE value) {
  while (bits != 0) {
    const int t = __ffsll((unsigned long long)bits) - 1;
    bits &= bits - 1;
    const float v = value(t / (16 * NJ), (t >> 4) % NJ, t & 15);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 16 * (i * NJ + j) + e == t ? v : acc[i][j][e];
  }
}

// INTERIOR: the host guarantees M % BM == 0, N % BN == 0, 16-byte aligned rows, no sigmoid, no
// auxiliary copy and no activation together with statistics, so the epilogue needs no checks.
// DMA: the slabs go from global memory straight into LDS (buffer loads with the LDS
// destination: lane l of a wave writes 16 bytes at base + 16*l, which is exactly the loader's
// linear slot order), three stages deep, so loads run two slabs ahead without holding
// registers.  A wave waits for its own loads of the slab it is about to read (vmcnt), then
// the workgroup barrier makes every wave's loads visible and also guarantees that the stage
// about to be refilled has been read by everybody.
//
// CHUNKS: any channel counts.  p.Cin is the channel count rounded up to whole 16-byte chunks (both operands are stored
// with that row length, zeros behind the channels), and K is walked chunk by chunk across tap borders: chunk q belongs
// to tap q / p.chunks, so every lane keeps the tap of the one chunk per slab it loads (its slot is the same in every
// pass of the loader) and advances it by a slab's CPR chunks.  Nothing but the tail of the last slab is multiplied in
// vain: 9 x 48 channels are 13.5 slabs, where slabs that end with their tap would be 18, and a 3-channel image 2.25
// instead of 9.  Chunks past the end read zeros (both operands: 0 x Inf would be NaN).  What it costs: the pixel
// offsets are formed for every slab, not once per tap, a dozen VALU instructions per 16 bytes loaded.
// Measured (bf16, 24 x 36 x 60 pixels): 48 -> 80 channels, 3x3, 25 us = 143 TFLOP/s, where one thread per output on the
// vector ALUs took 3.4 ms; two such layers at 64 x 64 x 8 forward and backward 140 us against 11.4 ms.
template <typename T, int BM, int BN, int WGM, int WGN, int BKB, bool INTERIOR, bool DMA, int EPI = 0, bool CHUNKS = false, bool DIRECT = false, bool TRI = false>
__global__ __launch_bounds__(WGM * WGN * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_igemm(IgemmParams p) {
  static_assert(!CHUNKS || (!INTERIOR && DMA && EPI == 0), "the chunk walk exists for checked tiles through the DMA pipeline");
  static_assert(EPI == 0 || INTERIOR, "the special epilogues exist for check-free tiles only");
  static_assert(!DIRECT || (!INTERIOR && sizeof(T) == 2), "bf16, checked tiles");
  static_assert(!TRI || (EPI == 0 && !CHUNKS && !DIRECT), "dense products");
  static_assert(WGM * WGN == 4 || WGM * WGN == 8, "four or eight wavefronts per workgroup");
  constexpr int NT = WGM * WGN * 64;            // threads: all of them load, each wavefront owns a WM x WN part of the tile
  static_assert(BKB == 64 || BKB == 128, "slab row bytes");
  constexpr int ES = (int)sizeof(T);
  constexpr int BK = BKB / ES;                  // K elements per slab
  constexpr int CPR = BKB / 16;                 // 16-byte chunks per slab row
  constexpr int RSTEP = NT / CPR;               // rows covered by one pass of the loader threads
  constexpr int WM = BM / WGM, WN = BN / WGN;   // wave tile
  constexpr int MI = WM / 32, NJ = WN / 32;     // 32x32 MFMA tiles per wave
  constexpr int BNL = BN < RSTEP ? RSTEP : BN;  // weight rows loaded: a whole pass at least (rows past N read zeros)
  constexpr int A_CHUNKS = BM / RSTEP, B_CHUNKS = BNL / RSTEP;
  constexpr int SW = WN + 16 / ES;              // staging row stride of the epilogue (elements): +16 bytes
  constexpr int NSTAGE = DMA ? (NT == 512 ? 4 : 3) : 2;   // eight wavefronts: one workgroup per compute unit, LDS for a fourth stage
  constexpr int SLAB_BYTES = NSTAGE * (BM + BNL) * BKB;
  constexpr int STAGE_BYTES = (NT / 64) * 32 * SW * ES;
  __shared__ __attribute__((aligned(16))) char smem[SLAB_BYTES > STAGE_BYTES ? SLAB_BYTES : STAGE_BYTES];
  char* const sA = smem;                        // [NSTAGE][BM*BKB]
  char* const sB = smem + NSTAGE * BM * BKB;    // [NSTAGE][BNL*BKB]
  __shared__ float sRed[WGM][2][BN];            // [wave row][sum | sumsq][column]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const IgemmTileId tile = igemm_tile_id<BM, BN, INTERIOR, TRI>(p);
  const int phase = tile.phase, split = tile.split;
  const int64_t tile_m = tile.m;
  const int tile_n = tile.n;
  const int64_t m0 = tile_m * BM;
  const int n0 = tile_n * BN;
  const int pad_h = p.pad - (phase >> 1), pad_w = p.pad - (phase & 1);
  const int Hin = p.Hv >> p.up, Win = p.Wv >> p.up;
  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rW = make_rsrc(p.w, p.w_bytes);

  // --- loader bookkeeping: thread t moves rows (t / CPR) + RSTEP*i, LDS slot t % CPR of each
  const int slot = tid % CPR;
  const int lrow = tid / CPR;
  const int fsw = BKB == 64 ? ((lrow >> 2) & 3) : ((lrow >> 1) & 7);   // RSTEP*i does not touch these bits
  const int gchunk = slot ^ fsw;
  int a_h[A_CHUNKS], a_w[A_CHUNKS];
  unsigned a_img[A_CHUNKS];                     // byte offset of the sample's image, kOob if the row is past M
  unsigned a_off[A_CHUNKS];                     // byte offset of the current tap's pixel (+ chunk), kOob if padding
#pragma unroll
  for (int i = 0; i < A_CHUNKS; ++i) {
    const int64_t m = m0 + lrow + i * RSTEP;
    const bool ok = m < p.M;
    const unsigned mu = ok ? (unsigned)m : 0u;
    a_w[i] = (int)(mu % (unsigned)p.Wc);
    const unsigned t = mu / (unsigned)p.Wc;
    a_h[i] = (int)(t % (unsigned)p.Hc);
    a_img[i] = ok ? (t / (unsigned)p.Hc) * (unsigned)(Hin * Win) * (unsigned)p.Cin * (unsigned)ES : kOob;
  }
  unsigned b_off[B_CHUNKS];
#pragma unroll
  for (int i = 0; i < B_CHUNKS; ++i) {
    const int row = n0 + lrow + i * RSTEP;
    b_off[i] = row < p.N && lrow + i * RSTEP < BN ? (unsigned)(phase * p.N + row) * (unsigned)p.K * (unsigned)ES + (unsigned)gchunk * 16u : kOob;
  }

  int k_lo, k_hi;
  if (!igemm_k_range<BM, BN, TRI>(p, m0, n0, k_lo, k_hi)) return;
  const int kt_lo = k_lo / BK, kt_hi = (k_hi + BK - 1) / BK;
  const int kt0 = INTERIOR ? kt_lo : max(kt_lo, split * p.slabs_per_split);   // first K slab of this workgroup
  // CHUNKS: the tap and the chunk within it of this lane's next load (q = chunk index along K)
  int q = 0, q_c = 0, q_r = 0, q_s = 0;
  if constexpr (CHUNKS) {
    q = kt0 * CPR + gchunk;
    const int tap = q / p.chunks;
    q_c = q - tap * p.chunks; q_r = tap / p.ksz; q_s = tap - q_r * p.ksz;
  }
  int rs = (kt0 * BK) / p.Cin, ci0 = (kt0 * BK) % p.Cin;                // filter tap and first channel of the next slab to load
  unsigned kbyte = (unsigned)(kt0 * BKB);       // byte offset of the next slab inside a weight row
#define IGEMM_TAP()                                                                                          \
  {                                                                                                          \
    const int r_ = rs / p.ksz, s_ = rs - r_ * p.ksz;                                                         \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i) {                                                   \
      const int hh = a_h[i] * p.stride + r_ - pad_h, ww = a_w[i] * p.stride + s_ - pad_w;                    \
      const bool ok = a_img[i] != kOob && hh >= 0 && hh < p.Hv && ww >= 0 && ww < p.Wv;                      \
      const unsigned pix = (unsigned)((hh >> p.up) * Win + (ww >> p.up));                                    \
      a_off[i] = ok ? a_img[i] + pix * (unsigned)p.Cin * (unsigned)ES + (unsigned)gchunk * 16u : kOob;       \
    }                                                                                                        \
  }
#define IGEMM_LOAD(RA, RB)                                                                                   \
  {                                                                                                          \
    if (ci0 == 0) IGEMM_TAP();                                                                               \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i)                                                     \
        RA[i] = __builtin_amdgcn_raw_buffer_load_b128(rX, a_off[i] + (unsigned)ci0 * (unsigned)ES, 0, 0);    \
    _Pragma("unroll") for (int i = 0; i < B_CHUNKS; ++i)                                                     \
        RB[i] = __builtin_amdgcn_raw_buffer_load_b128(rW, b_off[i] + kbyte, 0, 0);                           \
    ci0 += BK;                                                                                               \
    kbyte += BKB;                                                                                            \
    if (ci0 == p.Cin) { ci0 = 0; ++rs; }                                                                     \
  }
  const int st_off = lrow * BKB + slot * 16;    // this thread's byte offset inside a slab buffer (+ i*RSTEP*BKB)
#define IGEMM_STORE(BUF, RA, RB)                                                                             \
  {                                                                                                          \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i)                                                     \
        *reinterpret_cast<uint4v*>(sA + (BUF) * BM * BKB + st_off + i * RSTEP * BKB) = RA[i];                \
    _Pragma("unroll") for (int i = 0; i < B_CHUNKS; ++i)                                                     \
        *reinterpret_cast<uint4v*>(sB + (BUF) * BN * BKB + st_off + i * RSTEP * BKB) = RB[i];                \
  }
  // fragment reads: lane l wants row (l%32) of a 32-row MFMA tile, chunk 2*ks + l/32;
  // the lane-dependent part of the address is the same for A and B and for every tile
  const int frag_row = lane & 31, frag_c = lane >> 5;
  const int ffr = BKB == 64 ? ((frag_row >> 2) & 3) : ((frag_row >> 1) & 7);
  int lane_off[BKB / 32];
#pragma unroll
  for (int ks = 0; ks < BKB / 32; ++ks) lane_off[ks] = frag_row * BKB + (((ks * 2 + frag_c) ^ ffr) * 16);
#define IGEMM_COMPUTE(BUF)                                                                                   \
  {                                                                                                          \
    _Pragma("unroll") for (int ks = 0; ks < BKB / 32; ++ks) {                                                \
      uint4v a[MI], b[NJ];                                                                                   \
      _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                         \
          a[i] = *reinterpret_cast<const uint4v*>(sA + (BUF) * BM * BKB + (wm * WM + i * 32) * BKB + lane_off[ks]); \
      _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                                         \
          b[j] = *reinterpret_cast<const uint4v*>(sB + (BUF) * BN * BKB + (wn * WN + j * 32) * BKB + lane_off[ks]); \
      _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                         \
        _Pragma("unroll") for (int j = 0; j < NJ; ++j) mma_step<T>(a[i], b[j], acc[i][j]);                   \
    }                                                                                                        \
  }

  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int KT = INTERIOR ? kt_hi - kt0 : min(kt_hi - kt0, p.slabs_per_split);   // (tri launches have one split)
  if (!CHUNKS && ci0 != 0) IGEMM_TAP();          // a split that starts inside a tap (the loaders compute a tap's offsets at its first slab)
  if constexpr (DMA) {
    constexpr int L = A_CHUNKS + B_CHUNKS;       // loads per thread and slab
    static_assert(RSTEP * BKB == NT * 16, "one pass of the loader covers 16 bytes per thread");
    auto dma_chunks = [&](int stg) {
      char* const da = sA + stg * BM * BKB + wave * 1024;
      char* const db = sB + stg * BNL * BKB + wave * 1024;
      const bool in_k = q < p.ksz * p.ksz * p.chunks;
#pragma unroll
      for (int i = 0; i < A_CHUNKS; ++i) {
        const int hh = a_h[i] * p.stride + q_r - pad_h, ww = a_w[i] * p.stride + q_s - pad_w;
        const bool ok = in_k && a_img[i] != kOob && hh >= 0 && hh < p.Hv && ww >= 0 && ww < p.Wv;
        const unsigned pix = (unsigned)((hh >> p.up) * Win + (ww >> p.up));
        dma_load16(rX, da + i * (NT * 16), ok ? a_img[i] + (pix * (unsigned)p.chunks + (unsigned)q_c) * 16u : kOob);
      }
#pragma unroll
      for (int i = 0; i < B_CHUNKS; ++i) dma_load16(rW, db + i * (NT * 16), in_k ? b_off[i] + kbyte : kOob);
      kbyte += BKB;
      q += CPR;
      q_c += CPR;
      while (q_c >= p.chunks) {                  // (at most CPR turns)
        q_c -= p.chunks;
        if (++q_s == p.ksz) { q_s = 0; ++q_r; }
      }
    };
#define IGEMM_DMA(STG)                                                                                       \
  {                                                                                                          \
    if constexpr (CHUNKS) dma_chunks(STG);                                                                   \
    else IGEMM_DMA_TAP(STG);                                                                                 \
  }
#define IGEMM_DMA_TAP(STG)                                                                                   \
  {                                                                                                          \
    if (ci0 == 0) IGEMM_TAP();                                                                               \
    char* const da = sA + (STG) * BM * BKB + wave * 1024;                                                    \
    char* const db = sB + (STG) * BNL * BKB + wave * 1024;                                                   \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i)                                                     \
        dma_load16(rX, da + i * (NT * 16), a_off[i] + (unsigned)ci0 * (unsigned)ES);                         \
    _Pragma("unroll") for (int i = 0; i < B_CHUNKS; ++i)                                                     \
        dma_load16(rW, db + i * (NT * 16), b_off[i] + kbyte);                                                \
    ci0 += BK;                                                                                               \
    kbyte += BKB;                                                                                            \
    if (ci0 == p.Cin) { ci0 = 0; ++rs; }                                                                     \
  }
    constexpr int KS = BKB / 32;
    const unsigned lds_a = (unsigned)(size_t)(lds_char*)sA + (unsigned)(wm * WM * BKB);
    const unsigned lds_b = (unsigned)(size_t)(lds_char*)sB + (unsigned)(wn * WN * BKB);
    IGEMM_DMA(0);
    if (KT > 1) IGEMM_DMA(1);
    if constexpr (NSTAGE == 4) { if (KT > 2) IGEMM_DMA(2); }
    int cur = 0, nxt = NSTAGE - 1;
    for (int kt = 0; kt < KT; ++kt) {
      // vmcnt(n): at most n of this wave's loads outstanding (they complete in order): the slabs issued after slab kt;
      // the other counters are left alone (expcnt 7, lgkmcnt 15)
      if (NSTAGE == 4 && kt + 2 < KT) __builtin_amdgcn_s_waitcnt(((2 * L) & 15) | (((2 * L) >> 4) << 14) | 0x0F70);
      else if (kt + 1 < KT) __builtin_amdgcn_s_waitcnt((L & 15) | ((L >> 4) << 14) | 0x0F70);
      else __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
      uint4v fa[KS][MI], fb[KS][NJ];
      SlabReads<0, KS, MI, NJ, BKB>::run(fa, fb, lds_a + (unsigned)(cur * BM * BKB), lds_b + (unsigned)(cur * BNL * BKB), lane_off);
      if (kt + NSTAGE - 1 < KT) IGEMM_DMA(nxt);
      SlabSteps<T, KS, 0, MI, NJ>::run(fa, fb, acc);
      cur = cur == NSTAGE - 1 ? 0 : cur + 1;
      nxt = nxt == NSTAGE - 1 ? 0 : nxt + 1;
    }
#undef IGEMM_DMA
#undef IGEMM_DMA_TAP
    __syncthreads();                             // every wave is done with the slabs: the epilogue reuses the memory
  } else {
  uint4v ra0[A_CHUNKS], rb0[B_CHUNKS], ra1[A_CHUNKS], rb1[B_CHUNKS];
  IGEMM_LOAD(ra0, rb0);
  if (KT > 1) IGEMM_LOAD(ra1, rb1);
  IGEMM_STORE(0, ra0, rb0);
  __syncthreads();
  for (int kt = 0; kt < KT; kt += 2) {
    // even slab: LDS buffer 0; register set 1 holds slab kt+1; set 0 is free
    if (kt + 2 < KT) IGEMM_LOAD(ra0, rb0);
    IGEMM_COMPUTE(0);
    if (kt + 1 < KT) IGEMM_STORE(1, ra1, rb1);
    __syncthreads();
    if (kt + 1 >= KT) break;
    // odd slab: LDS buffer 1; register set 0 holds slab kt+2; set 1 is free
    if (kt + 3 < KT) IGEMM_LOAD(ra1, rb1);
    IGEMM_COMPUTE(1);
    if (kt + 2 < KT) IGEMM_STORE(0, ra0, rb0);
    __syncthreads();
  }
  }
#undef IGEMM_TAP
#undef IGEMM_LOAD
#undef IGEMM_STORE
#undef IGEMM_COMPUTE

  if constexpr (CHUNKS) {
    // A tap outside the image is a product with zero, NaN for an infinite weight: such an output of a row at the border is
    // summed again over the taps inside (at the pace of one thread per output; nothing but infinities and NaN gets here).
    const uint64_t bits = p.ksz > 1 ? nan_bits(acc) : 0;
    constexpr int EPC = 16 / ES;
    replace_bits(acc, bits, [&](int i, int j, int e) {
      const int64_t m = m0 + wm * WM + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
      const int n = n0 + wn * WN + j * 32 + (lane & 31);
      const unsigned mu = (unsigned)m, t = mu / (unsigned)p.Wc, img = t / (unsigned)p.Hc;
      const int h0 = (int)(t - img * (unsigned)p.Hc) * p.stride - pad_h, w0 = (int)(mu - t * (unsigned)p.Wc) * p.stride - pad_w;
      if (m >= p.M || n >= p.N || (h0 >= 0 && w0 >= 0 && h0 + p.ksz <= p.Hv && w0 + p.ksz <= p.Wv)) return __builtin_nanf("");
      const T* const x = reinterpret_cast<const T*>(p.x) + (int64_t)img * Hin * Win * p.Cin;
      const T* const wr = reinterpret_cast<const T*>(p.w) + ((int64_t)phase * p.N + n) * p.K;
      const int k_end = min((kt0 + KT) * BK, p.K);
      float v = 0.0f;
      for (int k = kt0 * BK; k < k_end && v == v; k += EPC) {  // (a chunk lies in one tap; NaN stays NaN)
        const int tap = k / p.Cin, ci = k - tap * p.Cin, r = tap / p.ksz, hh = h0 + r, ww = w0 + tap - r * p.ksz;
        if (hh < 0 || hh >= p.Hv || ww < 0 || ww >= p.Wv) continue;
        const T* const px = x + ((int64_t)(hh >> p.up) * Win + (ww >> p.up)) * p.Cin + ci;
        for (int c = 0; c < EPC; ++c) v = fmaf(Store<T>::ld(px + c), Store<T>::ld(wr + k + c), v);
      }
      return v;
    });
  }
  if constexpr (!INTERIOR) {
    if (p.split_out) {
      float* __restrict__ P = p.split_out + (int64_t)split * p.M * p.N;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int col = n0 + wn * WN + j * 32 + (lane & 31);
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int64_t m = m0 + wm * WM + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
            if (m < p.M && col < p.N) P[m * p.N + col] = acc[i][j][e];
          }
        }
      return;
    }
  }
  static_assert(EPI != 2 || BM * BN * ES <= SLAB_BYTES, "resid");
  igemm_epilogue<T, BM, BN, WGM, WGN, INTERIOR, EPI, CHUNKS, EPI == 2, DIRECT>(acc, p, smem, sRed, m0, n0, tile_m, phase);
}

// Operands that lie in LDS with K outermost, read transposed (ds_read_b64_tr_b16: within 16 lanes, lane 4j+q addresses 4 columns
// of k-row j, lane i receives column i of k-rows 0..3): k-rows 0..3 and 4..7 of a lane's column
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
struct TrFrag { uint2v lo, hi; };

__device__ __forceinline__ void tr_tie(TrFrag& f) {   // (as TieFrags)
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(f.lo), "+v"(f.hi));
#endif
}
template <int OFF, int STEP>                     // STEP: bytes of four k-rows
__device__ __forceinline__ void tr_read_at(TrFrag& f, unsigned addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.lo) : "v"(addr), "n"(OFF));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.hi) : "v"(addr), "n"(OFF + STEP));
#endif
}

// ---------------------------------------------------------------------------
// Dense bf16 products, check-free tiles: y[m][n] = x[m][:] w[n][:]^T, without the taps of k_igemm.
//
// The slabs are k_igemm's (64 bytes of K, straight from global memory into a ring of NSTAGE LDS stages, the same swizzle),
// the schedule is not: a K-step's MFMAs run on fragments that are already in registers while the next K-step's are read
// and the slab after the next two is asked for, one instruction between two MFMAs.  The workgroup barrier (slab kt + 1 has
// landed everywhere; the stage of slab kt - 1 is free) stands between the two K-steps of slab kt, so neither an LDS latency
// nor a burst of loads at the vector memory's issue port lies between a barrier and the next MFMA.
// What bounds it is power: at 16 384 x 4 096 x 4 096 the matrix cores are busy 78 % of the cycles at 1.46 GHz, and the
// loads alone cost 0.3 GHz (without them: 89 % at 1.78 GHz, 1.68 PFLOP/s); their place between the MFMAs, s_setprio, and
// tile orders of 4 to 8 rows made no difference of 2 %, orders of 2 or 16 rows cost 4 %.
// Measured against k_igemm's schedule with the same tiles (which read a slab's fragments behind the barrier that the slab's
// MFMAs wait for): 4 096^3 143 -> 126 us, the quantising product of 16 384 x 4 096 x 4 096 683 -> 594 us, the one that only sums
// its deviations 586 -> 537 us.  1 us a slab of 256 x 256 outputs, 0.55 us of it MFMAs at the full clock.
// Which tiles come here, and with how many stages: dense_stages and launch_conv_mfma.
// KN: the second operand lies [k][n] (launch_dense_kn): a slab is 32 k-rows of it, read with the transposing LDS reads; same sums in
// the same order.  d = 4 096: 126 us as well.  KG = 2: dense_halves.
// ---------------------------------------------------------------------------
template <int BM, int BN, int WGM, int WGN, int NSTAGE, int EPI = 0, bool TRI = false, bool KN = false, int KG = 1>
__global__ __launch_bounds__(WGM * WGN * 64 * KG) __attribute__((amdgpu_waves_per_eu(2))) void k_dense(IgemmParams p) {
  constexpr int NT = WGM * WGN * 64, BKB = 64, BK = 32;
  constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NJ = WN / 32;
  constexpr int RSTEP = NT / 4, AC = BM / RSTEP, BC = BN / RSTEP, L = AC + BC;   // loads per thread and slab
  static_assert(NSTAGE == 3 || NSTAGE == 4, "the waits below");
  constexpr int SA = BM * BKB, SB = BN * BKB, SW = WN + 8;
  constexpr int SLAB_BYTES = NSTAGE * (SA + SB), STAGE_BYTES = (NT / 64) * 32 * SW * 2;
  __shared__ __attribute__((aligned(16))) char smem_all[KG == 1 && SLAB_BYTES < STAGE_BYTES ? STAGE_BYTES : KG * SLAB_BYTES];
  __shared__ float sRed[WGM][2][BN];
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
  char* const smem = smem_all + kg * SLAB_BYTES;
  char* const sB = smem + NSTAGE * SA;
  const int tid = KG == 1 ? (int)threadIdx.x : (int)threadIdx.x - kg * NT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const IgemmTileId tile = igemm_tile_id<BM, BN, true, TRI>(p);
  const int64_t m0 = tile.m * BM;
  const int n0 = tile.n * BN;
  int k_lo, k_hi;
  if (!igemm_k_range<BM, BN, TRI>(p, m0, n0, k_lo, k_hi)) return;
  const int KT = ((k_hi + BK - 1) / BK - k_lo / BK) / KG, kt0 = k_lo / BK + kg * KT;
  const unsigned row_bytes = (unsigned)p.K * 2u;
  const unsigned w_row = KN ? (unsigned)p.N * 2u : row_bytes;
  const int grp = KN ? (int)(m0 / p.kn_group) : 0;
  const __amdgpu_buffer_rsrc_t rX = make_rsrc((const char*)p.x + (m0 - (int64_t)grp * p.kn_group) * row_bytes, BM * row_bytes);
  const __amdgpu_buffer_rsrc_t rW = KN ? make_rsrc((const char*)p.w + (int64_t)grp * p.K * w_row + n0 * 2, (unsigned)(p.K - 1) * w_row + BN * 2u)
                                       : make_rsrc((const char*)p.w + (int64_t)n0 * row_bytes, BN * row_bytes);
  const int lrow = tid >> 2;
  const unsigned off0 = (unsigned)lrow * row_bytes + (unsigned)(((tid & 3) ^ ((lrow >> 2) & 3)) * 16);   // rows lrow + i RSTEP: the same swizzle
  unsigned kbyte = (unsigned)kt0 * BKB;          // of the next slab to load
  // KN: a slab is 32 k-rows of BN values, 16-byte chunk c of row k in slot c ^ 4 (k & 3), so that the four rows of a
  // transposing read lie in different banks; 64 bytes of a row stay together
  constexpr int CPN = BN / 8, KROWS = NT / CPN;  // chunks per k-row; k-rows per pass
  static_assert(!KN || (KROWS % 4 == 0 && (BN == 128 || BN == 256)), "the swizzle is the same in every pass");
  const int krow = tid / CPN;
  const unsigned offw = KN ? (unsigned)krow * w_row + (unsigned)(((tid % CPN) ^ (4 * (krow & 3))) * 16) : off0;
  unsigned wbyte = (unsigned)kt0 * (KN ? BK * w_row : (unsigned)BKB);
  auto load = [&](auto c_, int stg) {            // load c of a slab into stage stg
    constexpr int c = decltype(c_)::value;
    if constexpr (c < AC) dma_load16s(rX, smem + stg * SA + c * (NT * 16) + wave * 1024, off0 + (unsigned)(c * RSTEP) * row_bytes, kbyte);
    else dma_load16s(rW, sB + stg * SB + (c - AC) * (NT * 16) + wave * 1024, offw + (unsigned)((c - AC) * (KN ? KROWS : RSTEP)) * w_row, wbyte);
    if constexpr (c == L - 1) { kbyte += BKB; wbyte += KN ? BK * w_row : (unsigned)BKB; }
  };
  const int fr = lane & 31, fsw = (fr >> 2) & 3;
  unsigned fa_addr[2], fb_addr[2];               // of this lane's fragments of either K-step, stage 0
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const unsigned o = (unsigned)(fr * BKB + (((ks * 2 + (lane >> 5)) ^ fsw) * 16));
    fa_addr[ks] = (unsigned)(size_t)(lds_char*)smem + (unsigned)(wm * WM * BKB) + o;
    fb_addr[ks] = (unsigned)(size_t)(lds_char*)sB + (unsigned)(wn * WN * BKB) + o;
  }
  unsigned tr_addr[KN ? NJ : 1];                 // KN: of this lane's transposing reads, K-step 0, stage 0 (wave column 32 j: 64 bytes)
  if constexpr (KN) {
    const int kr = (lane & 15) >> 2;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      tr_addr[j] = (unsigned)(size_t)(lds_char*)sB + (unsigned)(((lane >> 5) * 8 + kr) * (BN * 2) + (((wn * WN / 32 + j) ^ kr) * 64) +
                                                                ((lane >> 4) & 1) * 32 + (lane & 3) * 8);
  }
  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  uint4v fa[2][MI], fb[KN ? 1 : 2][NJ];
  TrFrag ft[2][KN ? NJ : 1];
  auto read_b = [&](auto ks_, auto j0_, auto j1_, int stg) {   // fragments j0 .. j1 - 1 of K-step ks
    constexpr int ks = decltype(ks_)::value, j0 = decltype(j0_)::value, j1 = decltype(j1_)::value;
    if constexpr (KN) unroll<j1 - j0>([&](auto j_) {
      constexpr int j = j0 + decltype(j_)::value;
      tr_read_at<ks * 16 * BN * 2, 4 * BN * 2>(ft[ks][j], tr_addr[j] + (unsigned)(stg * SB));
    });
    else LdsReadFrags<j0, j1, 32 * BKB>::run(fb[ks], fb_addr[ks] + (unsigned)(stg * SB));
  };
  auto wait_frags = [&](auto ks_) {
    constexpr int ks = decltype(ks_)::value;
    lds_wait_tie_a<0, MI>(fa[ks]);
    if constexpr (KN) unroll<NJ>([&](auto j_) { tr_tie(ft[ks][decltype(j_)::value]); });
    else lds_wait_tie_a<0, NJ>(fb[ks]);
  };
  // K-step ks: between its MFMAs the fragment reads of the other K-step (stage rstg; waited for behind the last MFMA, so
  // that nothing is in flight where the loop turns) and its half of a slab's loads (stage lstg; none if negative)
  auto step = [&](auto ks_, auto read_, int rstg, int lstg) {
    constexpr int ks = decltype(ks_)::value;
    constexpr bool read = decltype(read_)::value;
    constexpr int MM = MI * NJ, H = NSTAGE == 3 ? L : (L + 1) / 2, C0 = ks == 1 ? 0 : H, NL = ks == 1 ? H : L - H;
    const unsigned ra = fa_addr[ks ^ 1] + (unsigned)(rstg * SA);
    __builtin_amdgcn_sched_barrier(0);
    unroll<MM>([&](auto q_) {
      constexpr int q = decltype(q_)::value;
      if constexpr (KN) {
        const TrFrag& t = ft[ks][q % NJ];
        mma_step<bf16_t>(fa[ks][q / NJ], uint4v{t.lo.x, t.lo.y, t.hi.x, t.hi.y}, acc[q / NJ][q % NJ]);
      } else mma_step<bf16_t>(fa[ks][q / NJ], fb[ks][q % NJ], acc[q / NJ][q % NJ]);
      if constexpr (read) {                      // two reads behind each of the first MFMAs
        constexpr int r0 = 2 * q, r1 = 2 * q + 2;
        constexpr int b0 = r0 < NJ ? r0 : NJ, b1 = r1 < NJ ? r1 : NJ;
        constexpr int a0 = r0 < NJ ? 0 : (r0 - NJ < MI ? r0 - NJ : MI), a1 = r1 < NJ ? 0 : (r1 - NJ < MI ? r1 - NJ : MI);
        read_b(std::integral_constant<int, ks ^ 1>{}, std::integral_constant<int, b0>{}, std::integral_constant<int, b1>{}, rstg);
        LdsReadFrags<a0, a1, 32 * BKB>::run(fa[ks ^ 1], ra);
      }
      if constexpr (NL > 0) {
        if (lstg >= 0)
          unroll<NL>([&](auto c_) {
            constexpr int c = decltype(c_)::value;
            if constexpr ((2 * c + 1) * MM / (2 * NL) == q) load(std::integral_constant<int, C0 + c>{}, lstg);
          });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (read) wait_frags(std::integral_constant<int, ks ^ 1>{});
  };
  constexpr std::integral_constant<int, 0> k0{};
  constexpr std::integral_constant<int, 1> k1{};
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  unroll<NSTAGE - 1>([&](auto g_) {
    constexpr int g = decltype(g_)::value;
    if (g < KT) unroll<L>([&](auto c_) { load(c_, g); });
  });
  // vmcnt(n): at most n of this wave's loads outstanding (they complete in order)
  if (NSTAGE == 4 && KT > 2) __builtin_amdgcn_s_waitcnt(vm_imm(2 * L));
  else if (KT > 1) __builtin_amdgcn_s_waitcnt(vm_imm(L));
  else __builtin_amdgcn_s_waitcnt(vm_imm(0));
  __builtin_amdgcn_s_barrier();
  read_b(k0, k0, std::integral_constant<int, NJ>{}, 0);
  LdsReadFrags<0, MI, 32 * BKB>::run(fa[0], fa_addr[0]);
  wait_frags(k0);
  int cur = 0, pend = -1;                        // stage of slab kt; stage whose loads are half issued
  for (int kt = 0; kt + 1 < KT; ++kt) {
    step(k0, yes, cur, pend);
    // issued so far: the slabs up to kt + NSTAGE - 2; slab kt + 1 has to be there
    if (NSTAGE == 4 && kt + 2 < KT) __builtin_amdgcn_s_waitcnt(vm_imm(L));
    else __builtin_amdgcn_s_waitcnt(vm_imm(0));
    __builtin_amdgcn_s_barrier();                // (every wave has its last fragments of slab kt: the stage of slab kt - 1 is free)
    const int prev = cur == 0 ? NSTAGE - 1 : cur - 1;
    pend = kt + NSTAGE - 1 < KT ? prev : -1;
    cur = cur == NSTAGE - 1 ? 0 : cur + 1;
    step(k1, yes, cur, pend);
  }
  step(k0, yes, cur, -1);
  step(k1, no, 0, -1);
  __syncthreads();                               // every wave is done with the slabs: the epilogue reuses the memory
  if constexpr (KG == 2) {                       // the second half's sums, 16 bytes a lane at once, to the first
    static_assert(BM * BN * 4 <= SLAB_BYTES && EPI == 0, "the second half's own stages hold its sums; no barrier follows");
    float4v* const sum = reinterpret_cast<float4v*>(smem_all + SLAB_BYTES) + wave * (MI * NJ * 4 * 64) + lane;
    if (kg == 1) {
#pragma unroll
      for (int t = 0; t < MI * NJ * 4; ++t) {
        const floatx16& c = acc[t / 4 / NJ][t / 4 % NJ];
        sum[t * 64] = float4v{c[4 * (t % 4)], c[4 * (t % 4) + 1], c[4 * (t % 4) + 2], c[4 * (t % 4) + 3]};
      }
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int t = 0; t < MI * NJ * 4; ++t) {
      const float4v v = sum[t * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t / 4 / NJ][t / 4 % NJ][4 * (t % 4) + e] += v[e];
    }
  }
  static_assert(EPI != 2 || BM * BN * 2 <= SLAB_BYTES, "resid");
  igemm_epilogue<bf16_t, BM, BN, WGM, WGN, true, EPI, false, true>(acc, p, smem, sRed, m0, n0, tile.m);
}

// ---------------------------------------------------------------------------
// Binary32 products and convolutions (CONV: the gather of k_igemm) on the bf16 matrix cores.
//
// Every value is cut into three bfloat16 parts on its way into LDS, x = h + m + l (each rounded to nearest, the remainders
// exact: |m| <= 2^-8 |x|, |l| <= 2^-16 |x|, h + m + l = x), and a product is the six MFMAs hh + hm + mh + mm + hl + lh; what
// is dropped, ml + lm + ll, is of the size of one binary32 rounding of the product at worst.  hh goes to an accumulator of
// its own, the five small ones to a second one whose roundings are their own size: a K of 16 rounds the sum once, where
// eight binary32 MFMAs round it eight times.  Six bf16 MFMAs take 192 cycles for that K, the eight binary32 ones 512.
// Measured at d = 4096: 0.65 ms = 211 TFLOP/s against 1.01 ms = 136 (87 % of the binary32 MFMA's rate), the matrix cores
// busy 75 % of the cycles at the 1.6 GHz that the power limit leaves; errors at the rule in launch_conv_mfma.
//
// A workgroup is WGM x WGN wavefronts of 64 x 64 outputs (32 x 64 where there are only 64 columns).  Slabs of 16 k's are
// loaded into registers two slabs ahead, cut into parts between the MFMAs of the slab before (the split is a third of the VALU
// issue slots that the MFMAs leave) and stored to the next of three LDS stages, with one barrier per slab: a stage's last
// read lies before the barrier of the slab, its next store behind that of the slab after.  LDS: [stage][part][32-row block] of
// 1 KiB in fragment order, chunk c (8 of the 16 k's) of row r at 512 c + (16 r ^ 128 c): a fragment read is 1 KiB in lane
// order, and the 8-byte stores of 8 rows x 4 quarters fall into 64 different banks.
//
// A workgroup that meets an operand below 2^-110 other than zero, whose last part would end below the smallest bfloat16
// denormal, computes its tile again with the binary32 MFMA: such a value may be all there is of an output, whatever else its
// row holds.  (The bf16 MFMA flushes no denormals: 256-term sums of 2^-63 x 2^-63 products come out to 1.2 x 2^-24 of the sum
// of magnitudes, as at any size.  The check is 6 VALU instructions per 16 bytes, 1.4 % of a QR step of d = 4096.)  So does one
// with a sum that is no finite number: a value that rounds to infinity has no parts, the product of two parts rounded up may
// lie beyond the range where the product of the values does not, and where both accumulators leave it with different signs
// their sum would be NaN for an infinity.
// ---------------------------------------------------------------------------
template <int BM, int BN, int WGM, int WGN, bool INTERIOR, int EPI = 0, bool CONV = false, int TRI = TRI_NO>
__global__ __launch_bounds__(WGM * WGN * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_split(IgemmParams p) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NJ = WN / 32;
  constexpr int RSTEP = NT / 4;                  // rows per loader pass: four lanes of 16 bytes share a row
  constexpr int AC = BM / RSTEP, BC = BN / RSTEP;
  constexpr int PA = BM * 32, PB = BN * 32, STAGE = 3 * (PA + PB);
  constexpr int SW = WN + 4, STAGE_BYTES = (NT / 64) * 32 * SW * 4;
  __shared__ __attribute__((aligned(16))) char smem[3 * STAGE > STAGE_BYTES ? 3 * STAGE : STAGE_BYTES];
  __shared__ float sRed[WGM][2][BN];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  static_assert(TRI == TRI_NO || (EPI == 0 && !CONV), "dense products");
  constexpr bool WALK = TRI == TRI_PAIRS || TRI == TRI_LAST;
  static_assert(!WALK || INTERIOR, "check-free tiles");
  IgemmTileId tile = {};
  int64_t m0;
  int n0, k_lo, k_hi;
  const int ldx = WALK ? p.ldx : p.K, ldw = WALK ? p.ldw : p.K;
  float* yt = nullptr;
  if constexpr (WALK) {
    TriTile t;
    if (!(TRI == TRI_PAIRS ? tri_pair_tile<BM, BN>(p, t) : tri_last_tile<BM, BN>(p, t))) return;
    m0 = t.m0; n0 = t.n0; k_lo = t.k_lo; k_hi = t.k_hi;
    p.x = t.which ? p.tm[1].x : p.tm[0].x;
    p.w = t.which ? p.tm[1].w : p.tm[0].w;
    p.y = t.which ? p.tm[1].y : p.tm[0].y;
    yt = t.which ? p.tm[1].yt : p.tm[0].yt;
  } else {
    tile = igemm_tile_id<BM, BN, INTERIOR, TRI == TRI_RANGE>(p);
    m0 = tile.m * BM;
    n0 = tile.n * BN;
    if (!igemm_k_range<BM, BN, TRI == TRI_RANGE>(p, m0, n0, k_lo, k_hi)) return;
  }
  // slabs of 16 (K ranges start at multiples of 32)
  const int kt0 = INTERIOR ? k_lo / 16 : max(k_lo / 16, tile.split * p.slabs_per_split);
  const int KT = INTERIOR ? (k_hi + 15) / 16 - kt0 : min((k_hi + 15) / 16 - kt0, p.slabs_per_split);
  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rW = make_rsrc(p.w, p.w_bytes);
  const int lrow = tid >> 2, kq = tid & 3;
  // GEMM row m of A: where its K-bytes start (dense), or its pixel (CONV: grid position, image; a slab lies in one tap)
  struct Row { int h, w; unsigned img; };
  const int pad_h = p.pad - (tile.phase >> 1), pad_w = p.pad - (tile.phase & 1);
  auto row_of = [&](int64_t m) {
    Row x = {0, 0, kOob};
    if (m < p.M) {
      if constexpr (CONV) {
        const unsigned mu = (unsigned)m, t = mu / (unsigned)p.Wc, n = t / (unsigned)p.Hc;
        x.w = (int)(mu - t * (unsigned)p.Wc);
        x.h = (int)(t - n * (unsigned)p.Hc);
        x.img = n * (unsigned)((p.Hv >> p.up) * (p.Wv >> p.up)) * (unsigned)p.Cin * 4u;
      } else {
        x.img = (unsigned)m * (unsigned)ldx * 4u;
      }
    }
    return x;
  };
  auto tap_off = [&](const Row& x, int tap) {    // byte offset of the row's pixel under a tap (CONV)
    const int r_ = tap / p.ksz, s_ = tap - r_ * p.ksz;
    const int hh = x.h * p.stride + r_ - pad_h, ww = x.w * p.stride + s_ - pad_w;
    const bool ok = x.img != kOob && hh >= 0 && hh < p.Hv && ww >= 0 && ww < p.Wv;
    return ok ? x.img + (unsigned)((hh >> p.up) * (p.Wv >> p.up) + (ww >> p.up)) * (unsigned)p.Cin * 4u : kOob;
  };
  int tap = CONV ? kt0 * 16 / p.Cin : 0, ci = CONV ? kt0 * 16 - tap * p.Cin : kt0 * 16;   // of the next slab to load
  unsigned off[AC + BC];                         // byte offset of this lane's next 16 bytes of each row
  Row ar[CONV ? AC : 1];
#pragma unroll
  for (int i = 0; i < AC; ++i) {
    const Row x = row_of(m0 + lrow + i * RSTEP);
    if constexpr (CONV) ar[i] = x;
    off[i] = (CONV ? tap_off(x, tap) : x.img) + (unsigned)(ci * 4 + kq * 16);      // (kOob plus a row's bytes stays out of range)
  }
#pragma unroll
  for (int i = 0; i < BC; ++i) {
    const int n = n0 + lrow + i * RSTEP;
    off[AC + i] = n < p.N ? (unsigned)(tile.phase * p.N + n) * (unsigned)ldw * 4u + (unsigned)(kt0 * 64 + kq * 16) : kOob;
  }
  auto next_slab = [&]() {                       // CONV: behind the loads of a slab
    if constexpr (CONV) {
      ci += 16;
      if (ci == p.Cin) {
        ci = 0;
        ++tap;
#pragma unroll
        for (int i = 0; i < AC; ++i) off[i] = tap_off(ar[i], tap) + (unsigned)(kq * 16);
      }
    }
  };
  uint4v r[AC + BC];
  unsigned lo = ~0u;
  auto load = [&](int i) {                       // (past the last slab: values that nobody uses)
    r[i] = __builtin_amdgcn_raw_buffer_load_b128(i < AC ? rX : rW, off[i], 0, 0);
    off[i] += 64;
  };
  const int sc = kq >> 1;
  char* const st = smem + (lrow >> 5) * 1024 + sc * 512 + (((lrow & 31) * 16) ^ (sc * 128)) + (kq & 1) * 8;
  auto split = [&](int stage, int i) {           // the four values of one load: three 8-byte stores
    char* const dst = st + stage + (i < AC ? i * (RSTEP * 32) : 3 * PA + (i - AC) * (RSTEP * 32));
    const float4v f = __builtin_bit_cast(float4v, r[i]);
    track_smallest(lo, r[i]);
    float r0 = f[0], r1 = f[1], r2 = f[2], r3 = f[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint32_t w0 = pack_bf16(r0, r1), w1 = pack_bf16(r2, r3);
      *reinterpret_cast<uint2*>(dst + q * (i < AC ? PA : PB)) = make_uint2(w0, w1);
      r0 -= __uint_as_float(w0 << 16); r1 -= __uint_as_float(w0 & 0xFFFF0000u);
      r2 -= __uint_as_float(w1 << 16); r3 -= __uint_as_float(w1 & 0xFFFF0000u);
    }
  };
  floatx16 acc[MI][NJ], low[MI][NJ];             // the sum of the hh, of the five small products
  auto clear = [&](floatx16 (&c)[MI][NJ]) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) c[i][j][e] = 0.0f;
  };
  clear(acc);
  clear(low);
  const int f_off = (lane >> 5) * 512 + (((lane & 31) * 16) ^ ((lane >> 5) * 128));
  const char* const fa = smem + wm * WM * 32 + f_off;
  const char* const fb = smem + 3 * PA + wn * WN * 32 + f_off;
  uint4v a[3][MI], b[3][NJ];
  auto read_a = [&](int stage, int q) {
#pragma unroll
    for (int i = 0; i < MI; ++i) a[q][i] = *reinterpret_cast<const uint4v*>(fa + stage + q * PA + i * 1024);
  };
  auto read_b = [&](int stage, int q) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[q][j] = *reinterpret_cast<const uint4v*>(fb + stage + q * PB + j * 1024);
  };
  auto mma = [&](int qa, int qb) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) mma_step<bf16_t>(a[qa][i], b[qb][j], qa + qb == 0 ? acc[i][j] : low[i][j]);
  };
#pragma unroll
  for (int i = 0; i < AC + BC; ++i) load(i);
  next_slab();
#pragma unroll
  for (int i = 0; i < AC + BC; ++i) { split(0, i); load(i); }
  next_slab();
  __syncthreads();
  read_b(0, 0); read_a(0, 0);
  int cur = 0, nxt = STAGE;
  for (int kt = 1; kt < KT; ++kt) {
    // A slab: its first fragments are in registers.  The next slab goes into the stage read two slabs ago (every wave has
    // passed the barrier of the slab in between, so that stage is free) and its first fragments are fetched behind the
    // last two products.
    // (the scheduling barriers keep the reads ahead of the MFMAs they would otherwise be sunk to)
    read_b(cur, 1); read_a(cur, 1); read_b(cur, 2); read_a(cur, 2);
    __builtin_amdgcn_sched_barrier(0);
    mma(0, 0); mma(0, 1); mma(1, 0); mma(1, 1);
#pragma unroll
    for (int i = 0; i < AC + BC; ++i) { split(nxt, i); load(i); }
#pragma unroll
    for (int g = 0; g < 4 * MI * NJ; ++g) {      // the split spread between the MFMAs
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, (AC + BC) * 26 / (4 * MI * NJ) + 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    uint4v a2[MI], b2[NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i) a2[i] = a[0][i];
#pragma unroll
    for (int j = 0; j < NJ; ++j) b2[j] = b[0][j];
    read_b(nxt, 0); read_a(nxt, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) mma_step<bf16_t>(a2[i], b[2][j], low[i][j]);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) mma_step<bf16_t>(a[2][i], b2[j], low[i][j]);
    __builtin_amdgcn_sched_barrier(0);
    next_slab();
    cur = nxt;
    nxt = nxt == 2 * STAGE ? 0 : nxt + STAGE;
  }
  read_b(cur, 1); read_a(cur, 1); read_b(cur, 2); read_a(cur, 2);
  mma(0, 0); mma(0, 1); mma(1, 0); mma(1, 1); mma(0, 2); mma(2, 0);
  const bool odd = add_not_finite(acc, low) || parts_inexact(lo);
  if (__syncthreads_or(odd) != 0) {
    // fragments straight from global memory: lane l holds four k's of row l % 32, the same ones on both sides
    clear(acc);
    for (int h = 0; h < 2 * KT; ++h) {           // eight k's
      const int k = (kt0 * 2 + h) * 8, tap_x = CONV ? k / p.Cin : 0;
      uint4v f[MI + NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const Row x = row_of(m0 + wm * WM + i * 32 + (lane & 31));
        const unsigned o = (CONV ? tap_off(x, tap_x) : x.img) + (unsigned)((k - tap_x * p.Cin) * 4 + (lane >> 5) * 16);
        f[i] = __builtin_amdgcn_raw_buffer_load_b128(rX, o, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int n = n0 + wn * WN + j * 32 + (lane & 31);
        const unsigned o = n < p.N ? (unsigned)(tile.phase * p.N + n) * (unsigned)ldw * 4u + (unsigned)(k * 4 + (lane >> 5) * 16) : kOob;
        f[MI + j] = __builtin_amdgcn_raw_buffer_load_b128(rW, o, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) mma_step<float>(f[i], f[MI + j], acc[i][j]);
    }
  }
  if constexpr (!INTERIOR) {
    if (p.split_out) {
      float* __restrict__ P = p.split_out + (int64_t)tile.split * p.M * p.N;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int col = n0 + wn * WN + j * 32 + (lane & 31);
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int64_t m = m0 + wm * WM + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
            if (m < p.M && col < p.N) P[m * p.N + col] = acc[i][j][e];
          }
        }
      return;
    }
  }
  if constexpr (TRI == TRI_PAIRS) {
    if (p.negate) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = -acc[i][j];
    }
    if (yt) {                                    // four rows of a column are 16 bytes of the transpose
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4v*>(yt + (int64_t)(n0 + wn * WN + j * 32 + (lane & 31)) * p.N + m0 + wm * WM + i * 32 + g * 8 + (lane >> 5) * 4) =
                float4v{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
    }
  }
  igemm_epilogue<float, BM, BN, WGM, WGN, INTERIOR, EPI>(acc, p, smem, sRed, m0, n0, tile.m, tile.phase);
}

// y = act(round(sum over splits of partial[split] + bias)) for split-K launches
template <typename T>
__global__ void k_splitk_finish(const float* __restrict__ partial, int splits, int64_t M, int N, const float* __restrict__ bias,
                                int act, T* __restrict__ y, float* __restrict__ y_aux) {
  const int64_t total = M * N;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    float acc = 0.0f;
#pragma unroll 8
    for (int sp = 0; sp < splits; ++sp) acc += partial[(int64_t)sp * total + i];
    if (bias) acc += bias[(int)(i % N)];
    const float a = apply_act(round_to_storage<T>(acc), act);
    Store<T>::st(y + i, a);
    if (y_aux) y_aux[i] = a;
  }
}

template <typename T, int MI, int NJ>
__device__ __forceinline__ void mma_group(const uint4v (&a)[MI], const uint4v (&b)[NJ], floatx16 (&acc)[MI][NJ]) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) mma_step<T>(a[i], b[j], acc[i][j]);
}

// A-fragment reads of the patch kernel: one address per 32-pixel tile, K-step selected by ^ 32
template <int I, int N>
struct Conv3Reads {
  static __device__ __forceinline__ void run(uint4v (&f)[N], const unsigned (&addr)[N], unsigned kxor) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("ds_read_b128 %0, %1" : "=v"(f[I]) : "v"(addr[I] ^ kxor));
#endif
    Conv3Reads<I + 1, N>::run(f, addr, kxor);
  }
};
template <int N>
struct Conv3Reads<N, N> {
  static __device__ __forceinline__ void run(uint4v (&)[N], const unsigned (&)[N], unsigned) {}
};

// ---------------------------------------------------------------------------
// 3x3 convolution with the input patch resident in LDS and the weights straight in registers.
//
// The per-tap kernel above fetches every input pixel nine times (once per filter tap) through
// the vector cache, whose 64 bytes per clock and compute unit then bound the MFMA rate.  Here a
// workgroup owns TH = 256/W whole image rows (W = image width, a template parameter) and, for
// each slab of 64 bytes of input channels, loads the (TH+2) x (W+2) patch of pixels around its
// rows ONCE — zero padding included, delivered by the buffer range check — and forms all nine
// taps from it: tap (r,s) of pixel (th,tw) is patch cell (th+r, tw+s).
//
// LDS: the patch is double buffered, cells of 64 bytes stored linearly (the global-to-LDS load
// writes lane l at base + 16*l), chunk c of cell q in slot c ^ ((q>>2)&3), so that the 16 cells
// a fragment read touches per pass fall into 16 different 16-byte columns for any tap shift.
//
// Weights never enter LDS (two wavefronts at most share a column, and the LDS port is what
// the patch fragments need): they are packed in fragment order (ConvArgs::w_frag) — the 32
// rows x 32 K-bytes block (nb, kb) is one KiB at (nb * K-bytes/32 + kb) KiB, lane l's MFMA
// operand at byte 16 l of it — and a wave loads the operands of its own WN columns into
// registers two steps ahead (ring of three stages; nine taps, so a tap always uses stage
// tap % 3).  The K loop runs channel slab outer, tap inner (nine steps, fully unrolled); a
// share of the next slab's patch loads is issued at taps 0..6.  The workgroup needs two
// barriers per channel slab: before tap 8, when every wave's share of the next patch has
// landed (tap 8 reads that patch's first fragments), and before tap 0, when every wave has
// read its last fragments of the patch buffer that the loads issued from then on overwrite.
// ---------------------------------------------------------------------------
constexpr int patch_passes(int w) { return (((256 / w + 2) * (w + 2)) * 4 + 255) / 256; }
// patch passes of the next channel slab issued at tap `tap` (spread over taps 0..6)
constexpr int passes_at(int passes, int tap) { return tap < 7 ? passes / 7 + (tap < passes % 7 ? 1 : 0) : 0; }
constexpr int passes_before(int passes, int tap) {
  int n = 0;
  for (int t = 0; t < tap; ++t) n += passes_at(passes, t);
  return n;
}
template <int BN, int WGM, int WGN, int W, bool INTERIOR, int EPI = 0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_conv3_patch(IgemmParams p) {
  static_assert(WGM * WGN == 4, "four wavefronts per workgroup");
  constexpr int ES = 2;
  constexpr int BM = 256, BKB = 64;
  constexpr int TH = BM / W, PW = W + 2, PC = (TH + 2) * PW;
  constexpr int PASSES = patch_passes(W);
  constexpr int PATCH_BYTES = PASSES * 4096;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int MI = WM / 32, NJ = WN / 32;
  constexpr int SW = WN + 16 / ES;
  constexpr int OPER_BYTES = 2 * PATCH_BYTES;
  constexpr int EPI_BYTES = 4 * 32 * SW * ES + WGM * 2 * BN * 4;
  __shared__ __attribute__((aligned(64))) char smem[OPER_BYTES > EPI_BYTES ? OPER_BYTES : EPI_BYTES];
  char* const sP = smem;                        // [2][PATCH_BYTES]
  float (*sRed)[2][BN] = reinterpret_cast<float (*)[2][BN]>(smem + 4 * 32 * SW * ES);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int lb = xcd_logical_block((int)blockIdx.x, (int)gridDim.x);
  const int tile_n = lb % p.tiles_n;
  const int tile_m = lb / p.tiles_n;
  const int64_t m0 = (int64_t)tile_m * BM;
  const int n0 = tile_n * BN;
  const int tiles_per_img = p.Hc / TH;
  const int strip = tile_m % p.strips, row_tile = tile_m / p.strips;   // (strips = 1: the tile spans the image width)
  const int img = row_tile / tiles_per_img;
  const int h0 = (row_tile - img * tiles_per_img) * TH;
  const int w0 = strip * W;
  const int Hin = p.Hc >> p.up, Win = p.Wc >> p.up;
  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rW = make_rsrc(p.w, p.w_bytes);

  // patch loader: slot q = pass*256 + tid of the linear patch buffer
  unsigned a_off[PASSES];
#pragma unroll
  for (int i = 0; i < PASSES; ++i) {
    const int q = i * 256 + tid;
    const int cell = q >> 2;
    const int chunk = (q & 3) ^ ((cell >> 2) & 3);
    const int pr = cell / PW, pc = cell - pr * PW;
    const int hh = h0 - 1 + pr, ww = w0 + pc - 1;
    const bool ok = cell < PC && hh >= 0 && hh < p.Hc && ww >= 0 && ww < p.Wc;
    const unsigned pix = ((unsigned)img * (unsigned)Hin + (unsigned)(hh >> p.up)) * (unsigned)Win + (unsigned)(ww >> p.up);
    a_off[i] = ok ? pix * (unsigned)(p.Cin * ES) + (unsigned)chunk * 16u : kOob;
  }
  // weight operands: one KiB block per 32 columns and K-step, this lane's 16 bytes of it
  const unsigned kb32 = (unsigned)(p.K * ES) >> 5;
  unsigned wv[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) wv[j] = ((((unsigned)(n0 + wn * WN)) >> 5) + (unsigned)j) * kb32 * 1024u + (unsigned)lane * 16u;
  // fragment geometry
  const int frag_row = lane & 31, fc = lane >> 5;
  unsigned cell0[MI];                           // patch cell of this lane's pixel for tap (0,0)
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int ml = wm * WM + i * 32 + frag_row;
    cell0[i] = (unsigned)((ml / W) * PW + (ml % W));
  }
  const unsigned lds_p = (unsigned)(size_t)(lds_char*)sP;

  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int NC = (p.Cin * ES) / BKB;            // channel slabs
  const unsigned tap_bytes = (unsigned)(p.Cin * ES);
#define PATCH_DMA(BUF, PASS, CBYTE) dma_load16(rX, sP + (BUF) * PATCH_BYTES + (PASS) * 4096 + wave * 1024, a_off[PASS] + (CBYTE))
#define WFRAG_LOAD(STG, KBYTE)                                                                               \
  {                                                                                                          \
    const unsigned so = ((KBYTE) >> 5) << 10;                                                                \
    _Pragma("unroll") for (int j = 0; j < NJ; ++j) {                                                         \
      bq[STG][0][j] = __builtin_amdgcn_raw_buffer_load_b128(rW, wv[j], so, 0);                               \
      bq[STG][1][j] = __builtin_amdgcn_raw_buffer_load_b128(rW, wv[j], so + 1024u, 0);                       \
    }                                                                                                        \
  }
  // Patch fragment registers: set 0 holds K-step 0 of the current tap (read during the previous step), set 1
  // K-step 1 (read at the start of the step, behind the MFMAs of K-step 0); while the MFMAs of K-step 1 run,
  // set 0 is refilled for the next tap.  The waits for the weight registers are the compiler's.
  uint4v f0a[MI], f1a[MI];
  uint4v bq[3][2][NJ];
#define CONV3_ADDR(AA, CELLS, TAPV)                                                                          \
  _Pragma("unroll") for (int i = 0; i < MI; ++i) {                                                           \
    const unsigned cell = CELLS[i] + (unsigned)(((TAPV) / 3) * PW + (TAPV) % 3);                             \
    AA[i] = lds_p + (cell << 6) + ((((unsigned)fc) ^ ((cell >> 2) & 3u)) << 4);                              \
  }
  // prologue: the first patch, the weights of steps 0 and 1; fragments of (slab 0, tap 0, K-step 0)
#pragma unroll
  for (int i = 0; i < PASSES; ++i) PATCH_DMA(0, i, 0u);
  WFRAG_LOAD(0, 0u);
  WFRAG_LOAD(1, tap_bytes);
  __builtin_amdgcn_s_waitcnt(vm_imm(0));
  __builtin_amdgcn_s_barrier();
  {
    unsigned aa[MI];
    CONV3_ADDR(aa, cell0, 0)
    Conv3Reads<0, MI>::run(f0a, aa, 0u);
  }

  // One step: tap TAP of channel slab c.  `last` = this is the last channel slab.
#define CONV3_STEP(TAP)                                                                                      \
  {                                                                                                          \
    if ((TAP) == 8 && !last) {                                                                               \
      __builtin_amdgcn_s_waitcnt(vm_imm(2 * NJ));   /* (only the weights tap 7 asked for may be outstanding) */ \
      __builtin_amdgcn_s_barrier();                                                                          \
    }                                                                                                        \
    if ((TAP) == 0 && c > 0) __builtin_amdgcn_s_barrier();                                                   \
    if (!last) {                                                                                             \
      _Pragma("unroll") for (int q = 0; q < passes_at(PASSES, (TAP)); ++q)                                   \
          PATCH_DMA(nbuf, passes_before(PASSES, (TAP)) + q, cbyte + (unsigned)BKB);                          \
    }                                                                                                        \
    if (!last || (TAP) < 7)                                                                                  \
      WFRAG_LOAD(((TAP) + 2) % 3, (unsigned)(((TAP) + 2) % 9) * tap_bytes + cbyte + ((TAP) >= 7 ? (unsigned)BKB : 0u)) \
    {                                                                                                        \
      unsigned aa[MI];                                                                                       \
      CONV3_ADDR(aa, cellb, (TAP))                                                                           \
      Conv3Reads<0, MI>::run(f1a, aa, 32u);                                                                  \
    }                                                                                                        \
    lds_wait_tie_a<MI, MI>(f0a);                                                                             \
    mma_group<bf16_t, MI, NJ>(f0a, bq[(TAP) % 3][0], acc);                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
    lds_wait_tie_a<0, MI>(f1a);                                                                              \
    if (!(last && (TAP) == 8)) {                                                                             \
      unsigned aa[MI];                                                                                       \
      if ((TAP) == 8) { CONV3_ADDR(aa, celln, 0) } else { CONV3_ADDR(aa, cellb, ((TAP) + 1) % 9) }           \
      Conv3Reads<0, MI>::run(f0a, aa, 0u);                                                                   \
    }                                                                                                        \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
    mma_group<bf16_t, MI, NJ>(f1a, bq[(TAP) % 3][1], acc);                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
  }
  // (the last slab is a copy of its own with `last` a constant: where one body served both, the compiler's wait
  // for a weight register had to assume the fewer loads in flight of the last slab, and stalled every other slab's
  // taps 7 and 8 on loads issued a moment before)
#define CONV3_SLAB(LASTV)                                                                                    \
  {                                                                                                          \
    constexpr bool last = LASTV;                                                                             \
    const int nbuf = (c + 1) & 1;                                                                            \
    unsigned cellb[MI], celln[MI];               /* (the buffer offset is a multiple of 4 cells: same swizzle bits) */ \
    _Pragma("unroll") for (int i = 0; i < MI; ++i) {                                                         \
      cellb[i] = cell0[i] + (unsigned)((c & 1) * (PATCH_BYTES / 64));                                        \
      celln[i] = cell0[i] + (unsigned)(nbuf * (PATCH_BYTES / 64));                                           \
    }                                                                                                        \
    const unsigned cbyte = (unsigned)(c * BKB);                                                              \
    CONV3_STEP(0) CONV3_STEP(1) CONV3_STEP(2) CONV3_STEP(3) CONV3_STEP(4)                                    \
    CONV3_STEP(5) CONV3_STEP(6) CONV3_STEP(7) CONV3_STEP(8)                                                  \
  }
  int c = 0;
  for (; c + 1 < NC; ++c) CONV3_SLAB(false)
  CONV3_SLAB(true)
#undef CONV3_SLAB
#undef CONV3_STEP
#undef CONV3_ADDR
#undef WFRAG_LOAD
#undef PATCH_DMA
  __syncthreads();                               // every wave is done with the operands: the epilogue reuses the memory
  igemm_epilogue<bf16_t, BM, BN, WGM, WGN, INTERIOR, EPI>(acc, p, smem, sRed, m0, n0, (int64_t)tile_m);
}

struct IgemmTile { int bm, bn, bkb; };

// Largest tile that still gives every compute unit about two workgroups.
IgemmTile pick_tile(int64_t M, int cout, int cin, int es, bool wide = true, int min_wide_tiles = 256) {
  // large dense bf16 products whose 256 x 256 tiles all lie inside the output and still fill the chip: eight
  // wavefronts per workgroup, a third fewer operand bytes through LDS per multiply-add than 256 x 128
  if (wide && es == 2 && cout % 256 == 0 && M % 256 == 0 && (M / 256) * (cout / 256) >= min_wide_tiles) return IgemmTile{256, 256, 64};
  const int bn = cout > 64 ? 128 : 64;
  const int64_t tiles_n = (cout + bn - 1) / bn;
  int bm = es == 2 ? 256 : 128;                 // 256-row tiles: bf16 only (register budget)
  if (((M + 255) / 256) * tiles_n < 512) bm = 128;
  (void)cin;
  const int bkb = 64;                           // slabs of 64 bytes: with three LDS stages two (256 x 128) or three (128 x 128) workgroups per compute unit
  return IgemmTile{bm, bn, bkb};
}

// LDS stages of k_dense with 128 x 128 tiles.  Three (50 KiB) let a compute unit hold three workgroups, four (67 KiB) two whose
// loads run a slab further ahead.  Three where the compute units share the tiles unevenly (from 352) and where they save a round of
// workgroups (513 to 768); four where there is at most one workgroup per compute unit or little more, beyond 768, where a few
// columns of tiles stream their rows from memory and there is no round to save, and always for triangular K ranges.  us with three /
// four stages / k_igemm (three):
//   256 tiles, 2 048^3: 33.2 / 28.2 / 29.4.             324, 2 304^3: 46.8 / 45.2 / 45.6.  352, 2 048 x 2 816 x 4 096: 65.9 / 67.7 / 70.0
//   512, 4 096 x 2 048 x 4 096: 79.3 / 86.1 / 87.7.     576, 3 072^3: 84.2 / 94.4 / 89.2.  676, 3 328^3: 100.6 / 105.3 / 102.6
//   768, 98 304 x 128 x 256: 23.4 / 26.0 / 23.9.        784, 3 584^3: 153 / 138 / 139
//   512 in one column, K = 4 096: 144 / 135 / 134; in two: 108 / 104 / 109; 510 in three 89.3 / 87.5 / 89.4; 512 in four 79.5 / 85.1 / 86.5
//   LU steps of d = 2 048 and 3 072: 392 and 833 / 381 and 797 / 426 and 854
int dense_stages(int64_t tiles, int tiles_n) {
  return tiles >= 352 && tiles <= 768 && (tiles_n > 3 || tiles > 512) ? 3 : 4;
}

// With the second operand [k][n] and at most one 128 x 128 tile per compute unit: do two groups of four wavefronts take half of K each?
// Twice the loads in flight, at the price of handing 64 KiB of sums over.  us of the product (operands in the caches / from memory), whole
// K / halves, rows x K x columns: 1 024 x 4 096^2 45.8 / 39.9 (62.6 / 57.7), 512 x 4 096^2 42.0 / 33.1, 1 024 x 2 048^2 24.4 / 20.2, 1 024^3
// 14.1 / 12.4, 768^3 11.0 / 10.0, 512^3 8.8 / 8.3, 2 048 x 512^2 9.2 / 8.9, 4 096 x 256^2 6.8 / 7.3.  (With both operands k-contiguous it gains nothing:
// 1 024 x 4 096^2 44.8 / 45.4.)
bool dense_halves(int64_t tiles, int64_t K) { return tiles <= 256 && K % 64 == 0 && K >= 512; }

// Does k_dense take 256 x 128 tiles?  They leave it three stages at two workgroups per compute unit, like k_igemm, and its waits
// let one slab's loads be in flight instead of two: it gains where K is short and the weights stay in the caches, and for
// triangular K ranges (always).  us with k_dense / k_igemm, rows x columns x K:
//   131 072 x 128 x 128 24.7 / 25.7, x 768 52.3 / 54.3, x 1 024 72.5 / 71.3;  65 536 x 384 x 128 34.2 / 34.9, x 256 41.0 / 41.2,
//   x 512 53.5 / 53.3, x 2 048 149 / 144;  32 768 x 640 x 512 48.3 / 46.9, x 1 024 70.8 / 67.6;  32 768 x 1 152 x 64 43.3 / 44.6,
//   x 256 60.8 / 59.1;  16 384 x 1 152 x 4 096 206 / 202.  Both products of a transformation error: 65 536 x 384 107 / 111,
//   32 768 x 640 116 / 114, 32 768 x 896 162 / 170, 16 384 x 1 152 157 / 154, 8 192 x 2 176 249 / 245.  LU step of d = 4 096 1 158 / 1 164.
bool dense_tall(int64_t N, int64_t K, int epi) {
  return epi != CONV_EPI_NONE ? K < 1024 : N * K < (1 << 17);
}

}  // namespace

// The patch kernel takes 3x3 convolutions whose image width is 16..128 (a power of two), whose
// tiles of 256/W rows divide the image height, with enough tiles to fill the chip, and whose
// epilogue needs no run-time checks.
// column width of the patch kernel's tiles
static int conv3_patch_bn(const ConvArgs& a) { return a.cout % 128 == 0 ? 128 : 64; }
static bool conv3_patch_usable(const ConvArgs& a) {
  if (a.geom != CONV_PLAIN || a.k != 3 || a.dtype != AE_BF16 || !conv_mfma_supported(a)) return false;   // (binary32: k_gemm_split)
  // (a 128-pixel-wide tile would need 96 KB of LDS, one workgroup per compute unit: wider images are cut into column
  // strips of 64 pixels instead, whose halo columns come from the neighbouring strip)
  if (a.wc != 16 && a.wc != 32 && a.wc != 64 && a.wc != 128 && a.wc != 256) return false;
  // (measured on the 128 x 128 layers of the largest workload against the per-tap kernel: 93 against 109 us with four
  // channel slabs, 109 against 131 us with two)
  const int th = 256 / (a.wc > 64 ? 64 : a.wc);
  if (a.hc % th != 0 || a.cout % 64 != 0) return false;
  const int bn = conv3_patch_bn(a);
  const int64_t tiles = ((int64_t)a.n * a.hc * a.wc / 256) * (a.cout / bn);
  if (tiles < 256) return false;
  return !a.y_aux && a.act != ACT_SIGMOID && !(a.partial && a.act != ACT_NONE);
}

int conv_partial_rows(const ConvArgs& a, bool mfma) {
  if (!mfma) return kReduceRows;
  if (conv3_patch_usable(a)) return 256;
  return pick_tile((int64_t)a.n * a.hc * a.wc, a.cout, a.cin, (int)dtype_size(a.dtype)).bm;
}

// Split-K: layers with fewer than 128 output tiles (small batch x fully-connected) and a long K.
static int conv_mfma_splits(const ConvArgs& a0) {
  if (a0.partial || a0.epi != CONV_EPI_NONE || a0.geom == CONV_UP_PHASES || !conv_mfma_supported(a0) || conv3_patch_usable(a0)) return 1;
  const ConvArgs a = conv_effective(a0);
  const int es = (int)dtype_size(a.dtype);
  const int64_t M = (int64_t)a.n * a.hc * a.wc;
  const IgemmTile t = pick_tile(M, a.cout, a.cin, es, a0.tri == 0);
  const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((a.cout + t.bn - 1) / t.bn);
  const int64_t KT = (int64_t)a.k * a.k * a.cin * es / t.bkb;
  if (tiles >= 256 || KT < 16) return 1;          // one workgroup per compute unit or more: no split
  int64_t splits = (512 + tiles - 1) / tiles;
  if (splits > KT / 4) splits = KT / 4;
  return splits < 1 ? 1 : (int)splits;
}

int64_t conv_mfma_splitk_floats(const ConvArgs& a0) {
  const int splits = conv_mfma_splits(a0);
  const ConvArgs a = conv_effective(a0);
  return splits > 1 ? (int64_t)splits * a.n * a.hc * a.wc * a.cout : 0;
}

// Four 2x2 phase convolutions: the kernel's epilogue without run-time checks only, and
// enough workgroups without splitting K.
bool conv_up_phases_usable(const ConvArgs& a0) {
  if (a0.up != 1 || a0.k != 3 || (a0.hc & 1) || (a0.wc & 1)) return false;
  ConvArgs a = a0;
  a.geom = CONV_UP_PHASES;
  if (!conv_mfma_supported(a)) return false;
  if (a.partial || a.y_aux || a.act == ACT_SIGMOID) return false;
  const ConvArgs e = conv_effective(a);
  const int64_t M = (int64_t)e.n * e.hc * e.wc;
  const IgemmTile t = pick_tile(M, e.cout, e.cin, (int)dtype_size(e.dtype));
  if (M % t.bm != 0 || e.cout % t.bn != 0) return false;
  return (M / t.bm) * (e.cout / t.bn) * 4 >= 256;
}

// The special epilogues: 1x1 layers, check-free tiles of the shapes they are instantiated for, no split-K.
bool conv_epi_usable(const ConvArgs& a) {
  if (a.epi == CONV_EPI_NONE) return true;
  if (a.geom != CONV_PLAIN || a.k != 1 || a.up != 0 || a.hc != 1 || a.wc != 1 || !conv_mfma_supported(a)) return false;
  if (a.y_aux || a.act != ACT_NONE || a.cout % 128 != 0) return false;
  if (a.epi == CONV_EPI_RESID && (!a.partial || !a.resid)) return false;
  if (a.epi == CONV_EPI_MXQ && a.partial) return false;
  if (a.epi == CONV_EPI_MXQ) {
    const int epc = 16 / (int)dtype_size(a.dtype);
    if (a.mx_block < epc || a.mx_block > 64 || (a.mx_block & (a.mx_block - 1)) != 0) return false;
    if (a.mx_elem != MX_FP4 && a.mx_elem != MX_INT4 && a.mx_elem != MX_FP8) return false;
  }
  const IgemmTile t = pick_tile(a.n, a.cout, a.cin, (int)dtype_size(a.dtype));
  return (t.bn == 128 || t.bn == 256) && a.n % t.bm == 0;
}

bool conv_up_dgrad_usable(const ConvArgs& a0) {
  if (a0.k != 3 || a0.up != 0 || (a0.hc & 1) || (a0.wc & 1) || a0.partial || a0.y_aux || a0.bias || a0.act != ACT_NONE) return false;
  ConvArgs a = a0;
  a.geom = CONV_UP_DGRAD;
  return conv_mfma_supported(a);
}

// Number of row blocks whose column sums a launch with a companion tensor (ConvArgs::comp) leaves in `partial`, or 0
// if this launch cannot take one: the epilogue exists for bfloat16 launches whose tiles all lie inside the output,
// without split-K and without an epilogue variant of their own.
int conv_comp_blocks(const ConvArgs& a0) {
  if (a0.dtype != AE_BF16 || !conv_mfma_supported(a0) || a0.epi != CONV_EPI_NONE || a0.tri != 0 || a0.geom == CONV_UP_PHASES ||
      a0.y_aux || a0.act != ACT_NONE || a0.bias)
    return 0;
  const ConvArgs a = conv_effective(a0);
  const int64_t M = (int64_t)a.n * a.hc * a.wc;
  if (conv3_patch_usable(a0)) return (int)(M / 256);
  const IgemmTile t = pick_tile(M, a.cout, a.cin, 2, a0.geom == CONV_PLAIN, 256);
  if (t.bn == 256 || M % t.bm != 0 || a.cout % t.bn != 0) return 0;
  ConvArgs probe = a0;
  probe.partial = reinterpret_cast<float*>(1);     // only null / non-null matters: statistics keep K in one piece
  if (conv_mfma_splits(probe) != 1) return 0;
  return (int)(M / t.bm);
}

bool conv_weights_frag_order(const ConvArgs& a) { return conv3_patch_usable(a); }

// source and destination geometry of a launch; row_bytes: one stored pixel of x
static void igemm_geometry(const ConvArgs& a0, const ConvArgs& a, int row_bytes, IgemmParams* p) {
  p->Hc = a.hc; p->Wc = a.wc; p->ksz = a.k; p->up = a.up; p->act = a.act;
  p->Hv = a.hc; p->Wv = a.wc; p->stride = 1; p->pad = (a.k - 1) >> 1; p->phases = 1;
  if ((a.hc & (a.hc - 1)) == 0 && (a.wc & (a.wc - 1)) == 0) {
    p->log_w = p->log_h = 0;
    while ((1 << p->log_w) < a.wc) ++p->log_w;
    while ((1 << p->log_h) < a.hc) ++p->log_h;
  }
  p->x_bytes = (unsigned)((int64_t)a.n * (a.hc >> a.up) * (a.wc >> a.up) * row_bytes);
  p->w_bytes = (unsigned)((int64_t)a.cout * a.k * a.k * row_bytes);
  if (a0.geom == CONV_UP_PHASES) {
    p->pad = 1; p->phases = 4;
    p->w_bytes *= 4u;
  } else if (a0.geom == CONV_UP_DGRAD) {
    p->Hv = a0.hc; p->Wv = a0.wc; p->stride = 2; p->pad = 1;
    p->x_bytes = (unsigned)((int64_t)a0.n * a0.hc * a0.wc * row_bytes);
  }
}

// sum of a split launch's partial tiles, bias, rounding and activation
static int launch_splitk_finish(const ConvArgs& a, int splits, int64_t M, int N, hipStream_t s) {
  int64_t g = (M * N + 255) / 256;
  if (g > 8192) g = 8192;
  if (a.dtype == AE_BF16)
    hipLaunchKernelGGL((k_splitk_finish<bf16_t>), dim3((unsigned)g), dim3(256), 0, s, a.splitk_ws, splits, M, N, a.bias,
                       a.act, (bf16_t*)a.y, a.y_aux);
  else
    hipLaunchKernelGGL((k_splitk_finish<float>), dim3((unsigned)g), dim3(256), 0, s, a.splitk_ws, splits, M, N, a.bias,
                       a.act, (float*)a.y, a.y_aux);
  return launch_status("splitk_finish");
}

// Checked bf16 tiles whose rows are stored from the accumulators (DIRECT): rows of no whole 16 bytes, most of a tile's columns
// inside, 32-bit offsets.  (Phases, whose output rows take divisions, the sigmoid and its binary32 copy use the loop: 48 -> 3 channels behind
// an upsample 27 -> 16 us with it.)
static bool direct_stores(const IgemmParams& p, int dtype, int bn) {
  return dtype == AE_BF16 && !p.split_out && p.N % 8 != 0 && p.N < (1 << 20) && 2 * p.N > bn && !p.y_aux && p.act != ACT_SIGMOID && p.phases == 1;
}

int launch_conv_mfma(const ConvArgs& a0, hipStream_t s) {
  if (!conv_mfma_supported(a0)) return fail(AE_EINVAL, "conv_mfma: shape not supported");
  if (a0.w_frag != conv3_patch_usable(a0)) return fail(AE_EINVAL, "conv_mfma: the order of the packed weights does not fit the kernel of this launch (conv_weights_frag_order)");
  if (a0.geom == CONV_UP_PHASES && !conv_up_phases_usable(a0)) return fail(AE_EINVAL, "conv_mfma: phase form not usable here");
  if (!conv_epi_usable(a0)) return fail(AE_EINVAL, "conv_mfma: epilogue variant not usable for this shape");
  const ConvArgs a = conv_effective(a0);
  const int es = (int)dtype_size(a.dtype);
  IgemmParams p;
  p.x = a.x; p.w = a.w; p.bias = a.bias; p.y = a.y; p.y_aux = a.y_aux; p.partial = a.partial;
  p.M = (int64_t)a.n * a.hc * a.wc;
  p.N = a.cout; p.K = a.k * a.k * a.cin;
  p.Cin = a.cin;
  igemm_geometry(a0, a, a.cin * es, &p);
  p.resid = a0.resid;
  p.comp = a0.comp; p.comp_mode = a0.comp_mode; p.comp_bn = a0.comp_bn;
  if (a0.comp_mode != 0) {
    if (a0.comp_mode < 1 || a0.comp_mode > 2 || !a0.comp || !a0.partial || (a0.comp_mode == 2 && !a0.comp_bn) ||
        conv_comp_blocks(a0) == 0)
      return fail(AE_EINVAL, "conv_mfma: companion-tensor epilogue not usable for this launch");
  }
  p.mx_block = a0.mx_block;
  p.mx_elem = a0.mx_elem;
  p.tri = a0.tri;
  if (a0.tri != 0 && (a0.tri < 0 || a0.tri > CONV_TRI_UPPER_W_FULL || a.k != 1 || a.hc != 1 || a.wc != 1 || a.up != 0 || a.n != a.cout || a.cin != a.cout ||
                      a0.epi != CONV_EPI_NONE || a.partial))
    return fail(AE_EINVAL, "conv_mfma: triangular K ranges are for square dense products only");
  if (conv3_patch_usable(a0)) {
    const int bn = conv3_patch_bn(a);
    p.tiles_n = a.cout / bn;
    p.strips = a.wc > 64 ? a.wc / 64 : 1;
    p.log_wt = 6;                                // strips of 64 pixels
    dim3 pgrid((unsigned)((p.M / 256) * p.tiles_n));
#define PATCH_LAUNCH_E(WV, E)                                                                                \
  do {                                                                                                      \
    if (bn == 128) hipLaunchKernelGGL((k_conv3_patch<128, 2, 2, WV, true, E>), pgrid, dim3(256), 0, s, p);    \
    else hipLaunchKernelGGL((k_conv3_patch<64, 4, 1, WV, true, E>), pgrid, dim3(256), 0, s, p);              \
  } while (0)
    if (a0.comp_mode != 0) {            // (conv_comp_blocks: bfloat16 only)
      if (a0.comp_mode == 1) { if (a.wc == 16) PATCH_LAUNCH_E(16, 3); else if (a.wc == 32) PATCH_LAUNCH_E(32, 3); else PATCH_LAUNCH_E(64, 3); }
      else { if (a.wc == 16) PATCH_LAUNCH_E(16, 4); else if (a.wc == 32) PATCH_LAUNCH_E(32, 4); else PATCH_LAUNCH_E(64, 4); }
      return launch_status("conv3_patch");
    }
    if (a.wc == 16) PATCH_LAUNCH_E(16, 0);
    else if (a.wc == 32) PATCH_LAUNCH_E(32, 0);
    else PATCH_LAUNCH_E(64, 0);
#undef PATCH_LAUNCH_E
    return launch_status("conv3_patch");
  }
  // the wide tile exists without run-time checks only; tiles of very different K lengths (the triangular modes 1-3)
  // balance better when smaller unless there are at least four per compute unit (measured: d = 8192, not 4096)
  const bool wide_ok = a0.tri <= CONV_TRI_UPPER_W && !a.y_aux && a.act != ACT_SIGMOID && !(a.partial && a.act != ACT_NONE) && a0.geom == CONV_PLAIN;
  const IgemmTile t = pick_tile(p.M, a.cout, a.cin, es, wide_ok, a0.tri == 0 ? 256 : 1024);
  p.tiles_n = (a.cout + t.bn - 1) / t.bn;
  const int64_t tiles_m = (p.M + t.bm - 1) / t.bm;
  const int KT = (int)((int64_t)p.K * es / t.bkb);
  int splits = conv_mfma_splits(a0);
  if (splits > 1 && (!a.splitk_ws || (int64_t)splits * p.M * p.N > a.splitk_floats)) splits = 1;
  if (a0.tri != 0) splits = 1;
  p.tiles_mn = (int)(tiles_m * p.tiles_n);
  p.slabs_per_split = (KT + splits - 1) / splits;
  splits = (KT + p.slabs_per_split - 1) / p.slabs_per_split;
  p.split_out = splits > 1 ? a.splitk_ws : nullptr;
  dim3 grid((unsigned)(tiles_m * p.tiles_n * splits * p.phases));
  const bool interior = splits == 1 && p.M % t.bm == 0 && p.N % t.bn == 0 && !a.y_aux && a.act != ACT_SIGMOID &&
                        !(a.partial && a.act != ACT_NONE);
#define IGEMM_LAUNCH_K(T, BMV, BNV, GM, GN, KB)                                                        \
  do {                                                                                                 \
    if (interior) hipLaunchKernelGGL((k_igemm<T, BMV, BNV, GM, GN, KB, true, true>), grid, dim3(256), 0, s, p); \
    else if (sizeof(T) == 2 && direct) hipLaunchKernelGGL((k_igemm<T, BMV, BNV, GM, GN, KB, false, true, 0, false, sizeof(T) == 2>), grid, dim3(256), 0, s, p); \
    else hipLaunchKernelGGL((k_igemm<T, BMV, BNV, GM, GN, KB, false, true>), grid, dim3(256), 0, s, p); \
  } while (0)
  const bool direct = direct_stores(p, a.dtype, t.bn);
  const bool tri = a0.tri != 0;
  // Binary32: three bf16 parts (k_gemm_split), unless the caller asks for the binary32 MFMA or there are few columns and a
  // short K, where both only move the operands (65,536 rows, 64 -> 64 channels: 13.6 and 12.8 us; 131,072 rows, 48 -> 64 -> 48: 18.7
  // and 18.6, 22.4 and 22.9; from there on the parts win: 64 -> 512 -> 64 channels 60.5 against 45.6 and 45.0 against 37.4)
  const bool split_gemm = a.dtype == AE_F32 && !a0.f32_mfma && !(p.N <= 64 && p.K < 128);
  const bool dense = a.k == 1 && a.up == 0 && p.phases == 1 && p.stride == 1;
  if (split_gemm) {
    // Dense products whose tiles all lie inside the output: 128 x 128 tiles (two workgroups per compute unit), halves of them
    // where those would leave compute units idle, or 256 x 128 (one workgroup, the cheapest per output) where K is long
    // enough to outweigh their prologue and epilogue, which nothing runs beside.  The costs are rounds of workgroups, in
    // units of a full round of 512 of the first kind: 256 of them 0.63, 512 halves 0.69, 256 halves 0.45, 256 tall ones 0.89.
    // Measured (QR step, 30 products): d = 512, 768, 1024 0.71, 0.97, 1.21 ms with halves, 0.94, 1.29, 1.63 without; d = 1536 the same;
    // d = 2048 3.66 with, 3.34 without; d = 4096 19.9 ms with tall tiles, 22.7 without.  Tall ones from K = 512 on: forward pass of
    // one layer of K = 512 / 640 / 768 / 896, 128 to 1 024 columns, 2 048 to 65 536 rows: 1 to 14 % faster where the costs choose them (65 536 x 512 x 512 274 -> 267 us,
    // 20 480 x 256 x 640 65 -> 57, 8 192 x 1 024 x 896 129 -> 121), nowhere slower.  Triangular K ranges gain from halves
    // up to 256 tiles (d = 2048, LU step: 0.56 against 0.71 ms).
    auto rounds = [](int64_t n, int64_t slots, double half, double full) {
      const int64_t rem = n % slots;
      return (double)(n / slots) * full + (rem == 0 ? 0.0 : rem <= slots / 2 ? half : full);
    };
    const int64_t n128 = grid.x;
    const bool choice = dense && interior && t.bn == 128 && a0.epi == CONV_EPI_NONE;
    const double c128 = rounds(n128, 512, 0.63, 1.0), c64 = rounds(2 * n128, 512, 0.45, 0.69);
    // (not with column sums: the caller counts one block of them per 128 rows)
    const bool whole = a0.tri == CONV_TRI_NONE || a0.tri == CONV_TRI_LOWER_W_FULL || a0.tri == CONV_TRI_UPPER_W_FULL;      // every output, K ranges that make rounds of equal sums: as without them
    const double tall = whole && !p.partial && p.M % 256 == 0 && p.K >= 512 ? rounds(n128 / 2, 256, 0.89, 0.89) : 1e30;
    if (choice && tall < c128 && tall < c64) {
      p.tiles_mn /= 2;
      if (tri) hipLaunchKernelGGL((k_gemm_split<256, 128, 4, 2, true, 0, false, TRI_RANGE>), dim3(grid.x / 2), dim3(512), 0, s, p);
      else hipLaunchKernelGGL((k_gemm_split<256, 128, 4, 2, true>), dim3(grid.x / 2), dim3(512), 0, s, p);
    } else if (choice && (!whole ? n128 <= 256 : c64 < c128)) {
      p.tiles_n *= 2;
      p.tiles_mn *= 2;
      if (tri) hipLaunchKernelGGL((k_gemm_split<128, 64, 4, 1, true, 0, false, TRI_RANGE>), dim3(grid.x * 2), dim3(256), 0, s, p);
      else hipLaunchKernelGGL((k_gemm_split<128, 64, 4, 1, true>), dim3(grid.x * 2), dim3(256), 0, s, p);
    } else if (a0.epi == CONV_EPI_MXQ) hipLaunchKernelGGL((k_gemm_split<128, 128, 2, 2, true, 1>), grid, dim3(256), 0, s, p);   // (conv_epi_usable: interior)
    else if (a0.epi == CONV_EPI_RESID) hipLaunchKernelGGL((k_gemm_split<128, 128, 2, 2, true, 2>), grid, dim3(256), 0, s, p);
    else if (tri && interior) hipLaunchKernelGGL((k_gemm_split<128, 128, 2, 2, true, 0, false, TRI_RANGE>), grid, dim3(256), 0, s, p);
    else if (tri) hipLaunchKernelGGL((k_gemm_split<128, 128, 2, 2, false, 0, false, TRI_RANGE>), grid, dim3(256), 0, s, p);   // (64 columns: not by parts)
#define SPLIT_LAUNCH(BNV, GM, GN, IN, CV) hipLaunchKernelGGL((k_gemm_split<128, BNV, GM, GN, IN, 0, CV>), grid, dim3(256), 0, s, p)
#define SPLIT_LAUNCH_T(BNV, GM, GN)                                                                                    \
  do {                                                                                                                 \
    if (dense) { if (interior) SPLIT_LAUNCH(BNV, GM, GN, true, false); else SPLIT_LAUNCH(BNV, GM, GN, false, false); } \
    else { if (interior) SPLIT_LAUNCH(BNV, GM, GN, true, true); else SPLIT_LAUNCH(BNV, GM, GN, false, true); }         \
  } while (0)
    else if (t.bn == 128) SPLIT_LAUNCH_T(128, 2, 2);
    else SPLIT_LAUNCH_T(64, 4, 1);
#undef SPLIT_LAUNCH_T
#undef SPLIT_LAUNCH
    AE_TRY(launch_status("gemm_split"));
    return splits > 1 ? launch_splitk_finish(a, splits, p.M, p.N, s) : AE_OK;
  }
#define IGEMM_LAUNCH_T(T, BMV, BNV, GM, GN) IGEMM_LAUNCH_K(T, BMV, BNV, GM, GN, 64)   /* pick_tile: 64-byte slabs only */
#define IGEMM_LAUNCH(BMV, BNV, GM, GN)                                         \
  do {                                                                         \
    if (a.dtype == AE_BF16) IGEMM_LAUNCH_T(bf16_t, BMV, BNV, GM, GN);          \
    else IGEMM_LAUNCH_T(float, BMV, BNV, GM, GN);                              \
  } while (0)
  const bool dense_bf16 = a.dtype == AE_BF16 && dense && interior;
  const int stages = dense_stages(grid.x, p.tiles_n);
  const bool tall = dense_tall(p.N, p.K, a0.epi);
  if (a0.comp_mode != 0) {
    // (conv_comp_blocks: bfloat16, interior tiles, no split, not the eight-wavefront tile)
#define IGEMM_LAUNCH_COMP(BMV, BNV, GM, GN)                                                                           \
  do {                                                                                                                \
    if (a0.comp_mode == 1) hipLaunchKernelGGL((k_igemm<bf16_t, BMV, BNV, GM, GN, 64, true, true, 3>), grid, dim3(256), 0, s, p); \
    else hipLaunchKernelGGL((k_igemm<bf16_t, BMV, BNV, GM, GN, 64, true, true, 4>), grid, dim3(256), 0, s, p);         \
  } while (0)
    if (t.bm == 256 && t.bn == 128) IGEMM_LAUNCH_COMP(256, 128, 2, 2);
    else if (t.bm == 256) IGEMM_LAUNCH_COMP(256, 64, 4, 1);
    else if (t.bn == 128) IGEMM_LAUNCH_COMP(128, 128, 2, 2);
    else IGEMM_LAUNCH_COMP(128, 64, 2, 2);
#undef IGEMM_LAUNCH_COMP
    return launch_status("conv_mfma_comp");
  }
  if (a0.epi != CONV_EPI_NONE) {
    // (conv_epi_usable: interior tiles, BN = 128, no split; binary32 went to k_gemm_split above: a dense product of 128 columns or more)
    if (a.dtype != AE_BF16) return fail(AE_EINVAL, "conv_mfma: no such epilogue on the binary32 MFMA");
#define EPI_LAUNCH(E)                                                                                                        \
  do {                                                                                                                       \
    if (t.bn == 256) hipLaunchKernelGGL((k_dense<256, 256, 2, 4, 4, E>), grid, dim3(512), 0, s, p);                            \
    else if (t.bm == 256 && tall) hipLaunchKernelGGL((k_dense<256, 128, 2, 2, 3, E>), grid, dim3(256), 0, s, p);                \
    else if (t.bm == 256) hipLaunchKernelGGL((k_igemm<bf16_t, 256, 128, 2, 2, 64, true, true, E>), grid, dim3(256), 0, s, p);   \
    else if (stages == 3) hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 3, E>), grid, dim3(256), 0, s, p);                        \
    else hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 4, E>), grid, dim3(256), 0, s, p);                                         \
  } while (0)
    if (a0.epi == CONV_EPI_MXQ) EPI_LAUNCH(1);
    else EPI_LAUNCH(2);
#undef EPI_LAUNCH
    return launch_status("conv_mfma_epi");
  }
  if (tri) {
    // square products: 64-column tiles (d = 32, 64) are never check-free, nor are those of bf16 here (k_dense takes them)
#define TRI_LAUNCH(T, BMV, BNV, IN) hipLaunchKernelGGL((k_igemm<T, BMV, BNV, 2, 2, 64, IN, true, 0, false, false, true>), grid, dim3(256), 0, s, p)
    if (dense_bf16 && t.bn == 256) hipLaunchKernelGGL((k_dense<256, 256, 2, 4, 4, 0, true>), grid, dim3(512), 0, s, p);
    else if (dense_bf16 && t.bm == 256) hipLaunchKernelGGL((k_dense<256, 128, 2, 2, 3, 0, true>), grid, dim3(256), 0, s, p);
    else if (dense_bf16) hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 4, 0, true>), grid, dim3(256), 0, s, p);
    else if (a.dtype == AE_BF16 && t.bm == 256) TRI_LAUNCH(bf16_t, 256, 128, false);
    else if (a.dtype == AE_BF16 && t.bn == 128) TRI_LAUNCH(bf16_t, 128, 128, false);
    else if (a.dtype == AE_BF16) TRI_LAUNCH(bf16_t, 128, 64, false);
    else if (t.bn == 64) TRI_LAUNCH(float, 128, 64, false);
    else if (interior) TRI_LAUNCH(float, 128, 128, true);
    else TRI_LAUNCH(float, 128, 128, false);
#undef TRI_LAUNCH
    return launch_status("conv_mfma_tri");
  }
  if (dense_bf16 && t.bn == 256) hipLaunchKernelGGL((k_dense<256, 256, 2, 4, 4>), grid, dim3(512), 0, s, p);
  else if (dense_bf16 && t.bm == 256 && t.bn == 128 && tall) hipLaunchKernelGGL((k_dense<256, 128, 2, 2, 3>), grid, dim3(256), 0, s, p);
  else if (dense_bf16 && t.bm == 128 && t.bn == 128 && stages == 3) hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 3>), grid, dim3(256), 0, s, p);
  else if (dense_bf16 && t.bm == 128 && t.bn == 128) hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 4>), grid, dim3(256), 0, s, p);
  else if (t.bn == 256) hipLaunchKernelGGL((k_igemm<bf16_t, 256, 256, 2, 4, 64, true, true>), grid, dim3(512), 0, s, p);   // (pick_tile: interior only)
  else if (t.bm == 256 && t.bn == 128) IGEMM_LAUNCH_K(bf16_t, 256, 128, 2, 2, 64);
  else if (t.bm == 256) IGEMM_LAUNCH_K(bf16_t, 256, 64, 4, 1, 64);
  else if (t.bn == 128) IGEMM_LAUNCH(128, 128, 2, 2);
  else IGEMM_LAUNCH(128, 64, 2, 2);
#undef IGEMM_LAUNCH_K
#undef IGEMM_LAUNCH
#undef IGEMM_LAUNCH_T
  AE_TRY(launch_status("conv_mfma"));
  return splits > 1 ? launch_splitk_finish(a, splits, p.M, p.N, s) : AE_OK;
}

// y[m][n] = sum over k of x[m mod group][k] w[K (m div group) + k][n], bf16, check-free tiles: products whose second operand lies
// [k][n] (KN of k_dense), in groups of `group` output rows with the same x (one group: group = rows)
bool dense_kn_supported(int64_t rows, int64_t k, int64_t n, int64_t group) {
  return rows % group == 0 && group % 128 == 0 && n % 128 == 0 && k % 32 == 0 && k > 0 && (rows / 128) * (n / 128) < 0x7FFFFFFF &&
         group * k * 2 < 0x7FFFFFFF && k * n * 2 < 0x7FFFFFFF;
}
int launch_dense_kn(const void* x, const void* w, void* y, int64_t rows, int64_t k, int64_t n, int64_t group, hipStream_t s, int tri) {
  if (!dense_kn_supported(rows, k, n, group)) return fail(AE_EINVAL, "dense_kn: shape not supported");
  if (tri != 0 && (rows != n || k != n || group != rows || (tri != CONV_TRI_LOWER_UPPER && tri != CONV_TRI_UPPER_X))) return fail(AE_EINVAL, "dense_kn: bad triangular product");
  IgemmParams p = {};
  p.x = x; p.w = w; p.y = y;
  p.M = rows; p.N = (int)n; p.K = (int)k; p.phases = 1; p.act = ACT_NONE; p.kn_group = (int)group; p.tri = tri;
  // (tiles of very different K ranges: as in launch_conv_mfma)
  const bool wide = rows % 256 == 0 && group % 256 == 0 && n % 256 == 0 && (rows / 256) * (n / 256) >= (tri != 0 ? 1024 : 256);
  const bool tall = tri != 0 && !wide && rows % 256 == 0 && (rows / 256) * (n / 128) >= 512;
  p.tiles_n = (int)(n / (wide ? 256 : 128));
  p.tiles_mn = (int)((rows / (wide || tall ? 256 : 128)) * p.tiles_n);
  const dim3 grid((unsigned)p.tiles_mn);
  if (tri != 0) {
    if (wide) hipLaunchKernelGGL((k_dense<256, 256, 2, 4, 4, 0, true, true>), grid, dim3(512), 0, s, p);
    else if (tall) hipLaunchKernelGGL((k_dense<256, 128, 2, 2, 3, 0, true, true>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 4, 0, true, true>), grid, dim3(256), 0, s, p);
  } else if (wide) hipLaunchKernelGGL((k_dense<256, 256, 2, 4, 4, 0, false, true>), grid, dim3(512), 0, s, p);
  else if (dense_halves(grid.x, p.K)) hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 4, 0, false, true, 2>), grid, dim3(512), 0, s, p);
  else if (dense_stages(grid.x, p.tiles_n) == 3) hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 3, 0, false, true>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((k_dense<128, 128, 2, 2, 4, 0, false, true>), grid, dim3(256), 0, s, p);
  return launch_status("dense_kn");
}

// ---- the triangular inverse's products -----------------------------------------------------------------------------------
int launch_tri_pairs(const TriProduct* f, int count, int dp, int b, int d, bool negate, hipStream_t s) {
  if (count < 1 || count > 2 || b < 128 || b % 128 != 0 || dp % (2 * b) != 0 || d < 1 || d > dp || d % 128 != 0 || (int64_t)dp * dp * 4 >= 0x7FFFFFFF)
    return fail(AE_EINVAL, "tri_pairs: bad sizes");
  IgemmParams p = {};
  p.M = dp; p.N = p.K = dp; p.phases = 1; p.act = ACT_NONE;
  p.ldx = dp; p.ldw = f[0].ldw; p.tri_b = b; p.tri_d = d; p.tri_pairs = (d + 2 * b - 1) / (2 * b);   // pairs wholly inside the identity padding stay as they are
  p.negate = negate;
  p.x_bytes = (unsigned)((int64_t)dp * dp * 4);
  p.w_bytes = (unsigned)((int64_t)p.ldw * p.ldw * 4);
  for (int i = 0; i < count; ++i) p.tm[i] = IgemmParams::Tri{f[i].x, f[i].w, f[i].y, f[i].yt, f[i].lower};
  // Tiles: launches that wait for one another; the longest K range of a tile is a chain of slabs, and a slab of a smaller tile is shorter, so quarters
  // of 64 x 64 while those that lie inside are at most 256 of 128 x 128 (of the last pair, only columns or rows up to d do).  us of a binary32 inverse with
  // quarters up to 64, 128 and 256: d = 2 048 222, 206, 206; 2 176 395, 387, 375; 3 072 532, 524, 514; with halves between 256 and 512, d = 4 096 718, without 708.
  const int64_t t = b / 128, tiles = count * p.tri_pairs * t * t, inside = count * ((p.tri_pairs - 1) * t * t + t * std::max(0, std::min((int)t, (d - (2 * p.tri_pairs - 1) * b) / 128)));
  if (inside <= 256) hipLaunchKernelGGL((k_gemm_split<64, 64, 2, 2, true, 0, false, TRI_PAIRS>), dim3((unsigned)tiles * 4), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((k_gemm_split<128, 128, 2, 2, true, 0, false, TRI_PAIRS>), dim3((unsigned)tiles), dim3(256), 0, s, p);
  return launch_status("tri_pairs");
}
// side of the square of outputs that share a K range, which starts at its first row: x and w hold zeros in the other triangle of
// the diagonal blocks of that size: 256 (tiles of 256 x 128) where they fill the chip for long enough.  us of a binary32 inverse with 128 / 256: d = 1 024
// 103 / 115, 2 304 383 / 396, 2 816 517 / 509, 3 072 578 / 576, 3 328 575 / 579, 3 840 668 / 661, 4 096 731 / 722, 4 352 1 350 / 1 361, 5 120 2 395 / 2 375, 6 144 3 034 / 2 998,
// 8 192 4 365 / 4 261: even between 2 560 and 4 352, the larger squares win beyond
static int tri_last_side(int d) { return d % 256 == 0 && d >= 4096 ? 256 : 128; }
int tri_last_split(int d) { return d / tri_last_side(d) / 2 * tri_last_side(d); }
int launch_tri_last(const float* x, const float* w, int ld, float* y, float* y2, int d, hipStream_t s) {
  if (d < 128 || d % 128 != 0 || ld < d || (int64_t)ld * ld * 4 >= 0x7FFFFFFF) return fail(AE_EINVAL, "tri_last: bad sizes");
  IgemmParams p = {};
  p.M = d; p.N = p.K = d; p.phases = 1; p.act = ACT_NONE;
  p.ldx = p.ldw = ld;
  p.x_bytes = p.w_bytes = (unsigned)((int64_t)ld * ld * 4);
  p.tm[0] = IgemmParams::Tri{x, w, y, nullptr, false};
  p.tm[1] = IgemmParams::Tri{x, w, y2, nullptr, false};
  const int side = tri_last_side(d), t = d / side, half = t / 2;
  const unsigned n = (unsigned)(t * t + half * half);
  if (side == 256) hipLaunchKernelGGL((k_gemm_split<256, 128, 4, 2, true, 0, false, TRI_LAST>), dim3(n * 2), dim3(512), 0, s, p);
  else if (t * t <= 256) hipLaunchKernelGGL((k_gemm_split<128, 64, 4, 1, true, 0, false, TRI_LAST>), dim3(n * 2), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((k_gemm_split<128, 128, 2, 2, true, 0, false, TRI_LAST>), dim3(n), dim3(256), 0, s, p);
  return launch_status("tri_last");
}

// ---- any channel counts: the chunk walk of k_igemm ---------------------------------------------------------------
// a.x holds whole 16-byte chunks per pixel and a.w per tap (chan_pad channels, zeros behind the layer's own)
int launch_conv_chunks(const ConvArgs& a0, hipStream_t s) {
  if (!conv_chunks_supported(a0) || a0.w_frag) return fail(AE_EINVAL, "conv_chunks: shape not supported");
  const ConvChunksPlan c = plan_conv_chunks(a0);
  const ConvArgs a = conv_effective(a0);
  IgemmParams p = {};
  p.x = a.x; p.w = a.w; p.bias = a.bias; p.y = a.y; p.y_aux = a.y_aux; p.partial = a.partial;
  p.M = c.M; p.N = a.cout; p.K = a.k * a.k * chan_pad(a.cin, a.dtype); p.Cin = chan_pad(a.cin, a.dtype); p.chunks = c.chunks;
  igemm_geometry(a0, a, 16 * c.chunks, &p);
  p.tiles_n = (a.cout + c.bn - 1) / c.bn;
  int splits = c.splits;
  if (splits > 1 && (!a.splitk_ws || (int64_t)splits * c.M * p.N > a.splitk_floats)) splits = 1;
  p.tiles_mn = (int)c.tiles;
  p.slabs_per_split = (c.KT + splits - 1) / splits;
  splits = (c.KT + p.slabs_per_split - 1) / p.slabs_per_split;
  p.split_out = splits > 1 ? a.splitk_ws : nullptr;
  const dim3 grid((unsigned)(c.tiles * splits * p.phases));
  const bool direct = direct_stores(p, a.dtype, c.bn);
#define CHUNKS_LAUNCH(T, BMV, BNV, GM, GN)                                                                                           \
  do {                                                                                                                               \
    if (direct) hipLaunchKernelGGL((k_igemm<T, BMV, BNV, GM, GN, 64, false, true, 0, true, sizeof(T) == 2>), grid, dim3(256), 0, s, p); \
    else hipLaunchKernelGGL((k_igemm<T, BMV, BNV, GM, GN, 64, false, true, 0, true>), grid, dim3(256), 0, s, p);                        \
  } while (0)
#define CHUNKS_TILE(T)                                                              \
  do {                                                                              \
    if (c.bn == 128) CHUNKS_LAUNCH(T, 128, 128, 2, 2);                            \
    else if (c.bn == 64) CHUNKS_LAUNCH(T, 128, 64, 2, 2);                         \
    else if (c.bm == 256) CHUNKS_LAUNCH(T, 256, 32, 4, 1);                        \
    else CHUNKS_LAUNCH(T, 128, 32, 4, 1);                                           \
  } while (0)
  if (a.dtype == AE_F32) CHUNKS_TILE(float);
  else if (c.bn == 128 && c.bm == 64) CHUNKS_LAUNCH(bf16_t, 64, 128, 2, 2);
  else if (c.bn == 64 && c.bm == 256) CHUNKS_LAUNCH(bf16_t, 256, 64, 4, 1);
  else CHUNKS_TILE(bf16_t);
#undef CHUNKS_TILE
#undef CHUNKS_LAUNCH
  AE_TRY(launch_status("conv_chunks"));
  return splits > 1 ? launch_splitk_finish(a, splits, p.M, p.N, s) : AE_OK;
}

}  // namespace ae

// ===========================================================================
// Weight gradient on the matrix cores (bf16).
//
//   dW[co][(r,s,ci)] = sum over pixels m of dY[m][co] * Xg[m][(r,s,ci)]
// where Xg is the gathered input of tap (r,s).  Both operands are stored with the
// reduction index (the pixel) outermost, so the MFMA operands (8 consecutive pixels
// of one channel per lane) are transposes of what memory holds.  The slabs go to
// LDS exactly as loaded, [pixel][channel], and are read back with the gfx950 LDS
// transpose load (ds_read_b64_tr_b16): within a group of 16 lanes, the lane with
// local index 4*j+q supplies the address of 4 channels (4q..4q+3) of pixel j, and
// lane i receives channel i of pixels 0..3.
//
// A workgroup owns one output tile (BM output channels x BN input channels of one
// tap) and one contiguous range of pixels; partial tiles go to a workspace
// [split][C_out][k*k*C_in] (fp32) that a second kernel sums in a fixed order and
// writes in the canonical [C_out][C_in][k][k] layout, so the result is deterministic.
// ===========================================================================
namespace ae {
namespace {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v lds_short4v;

// quotient by a divisor fixed at launch, for dividends below 2^31: l = ceil(log2 d), mul = ceil(2^(31+l) / d); the error
// of mul, below one part in 2^31 of a quotient step, cannot carry a dividend that small over a border
struct FastDiv {
  uint32_t mul;
  int shift;
  __device__ __forceinline__ unsigned quot(unsigned n) const { return (unsigned)(((uint64_t)n * mul) >> shift); }
};

struct WgradParams {
  const void* x; const void* dy; float* partial;
  int64_t M;            // pixels
  int Cout, Cin, Hc, Wc, ksz, up;
  int tiles_m, tiles_n; // tiles over C_out and over C_in
  int rows_per_split;   // multiple of 32
  int K;                // k*k*C_in
  int log_w, log_h;     // log2 of Wc / Hc when both are powers of two (POW2 kernels)
  unsigned x_bytes, dy_bytes;
  int chunks = 0, dy_chunks = 0;   // k_wgrad_chunks: 16-byte chunks of a stored pixel of x and of dY
  FastDiv div_w = {}, div_h = {};  // k_wgrad_chunks: division by Wc and Hc
};

__device__ __forceinline__ bf16x8 lds_tr_frag(const bf16_t* base0, const bf16_t* base1) {
  // two transposing 64-bit loads: pixels p..p+3 and p+4..p+7 of this lane's channel
  short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)base0);
  short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)base1);
  union { short s[8]; bf16x8 v; } u;
  u.s[0] = lo[0]; u.s[1] = lo[1]; u.s[2] = lo[2]; u.s[3] = lo[3];
  u.s[4] = hi[0]; u.s[5] = hi[1]; u.s[6] = hi[2]; u.s[7] = hi[3];
  return u.v;
}

// One slab of MFMAs of the weight-gradient kernel.  sa / sb point at the wave's first
// channel of the [pixel][channel] slabs.
template <typename T, int MI, int NJ, int BK, int LA, int LB>
__device__ __forceinline__ void wgrad_compute(const T* sa, const T* sb, int lane, floatx16 (&acc)[MI][NJ]) {
  if constexpr (sizeof(T) == 2) {
    // transposing-load geometry of this lane: 16-lane group G covers channels 16*(G&1).. of
    // the 32-channel MFMA tile and pixels 8*(G>>1)..; local lane sl addresses pixel sl/4,
    // channels 4*(sl%4)..
    const int grp = lane >> 4, sl = lane & 15;
    const int t_pix = 8 * (grp >> 1) + (sl >> 2);
    const int t_ch = 16 * (grp & 1) + 4 * (sl & 3);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 a[MI], bb[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const bf16_t* q = &sa[(ks * 16 + t_pix) * LA + i * 32 + t_ch];
        a[i] = lds_tr_frag(q, q + 4 * LA);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bf16_t* q = &sb[(ks * 16 + t_pix) * LB + j * 32 + t_ch];
        bb[j] = lds_tr_frag(q, q + 4 * LB);
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bb[j], acc[i][j], 0, 0, 0);
    }
  } else {
    // fp32: lane l supplies channel l%32 of pixel 2*st + l/32 — a plain 4-byte read
    const int ch = lane & 31, half = lane >> 5;
#pragma unroll
    for (int st = 0; st < BK / 2; ++st) {
      float a[MI], bb[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = sa[(2 * st + half) * LA + i * 32 + ch];
#pragma unroll
      for (int j = 0; j < NJ; ++j) bb[j] = sb[(2 * st + half) * LB + j * 32 + ch];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], bb[j], acc[i][j], 0, 0, 0);
    }
  }
}

template <int BM, int BN, bool POW2>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad(WgradParams p) {
  constexpr int ES = 2;
  constexpr int EPC = 8;                         // elements per 16-byte chunk
  constexpr int BK = 32;                         // pixels per slab
  // LDS row strides in elements (64 banks): +64 bytes, so that the 4 pixel rows x 64 bytes that 32 lanes of a
  // transposing load touch tile the 256-byte bank space.
  constexpr int LPAD = 32;
  constexpr int LA = BM + LPAD, LB = BN + LPAD;
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int MI = WM / 32, NJ = WN / 32;
  constexpr int A_TPR = BM / EPC, B_TPR = BN / EPC;  // 16-byte chunks per pixel row
  constexpr int A_CHUNKS = BK * A_TPR / 256, B_CHUNKS = BK * B_TPR / 256;
  __shared__ __attribute__((aligned(16))) bf16_t sA[2][BK * LA];
  __shared__ __attribute__((aligned(16))) bf16_t sB[2][BK * LB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  // block -> (split, tile_m, tile_n, tap): the tap varies fastest so that the blocks
  // sharing a dY slab and overlapping x slabs run at the same time
  const int taps = p.ksz * p.ksz;
  int b = xcd_logical_block((int)blockIdx.x, (int)gridDim.x);
  const int tap = b % taps; b /= taps;
  const int tn = b % p.tiles_n; b /= p.tiles_n;
  const int tm = b % p.tiles_m;
  const int split = b / p.tiles_m;
  const int r = tap / p.ksz, s = tap - r * p.ksz;
  const int pad = (p.ksz - 1) >> 1;
  const int co0 = tm * BM, ci0 = tn * BN;
  const int Hin = p.Hc >> p.up, Win = p.Wc >> p.up;
  const int64_t m_begin = (int64_t)split * p.rows_per_split;
  const int64_t m_end = (m_begin + p.rows_per_split < p.M) ? m_begin + p.rows_per_split : p.M;
  const int KT = (int)((m_end - m_begin + BK - 1) / BK);

  // Buffer loads: rows past the split's end and taps that fall into the zero padding get an
  // offset beyond the tensor and read as zero.  Pixel coordinates come from shifts when the
  // image sides are powers of two (POW2), from divisions otherwise.
  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rDY = make_rsrc(p.dy, p.dy_bytes);
  const unsigned a_col = (unsigned)(co0 * ES);   // + chunk below
  const unsigned b_col = (unsigned)(ci0 * ES);
  int kload = 0;
#define WGRAD_LOAD(RA, RB)                                                                                   \
  {                                                                                                          \
    const int64_t mb = m_begin + (int64_t)kload * BK;                                                        \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i) {                                                   \
      const int id = tid + i * 256;                                                                          \
      const int64_t m = mb + id / A_TPR;                                                                     \
      const unsigned off = m < m_end ? (unsigned)m * (unsigned)(p.Cout * ES) + a_col + (unsigned)(id % A_TPR) * 16u : kOob; \
      RA[i] = __builtin_amdgcn_raw_buffer_load_b128(rDY, off, 0, 0);                                         \
    }                                                                                                        \
    _Pragma("unroll") for (int i = 0; i < B_CHUNKS; ++i) {                                                   \
      const int id = tid + i * 256;                                                                          \
      const int64_t m = mb + id / B_TPR;                                                                     \
      const unsigned mm = (unsigned)m;                                                                       \
      unsigned w, h, n;                                                                                      \
      if (POW2) {                                                                                            \
        w = mm & (unsigned)(p.Wc - 1); h = (mm >> p.log_w) & (unsigned)(p.Hc - 1); n = mm >> (p.log_w + p.log_h); \
      } else {                                                                                               \
        w = mm % (unsigned)p.Wc; const unsigned t = mm / (unsigned)p.Wc;                                     \
        h = t % (unsigned)p.Hc; n = t / (unsigned)p.Hc;                                                      \
      }                                                                                                      \
      const int hh = (int)h + r - pad, ww = (int)w + s - pad;                                                \
      const bool ok = m < m_end && hh >= 0 && hh < p.Hc && ww >= 0 && ww < p.Wc;                             \
      const unsigned pix = (n * (unsigned)Hin + (unsigned)(hh >> p.up)) * (unsigned)Win + (unsigned)(ww >> p.up); \
      const unsigned off = ok ? pix * (unsigned)(p.Cin * ES) + b_col + (unsigned)(id % B_TPR) * 16u : kOob;  \
      RB[i] = __builtin_amdgcn_raw_buffer_load_b128(rX, off, 0, 0);                                          \
    }                                                                                                        \
    ++kload;                                                                                                 \
  }
#define WGRAD_STORE(BUF, RA, RB)                                                                             \
  {                                                                                                          \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i) {                                                   \
      const int id = tid + i * 256;                                                                          \
      *reinterpret_cast<uint4v*>(&sA[BUF][(id / A_TPR) * LA + (id % A_TPR) * EPC]) = RA[i];                  \
    }                                                                                                        \
    _Pragma("unroll") for (int i = 0; i < B_CHUNKS; ++i) {                                                   \
      const int id = tid + i * 256;                                                                          \
      *reinterpret_cast<uint4v*>(&sB[BUF][(id / B_TPR) * LB + (id % B_TPR) * EPC]) = RB[i];                  \
    }                                                                                                        \
  }
#define WGRAD_COMPUTE(BUF) wgrad_compute<bf16_t, MI, NJ, BK, LA, LB>(&sA[BUF][wm * WM], &sB[BUF][wn * WN], lane, acc)

  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // KT >= 1: every split owns at least one pixel (the host sizes the splits that way)
  uint4v ra0[A_CHUNKS], rb0[B_CHUNKS], ra1[A_CHUNKS], rb1[B_CHUNKS];
  WGRAD_LOAD(ra0, rb0);
  if (KT > 1) WGRAD_LOAD(ra1, rb1);
  WGRAD_STORE(0, ra0, rb0);
  __syncthreads();
  for (int kt = 0; kt < KT; kt += 2) {
    if (kt + 2 < KT) WGRAD_LOAD(ra0, rb0);
    WGRAD_COMPUTE(0);
    if (kt + 1 < KT) WGRAD_STORE(1, ra1, rb1);
    __syncthreads();
    if (kt + 1 >= KT) break;
    if (kt + 3 < KT) WGRAD_LOAD(ra1, rb1);
    WGRAD_COMPUTE(1);
    if (kt + 2 < KT) WGRAD_STORE(0, ra0, rb0);
    __syncthreads();
  }
#undef WGRAD_LOAD
#undef WGRAD_STORE
#undef WGRAD_COMPUTE

  // partial[split][co][tap*Cin + ci]
  float* __restrict__ P = p.partial + (int64_t)split * p.Cout * p.K;
  const int col_lane = lane & 31, row_lane = (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int ci = ci0 + wn * WN + j * 32 + col_lane;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int co = co0 + wm * WM + i * 32 + (e >> 2) * 8 + row_lane + (e & 3);
        if (co < p.Cout && ci < p.Cin) P[(int64_t)co * p.K + tap * p.Cin + ci] = acc[i][j][e];
      }
    }
}

// partial[split][co][tap*Cin + ci] of a tile whose columns are the chunks of all taps in a row
template <int EPC, int BM, int BN>
__device__ __forceinline__ void wgrad_store_chunks(const WgradParams& p, const floatx16 (&acc)[BM / 64][BN / 64], int split, int tm, int tn,
                                                   int wm, int wn, int lane) {
  constexpr int WM = BM / 2, WN = BN / 2, MI = WM / 32, NJ = WN / 32;
  const int kc = p.ksz * p.ksz * p.chunks;
  float* __restrict__ P = p.partial + (int64_t)split * p.Cout * p.K;
  const int col_lane = lane & 31, row_lane = (lane >> 5) * 4;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int col = tn * BN + wn * WN + j * 32 + col_lane, q = col / EPC;
    const int tap_o = q / p.chunks, ci = (q - tap_o * p.chunks) * EPC + col % EPC;
    if (q >= kc || ci >= p.Cin) continue;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int co = tm * BM + wm * WM + i * 32 + (e >> 2) * 8 + row_lane + (e & 3);
        if (co < p.Cout) P[(int64_t)co * p.K + tap_o * p.Cin + ci] = acc[i][j][e];
      }
  }
}

// Gradients that are NaN summed again over the pixels whose tap lies inside the image: outside it the kernels multiply by zero,
// NaN for an infinite dY (at the pace of one thread per weight; nothing but infinities and NaN gets here)
template <typename T, int BM, int BN>
__device__ __forceinline__ void wgrad_resum_nan(const WgradParams& p, floatx16 (&acc)[BM / 64][BN / 64], unsigned m_begin, unsigned m_end,
                                                int tm, int tn, int wm, int wn, int lane) {
  constexpr int EPC = 16 / (int)sizeof(T), MI = BM / 64, NJ = BN / 64;
  const uint64_t bits = p.ksz > 1 ? nan_bits(acc) : 0;
  replace_bits<MI, NJ>(acc, bits, [&](int i, int j, int e) {
    const int co = tm * BM + wm * (BM / 2) + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
    const int col = tn * BN + wn * (BN / 2) + j * 32 + (lane & 31), q = col / EPC;
    const int tap = q / p.chunks, ci = (q - tap * p.chunks) * EPC + col % EPC, pad = (p.ksz - 1) >> 1;
    const int dh = tap / p.ksz - pad, dw = tap % p.ksz - pad, Hin = p.Hc >> p.up, Win = p.Wc >> p.up;
    if (co >= p.Cout || tap >= p.ksz * p.ksz || ci >= p.Cin || (dh == 0 && dw == 0)) return __builtin_nanf("");
    const T* const x = reinterpret_cast<const T*>(p.x) + ci;
    const T* const dy = reinterpret_cast<const T*>(p.dy) + co;
    float v = 0.0f;
    for (unsigned m = m_begin; m < m_end && v == v; ++m) {      // (NaN stays NaN)
      const unsigned t = m / (unsigned)p.Wc, n = t / (unsigned)p.Hc;
      const int hh = (int)(t - n * (unsigned)p.Hc) + dh, ww = (int)(m - t * (unsigned)p.Wc) + dw;
      if (hh < 0 || hh >= p.Hc || ww < 0 || ww >= p.Wc) continue;
      const int64_t pix = ((int64_t)n * Hin + (hh >> p.up)) * Win + (ww >> p.up);
      v = fmaf(Store<T>::ld(dy + (int64_t)m * p.dy_chunks * EPC), Store<T>::ld(x + pix * p.chunks * EPC), v);
    }
    return v;
  });
}

// The same for any channel counts.  Pixels of x and dY are stored as whole 16-byte chunks (zeros behind the channels),
// and the columns of the product are the chunks of all taps in a row, (tap, chunk), cut into tiles of BN wherever a tile
// ends: a loader thread moves the same column chunk in every pass, so its tap is fixed for the whole loop and the tile
// border costs nothing.  9 x 48 channels fill 3.4 tiles of 128 columns, where a tile per tap would be 9 with a quarter
// of each empty; a 3-channel image fills 0.6 tiles instead of 9.  Chunks past the end read zeros and are not stored.
// Measured (bf16, 24 x 36 x 60 pixels, 80 x 9 x 48 weights): 22 us = 160 TFLOP/s, where a thread per weight that walks the
// pixels alone took 4.5 ms.
template <int BM, int BN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad_chunks(WgradParams p) {
  constexpr int ES = 2;
  constexpr int EPC = 8;
  constexpr int BK = 32;                         // pixels per slab
  constexpr int LPAD = 32;                       // (as in k_wgrad)
  constexpr int LA = BM + LPAD, LB = BN + LPAD;
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int MI = WM / 32, NJ = WN / 32;
  constexpr int A_TPR = BM / EPC, B_TPR = BN / EPC;
  constexpr int A_CHUNKS = BK * A_TPR / 256, B_CHUNKS = BK * B_TPR / 256;
  static_assert(256 % A_TPR == 0 && 256 % B_TPR == 0, "a thread keeps its column chunk");
  __shared__ __attribute__((aligned(16))) bf16_t sA[2][BK * LA];
  __shared__ __attribute__((aligned(16))) bf16_t sB[2][BK * LB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int b = xcd_logical_block((int)blockIdx.x, (int)gridDim.x);     // column tiles fastest: they share a dY slab
  const int tn = b % p.tiles_n; b /= p.tiles_n;
  const int tm = b % p.tiles_m;
  const int split = b / p.tiles_m;
  const int pad = (p.ksz - 1) >> 1, kc = p.ksz * p.ksz * p.chunks;
  const int Hin = p.Hc >> p.up, Win = p.Wc >> p.up;
  const unsigned m_begin = (unsigned)split * (unsigned)p.rows_per_split;
  const unsigned m_end = min(m_begin + (unsigned)p.rows_per_split, (unsigned)p.M);
  const int KT = (int)((m_end - m_begin + BK - 1) / BK);
  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rDY = make_rsrc(p.dy, p.dy_bytes);

  const int ca = tm * A_TPR + tid % A_TPR;       // this thread's column chunk of dY ...
  const int cb = tn * B_TPR + tid % B_TPR;       // ... and of the gathered input: tap (r, s), channels 16-byte chunk cc
  const int tap = cb / p.chunks, cc = cb - tap * p.chunks, r = tap / p.ksz, s = tap - r * p.ksz;
  const bool a_in = ca < p.dy_chunks, b_in = cb < kc;
  unsigned ma = m_begin + (unsigned)(tid / A_TPR), mb = m_begin + (unsigned)(tid / B_TPR);   // pixels of the next slab
  auto load = [&](uint4v (&ra)[A_CHUNKS], uint4v (&rb)[B_CHUNKS]) {
#pragma unroll
    for (int i = 0; i < A_CHUNKS; ++i) {
      const unsigned m = ma + i * (256 / A_TPR);
      ra[i] = __builtin_amdgcn_raw_buffer_load_b128(rDY, a_in && m < m_end ? (m * (unsigned)p.dy_chunks + (unsigned)ca) * 16u : kOob, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < B_CHUNKS; ++i) {
      const unsigned m = mb + i * (256 / B_TPR);
      const unsigned t = p.div_w.quot(m), n = p.div_h.quot(t);
      const int hh = (int)(t - n * (unsigned)p.Hc) + r - pad, ww = (int)(m - t * (unsigned)p.Wc) + s - pad;
      const bool ok = b_in && m < m_end && hh >= 0 && hh < p.Hc && ww >= 0 && ww < p.Wc;
      const unsigned pix = (n * (unsigned)Hin + (unsigned)(hh >> p.up)) * (unsigned)Win + (unsigned)(ww >> p.up);
      rb[i] = __builtin_amdgcn_raw_buffer_load_b128(rX, ok ? (pix * (unsigned)p.chunks + (unsigned)cc) * 16u : kOob, 0, 0);
    }
    ma += BK;
    mb += BK;
  };
  auto store = [&](int buf, const uint4v (&ra)[A_CHUNKS], const uint4v (&rb)[B_CHUNKS]) {
#pragma unroll
    for (int i = 0; i < A_CHUNKS; ++i)
      *reinterpret_cast<uint4v*>(&sA[buf][(tid / A_TPR + i * (256 / A_TPR)) * LA + (tid % A_TPR) * EPC]) = ra[i];
#pragma unroll
    for (int i = 0; i < B_CHUNKS; ++i)
      *reinterpret_cast<uint4v*>(&sB[buf][(tid / B_TPR + i * (256 / B_TPR)) * LB + (tid % B_TPR) * EPC]) = rb[i];
  };
  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // KT >= 1: every split owns at least one pixel (the host sizes the splits that way)
  uint4v ra0[A_CHUNKS], rb0[B_CHUNKS], ra1[A_CHUNKS], rb1[B_CHUNKS];
  load(ra0, rb0);
  if (KT > 1) load(ra1, rb1);
  store(0, ra0, rb0);
  __syncthreads();
  for (int kt = 0; kt < KT; kt += 2) {
    if (kt + 2 < KT) load(ra0, rb0);
    wgrad_compute<bf16_t, MI, NJ, BK, LA, LB>(&sA[0][wm * WM], &sB[0][wn * WN], lane, acc);
    if (kt + 1 < KT) store(1, ra1, rb1);
    __syncthreads();
    if (kt + 1 >= KT) break;
    if (kt + 3 < KT) load(ra1, rb1);
    wgrad_compute<bf16_t, MI, NJ, BK, LA, LB>(&sA[1][wm * WM], &sB[1][wn * WN], lane, acc);
    if (kt + 2 < KT) store(0, ra0, rb0);
    __syncthreads();
  }

  wgrad_resum_nan<bf16_t, BM, BN>(p, acc, m_begin, m_end, tm, tn, wm, wn, lane);
  wgrad_store_chunks<EPC, BM, BN>(p, acc, split, tm, tn, wm, wn, lane);
}

// The same for binary32: the three bfloat16 parts of k_gemm_split, cut on the way into LDS ([part][pixel][channel], read back
// with the transposing loads), the six part products in two accumulators.  Slabs of 16 pixels, two LDS stages, one
// barrier per slab, the split of the next slab between the MFMAs of this one.  128 x 9 x 128 weights over 65,536 pixels: 106 us
// where the binary32 MFMA took 143 (both beside the input gradients on the other stream).  A workgroup that meets an operand
// below 2^-110 other than zero, or has a sum that is no finite number, computes its tile again with the binary32 MFMA (the reasons
// as there).
template <int BM, int BN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad_split(WgradParams p) {
  constexpr int BK = 16;                         // pixels per slab
  constexpr int LA = BM + 32, LB = BN + 32;      // (parts: as in k_wgrad; binary32: +128 bytes, the two pixel rows of a 64-lane 4-byte read are 32 banks apart)
  constexpr int WM = BM / 2, WN = BN / 2, MI = WM / 32, NJ = WN / 32;
  constexpr int A_TPR = BM / 4, B_TPR = BN / 4;
  constexpr int AC = BK * A_TPR / 256, BC = BK * B_TPR / 256;
  constexpr int PA = BK * LA * 2, PB = BK * LB * 2, STAGE = 3 * (PA + PB);
  static_assert(2 * STAGE >= 2 * BK * (LA + LB) * 4, "the binary32 loop fits into the same memory");
  __shared__ __attribute__((aligned(16))) char smem[2 * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int b = xcd_logical_block((int)blockIdx.x, (int)gridDim.x);
  const int tn = b % p.tiles_n; b /= p.tiles_n;
  const int tm = b % p.tiles_m;
  const int split_id = b / p.tiles_m;
  const int pad = (p.ksz - 1) >> 1, kc = p.ksz * p.ksz * p.chunks;
  const int Hin = p.Hc >> p.up, Win = p.Wc >> p.up;
  const unsigned m_begin = (unsigned)split_id * (unsigned)p.rows_per_split;
  const unsigned m_end = min(m_begin + (unsigned)p.rows_per_split, (unsigned)p.M);
  const int KT = (int)((m_end - m_begin + BK - 1) / BK);
  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rDY = make_rsrc(p.dy, p.dy_bytes);
  const int ca = tm * A_TPR + tid % A_TPR, cb = tn * B_TPR + tid % B_TPR;
  const int tap = cb / p.chunks, cc = cb - tap * p.chunks, r = tap / p.ksz, s = tap - r * p.ksz;
  const bool a_in = ca < p.dy_chunks, b_in = cb < kc;
  unsigned ma = m_begin + (unsigned)(tid / A_TPR), mb = m_begin + (unsigned)(tid / B_TPR);   // pixels of the next slab
  auto load_a = [&](uint4v& v, int i) {
    const unsigned m = ma + i * (256 / A_TPR);
    v = __builtin_amdgcn_raw_buffer_load_b128(rDY, a_in && m < m_end ? (m * (unsigned)p.dy_chunks + (unsigned)ca) * 16u : kOob, 0, 0);
  };
  auto load_b = [&](uint4v& v, int i) {
    const unsigned m = mb + i * (256 / B_TPR);
    const unsigned t = p.div_w.quot(m), n = p.div_h.quot(t);
    const int hh = (int)(t - n * (unsigned)p.Hc) + r - pad, ww = (int)(m - t * (unsigned)p.Wc) + s - pad;
    const bool ok = b_in && m < m_end && hh >= 0 && hh < p.Hc && ww >= 0 && ww < p.Wc;
    const unsigned pix = (n * (unsigned)Hin + (unsigned)(hh >> p.up)) * (unsigned)Win + (unsigned)(ww >> p.up);
    v = __builtin_amdgcn_raw_buffer_load_b128(rX, ok ? (pix * (unsigned)p.chunks + (unsigned)cc) * 16u : kOob, 0, 0);
  };
  uint4v ra[AC], rb[BC];
  unsigned lo = ~0u;
  auto split = [&](char* dst, int plane, const uint4v& v) {
    track_smallest(lo, v);
    float4v x = __builtin_bit_cast(float4v, v);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint32_t w0 = pack_bf16(x[0], x[1]), w1 = pack_bf16(x[2], x[3]);
      *reinterpret_cast<uint2*>(dst + q * plane) = make_uint2(w0, w1);
      x[0] -= __uint_as_float(w0 << 16); x[1] -= __uint_as_float(w0 & 0xFFFF0000u);
      x[2] -= __uint_as_float(w1 << 16); x[3] -= __uint_as_float(w1 & 0xFFFF0000u);
    }
  };
  char* const sta = smem + ((tid / A_TPR) * LA + (tid % A_TPR) * 4) * 2;
  char* const stb = smem + 3 * PA + ((tid / B_TPR) * LB + (tid % B_TPR) * 4) * 2;
  auto refill = [&](int buf) {                   // registers into a stage, then the slab after that into the registers
#pragma unroll
    for (int i = 0; i < AC; ++i) { split(sta + buf * STAGE + i * (256 / A_TPR) * LA * 2, PA, ra[i]); load_a(ra[i], i); }
#pragma unroll
    for (int i = 0; i < BC; ++i) { split(stb + buf * STAGE + i * (256 / B_TPR) * LB * 2, PB, rb[i]); load_b(rb[i], i); }
    ma += BK;
    mb += BK;
  };
  floatx16 acc[MI][NJ], low[MI][NJ];             // the leading products, the five small ones
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.0f;
  // transposing-load geometry: as in wgrad_compute
  const int grp = lane >> 4, sl = lane & 15;
  const int t_pix = 8 * (grp >> 1) + (sl >> 2), t_ch = 16 * (grp & 1) + 4 * (sl & 3);
  bf16x8 fa[3][MI], fb[3][NJ];
  auto read = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const bf16_t* a = reinterpret_cast<const bf16_t*>(smem + buf * STAGE + q * PA) + t_pix * LA + wm * WM + i * 32 + t_ch;
        fa[q][i] = lds_tr_frag(a, a + 4 * LA);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bf16_t* x = reinterpret_cast<const bf16_t*>(smem + buf * STAGE + 3 * PA + q * PB) + t_pix * LB + wn * WN + j * 32 + t_ch;
        fb[q][j] = lds_tr_frag(x, x + 4 * LB);
      }
    }
  };
  auto products = [&]() {
    constexpr int QA[6] = {0, 0, 1, 1, 0, 2}, QB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          floatx16& c = t == 0 ? acc[i][j] : low[i][j];
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[QA[t]][i], fb[QB[t]][j], c, 0, 0, 0);
        }
  };
#pragma unroll
  for (int i = 0; i < AC; ++i) load_a(ra[i], i);
#pragma unroll
  for (int i = 0; i < BC; ++i) load_b(rb[i], i);
  ma += BK;
  mb += BK;
  refill(0);
  __syncthreads();
  for (int kt = 1; kt < KT; ++kt) {              // (KT >= 1: every split owns at least one pixel)
    const int buf = (kt & 1) ^ 1;
    read(buf);
    __builtin_amdgcn_sched_barrier(0);           // (the reads stay ahead of the MFMAs they would otherwise be sunk to)
    products();
    refill(buf ^ 1);
#pragma unroll
    for (int g = 0; g < 6 * MI * NJ; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, (AC * 36 + BC * 56) / (6 * MI * NJ) + 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
  }
  read((KT & 1) ^ 1);
  products();
  const bool odd = add_not_finite(acc, low) || parts_inexact(lo);
  if (__syncthreads_or(odd) != 0) {
    float* const sA = reinterpret_cast<float*>(smem);
    float* const sB = sA + BK * LA;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    ma = m_begin + (unsigned)(tid / A_TPR);
    mb = m_begin + (unsigned)(tid / B_TPR);
    for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
      for (int i = 0; i < AC; ++i) { load_a(ra[i], i); *reinterpret_cast<uint4v*>(&sA[(tid / A_TPR + i * (256 / A_TPR)) * LA + (tid % A_TPR) * 4]) = ra[i]; }
#pragma unroll
      for (int i = 0; i < BC; ++i) { load_b(rb[i], i); *reinterpret_cast<uint4v*>(&sB[(tid / B_TPR + i * (256 / B_TPR)) * LB + (tid % B_TPR) * 4]) = rb[i]; }
      ma += BK;
      mb += BK;
      __syncthreads();
      wgrad_compute<float, MI, NJ, BK, LA, LB>(&sA[wm * WM], &sB[wn * WN], lane, acc);
      __syncthreads();
    }
    wgrad_resum_nan<float, BM, BN>(p, acc, m_begin, m_end, tm, tn, wm, wn, lane);
  }
  wgrad_store_chunks<4, BM, BN>(p, acc, split_id, tm, tn, wm, wn, lane);
}

// The same kernel for images whose width is a multiple of the slab depth BK: a slab is then BK
// consecutive pixels of ONE image row, so the sample, the row and the row's validity for the
// block's tap are uniform (scalar registers, advanced incrementally) and a thread's share of the
// address arithmetic is one add, one compare and one select per 16-byte load.  The output
// gradient advances through the scalar offset of the buffer load.  Every slab is full (the
// host makes the splits multiples of BK).
template <int BM, int BN, int BK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad_rows(WgradParams p) {
  constexpr int ES = 2;
  constexpr int EPC = 8;
  constexpr int LPAD = 32;
  constexpr int LA = BM + LPAD, LB = BN + LPAD;
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int MI = WM / 32, NJ = WN / 32;
  constexpr int A_TPR = BM / EPC, B_TPR = BN / EPC;
  constexpr int A_CHUNKS = BK * A_TPR / 256, B_CHUNKS = BK * B_TPR / 256;
  static_assert(A_CHUNKS >= 1 && B_CHUNKS >= 1, "slab too small for 256 loader threads");
  __shared__ __attribute__((aligned(16))) bf16_t sA[2][BK * LA];
  __shared__ __attribute__((aligned(16))) bf16_t sB[2][BK * LB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int taps = p.ksz * p.ksz;
  int b = xcd_logical_block((int)blockIdx.x, (int)gridDim.x);
  const int tap = b % taps; b /= taps;
  const int tn = b % p.tiles_n; b /= p.tiles_n;
  const int tm = b % p.tiles_m;
  const int split = b / p.tiles_m;
  const int r = tap / p.ksz, s = tap - r * p.ksz;
  const int pad = (p.ksz - 1) >> 1;
  const int co0 = tm * BM, ci0 = tn * BN;
  const int Hin = p.Hc >> p.up, Win = p.Wc >> p.up;
  const int64_t m_begin = (int64_t)split * p.rows_per_split;
  const int64_t m_end = (m_begin + p.rows_per_split < p.M) ? m_begin + p.rows_per_split : p.M;
  const int KT = (int)((m_end - m_begin) / BK);

  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rDY = make_rsrc(p.dy, p.dy_bytes);
  unsigned a_voff[A_CHUNKS], b_voff[B_CHUNKS];
  int b_pw[B_CHUNKS];
#pragma unroll
  for (int i = 0; i < A_CHUNKS; ++i) {
    const int id = tid + i * 256;
    a_voff[i] = (unsigned)(id / A_TPR) * (unsigned)(p.Cout * ES) + (unsigned)(co0 * ES) + (unsigned)(id % A_TPR) * 16u;
  }
#pragma unroll
  for (int i = 0; i < B_CHUNKS; ++i) {
    const int id = tid + i * 256;
    b_pw[i] = id / B_TPR + s - pad;
    b_voff[i] = (unsigned)(ci0 * ES) + (unsigned)(id % B_TPR) * 16u;
  }
  // coordinates of the next slab to load (uniform)
  unsigned a_soff = (unsigned)m_begin * (unsigned)(p.Cout * ES);
  int w0 = (int)((unsigned)m_begin % (unsigned)p.Wc);
  int h = (int)(((unsigned)m_begin / (unsigned)p.Wc) % (unsigned)p.Hc);
  int n = (int)((unsigned)m_begin / ((unsigned)p.Wc * (unsigned)p.Hc));
  const unsigned cin_bytes = (unsigned)(p.Cin * ES);
#define WGRAD_LOAD(RA, RB)                                                                                   \
  {                                                                                                          \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i)                                                     \
        RA[i] = __builtin_amdgcn_raw_buffer_load_b128(rDY, a_voff[i], a_soff, 0);                            \
    const int hh = h + r - pad;                                                                              \
    const bool row_ok = hh >= 0 && hh < p.Hc;                                                                \
    const unsigned row_base = ((unsigned)n * (unsigned)Hin + (unsigned)((row_ok ? hh : 0) >> p.up)) * (unsigned)Win * cin_bytes; \
    _Pragma("unroll") for (int i = 0; i < B_CHUNKS; ++i) {                                                   \
      const int ww = w0 + b_pw[i];                                                                           \
      const bool ok = row_ok && (unsigned)ww < (unsigned)p.Wc;                                               \
      const unsigned off = ok ? row_base + (unsigned)(ww >> p.up) * cin_bytes + b_voff[i] : kOob;            \
      RB[i] = __builtin_amdgcn_raw_buffer_load_b128(rX, off, 0, 0);                                          \
    }                                                                                                        \
    a_soff += (unsigned)(BK * p.Cout * ES);                                                                  \
    w0 += BK;                                                                                                \
    if (w0 == p.Wc) { w0 = 0; if (++h == p.Hc) { h = 0; ++n; } }                                             \
  }
#define WGRAD_STORE(BUF, RA, RB)                                                                             \
  {                                                                                                          \
    _Pragma("unroll") for (int i = 0; i < A_CHUNKS; ++i) {                                                   \
      const int id = tid + i * 256;                                                                          \
      *reinterpret_cast<uint4v*>(&sA[BUF][(id / A_TPR) * LA + (id % A_TPR) * EPC]) = RA[i];                  \
    }                                                                                                        \
    _Pragma("unroll") for (int i = 0; i < B_CHUNKS; ++i) {                                                   \
      const int id = tid + i * 256;                                                                          \
      *reinterpret_cast<uint4v*>(&sB[BUF][(id / B_TPR) * LB + (id % B_TPR) * EPC]) = RB[i];                  \
    }                                                                                                        \
  }
#define WGRAD_COMPUTE(BUF) wgrad_compute<bf16_t, MI, NJ, BK, LA, LB>(&sA[BUF][wm * WM], &sB[BUF][wn * WN], lane, acc)

  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  uint4v ra0[A_CHUNKS], rb0[B_CHUNKS], ra1[A_CHUNKS], rb1[B_CHUNKS];
  WGRAD_LOAD(ra0, rb0);
  if (KT > 1) WGRAD_LOAD(ra1, rb1);
  WGRAD_STORE(0, ra0, rb0);
  __syncthreads();
  for (int kt = 0; kt < KT; kt += 2) {
    if (kt + 2 < KT) WGRAD_LOAD(ra0, rb0);
    WGRAD_COMPUTE(0);
    if (kt + 1 < KT) WGRAD_STORE(1, ra1, rb1);
    __syncthreads();
    if (kt + 1 >= KT) break;
    if (kt + 3 < KT) WGRAD_LOAD(ra1, rb1);
    WGRAD_COMPUTE(1);
    if (kt + 2 < KT) WGRAD_STORE(0, ra0, rb0);
    __syncthreads();
  }
#undef WGRAD_LOAD
#undef WGRAD_STORE
#undef WGRAD_COMPUTE

  float* __restrict__ P = p.partial + (int64_t)split * p.Cout * p.K;
  const int col_lane = lane & 31, row_lane = (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int ci = ci0 + wn * WN + j * 32 + col_lane;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int co = co0 + wm * WM + i * 32 + (e >> 2) * 8 + row_lane + (e & 3);
        P[(int64_t)co * p.K + tap * p.Cin + ci] = acc[i][j][e];   // tiles divide C_out and C_in exactly
      }
    }
}

// ---------------------------------------------------------------------------
// Weight gradient of a 3x3 convolution, three taps (one filter row r) per workgroup (bf16).
//
// With one tap per workgroup the slabs of dY and of the shifted input stream through the vector
// cache once per tap, and its 64 bytes per clock bound the kernel at about half the MFMA rate.
// Here a workgroup owns BM output channels x 64 input channels x the three taps (r, s = 0..2): per
// slab of 64 consecutive pixels it loads the dY slab once and ONE input patch — the slab's pixels
// of row h + r - 1 plus one pixel of halo on each side — from which the three taps are shifted
// views.  Slabs never straddle image rows (the host checks W % 64 == 0 or 64 % W == 0); a slab of
// a narrow image (W = SW < 64) is 64/SW whole rows, each with its own halo.
// LDS (three stages, filled by global-to-LDS loads): dY slab [64 px][BM] and patch
// [64/SW segments][SW + 4 cells][64 ci]; cell 1 of a segment is the left halo, cells 2..SW+1 the
// slab's pixels, cell SW+2 the right halo.  The 64-byte columns of a row are XOR-swizzled with
// the pixel / cell index such that the transposing reads (8 pixels x 64 bytes per instruction)
// spread evenly over the banks; for every fragment the swizzle is a per-lane constant, so all
// reads are base + immediate.  Schedule per slab: wait for the next slab's loads, barrier, issue
// the loads of the slab after that, then four K-steps of 16 pixels with the fragments of the
// next K-step (the first of the next slab included) in flight behind the MFMAs.
// ---------------------------------------------------------------------------
// The patch operand of a K-step for all taps of a filter row at once: pixels 0..11 of a lane's channel, from the
// lane's cell on.  Tap s of pixel j reads cell j + s, so the operand of tap s is pixels s .. s+7 of this run: the taps
// are cut out of one 12-pixel read in registers (funnel shifts for the odd tap) instead of being read from LDS once
// each — three 8-byte reads per K-step instead of six, on the port that bounds this kernel.
struct TrRun { uint2v lo, hi, ex; };            // pixels 0..3, 4..7, 8..11
template <int OFF>
__device__ __forceinline__ void tr_read_run(TrRun& f, unsigned addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.lo) : "v"(addr), "n"(OFF));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.hi) : "v"(addr), "n"(OFF + 4 * 128));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.ex) : "v"(addr), "n"(OFF + 8 * 128));
#endif
}
template <int NTAP>
__device__ __forceinline__ void tr_run_taps(TrRun& f, bf16x8 (&bv)[NTAP]) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(f.lo), "+v"(f.hi), "+v"(f.ex));
#endif
  const unsigned d0 = f.lo[0], d1 = f.lo[1], d2 = f.hi[0], d3 = f.hi[1], d4 = f.ex[0];
  union { unsigned w[4]; bf16x8 v; } u;
  u.w[0] = d0; u.w[1] = d1; u.w[2] = d2; u.w[3] = d3;
  bv[0] = u.v;
  if (NTAP > 1) {
    u.w[0] = __builtin_amdgcn_alignbit(d1, d0, 16); u.w[1] = __builtin_amdgcn_alignbit(d2, d1, 16);
    u.w[2] = __builtin_amdgcn_alignbit(d3, d2, 16); u.w[3] = __builtin_amdgcn_alignbit(d4, d3, 16);
    bv[1] = u.v;
  }
  if (NTAP > 2) {
    u.w[0] = d1; u.w[1] = d2; u.w[2] = d3; u.w[3] = d4;
    bv[NTAP > 2 ? 2 : 0] = u.v;
  }
}
__device__ __forceinline__ bf16x8 tr_value(TrFrag& f) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(f.lo), "+v"(f.hi));
#endif
  union { uint2v h[2]; bf16x8 v; } u;
  u.h[0] = f.lo; u.h[1] = f.hi;
  return u.v;
}

template <int BM, int SW>
struct Wgrad3 {
  static constexpr int BK = 64, SR = BK / SW, PCW = SW + 4, PCELLS = SR * PCW;
  static constexpr int RBA = BM * 2;            // bytes per pixel of the dY slab (256 or 128)
  static constexpr int A_BYTES = BK * RBA, A_PASSES = A_BYTES / 4096;
  static constexpr int X_UNITS = (PCELLS * 128 + 1023) / 1024;      // 1 KB = one wave-wide load
  static constexpr int XU = (X_UNITS + 3) / 4;   // units per wave
  static constexpr int STAGE = A_BYTES + X_UNITS * 1024;
  static constexpr int MI = BM / 64;            // 2x2 waves, wave tile (BM/2) x 32 per tap
  // K-step ks covers slab pixels 16*ks .. 16*ks+15: first cell (tap s = 0, before the +1+s) of the patch
  static constexpr int cell_base(int ks) { return ((ks * 16) / SW) * PCW + (ks * 16) % SW; }
};

// fragments of one K-step: MI of dY, the patch run that holds every tap (b_addr: the lane's address for tap 0)
template <int BM, int SW, int KS>
__device__ __forceinline__ void wgrad3_reads(TrFrag (&fa)[BM / 64], TrRun& fb, unsigned a_addr, unsigned b_addr) {
  typedef Wgrad3<BM, SW> G;
#pragma unroll
  for (int i = 0; i < G::MI; ++i) {
    // column i of the wave's co range: the swizzled column differs from a_addr's by (i << 6) XORed in
    if (i == 0) tr_read_at<KS * 16 * G::RBA, 4 * G::RBA>(fa[0], a_addr);
    else tr_read_at<KS * 16 * G::RBA, 4 * G::RBA>(fa[i], a_addr ^ 64u);
  }
  tr_read_run<G::cell_base(KS) * 128>(fb, b_addr);
}

// UP2: the convolution reads its input through a x2 nearest-neighbour upsample.  An output pixel (2i+a, 2j+b) then
// sees only 2 x 2 distinct stored pixels, (i + u - (1-a), j + v - (1-b)), u, v in {0,1}, and the nine taps fall onto
// them: r -> u = (a == 0 ? r > 0 : r > 1), s -> v likewise.  So the kernel forms, per output parity (a, b), the four
// correlations of that phase's quarter of dY with the shifted stored input — 16 tap matrices of a quarter of the
// pixels each, 4/9 of the multiply-adds — and k_wgrad_reduce_up2 adds, for every weight (r, s), the four phase
// matrices it belongs to (exact in real arithmetic; every product is of the same bf16 values as in the plain form).
// A workgroup owns (a, b, u) and the two taps v = 0, 1: a slab is 64 pixels of one phase (every other pixel of every
// other dY row, gathered by the global-to-LDS load), the patch is a row of the STORED image with its halo, and SW,
// Hc, Wc, M below are those of the stored image.
template <int BM, int SW, bool UP2>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad_row3(WgradParams p) {
  typedef Wgrad3<BM, SW> G;
  constexpr int MI = G::MI;
  constexpr int NTAP = UP2 ? 2 : 3;
  // (XOR address arithmetic below needs the alignment; 256 bytes of slack: the last pixels of a patch run may lie one
  // cell past the last stage's patch — they are read, never used)
  __shared__ __attribute__((aligned(1024))) char smem[3 * G::STAGE + 256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int b = xcd_logical_block((int)blockIdx.x, (int)gridDim.x);
  const int r = b % (UP2 ? 8 : 3); b /= (UP2 ? 8 : 3);      // UP2: r = (a, b, u) as three bits
  const int par_a = (r >> 2) & 1, par_b = (r >> 1) & 1, par_u = r & 1;
  const int tn = b % p.tiles_n; b /= p.tiles_n;
  const int tm = b % p.tiles_m;
  const int split = b / p.tiles_m;
  const int co0 = tm * BM, ci0 = tn * 64;
  const int Hin = UP2 ? p.Hc : (p.Hc >> p.up), Win = UP2 ? p.Wc : (p.Wc >> p.up);
  const int64_t m_begin = (int64_t)split * p.rows_per_split;
  const int64_t m_end = (m_begin + p.rows_per_split < p.M) ? m_begin + p.rows_per_split : p.M;
  const int KT = (int)((m_end - m_begin) / G::BK);
  const __amdgpu_buffer_rsrc_t rX = make_rsrc(p.x, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rDY = make_rsrc(p.dy, p.dy_bytes);

  // ---- loaders.  dY: slot q = pass*256 + tid of the linear slab: pixel q / CPP, chunk q % CPP
  constexpr int CPP = G::RBA / 16;
  unsigned a_voff[G::A_PASSES];
#pragma unroll
  for (int i = 0; i < G::A_PASSES; ++i) {
    const int q = i * 256 + tid;
    const int px = q / CPP, chunk = q % CPP;
    const int sw = G::RBA == 256 ? (px & 3) : ((px >> 1) & 1);
    // UP2: slab pixel px = (segment row px / SW, column px % SW) of the stored image is dY pixel (2 row + a, 2 column + b)
    const unsigned dpx = UP2 ? (unsigned)((px / SW) * 2 * (2 * p.Wc) + (px % SW) * 2) : (unsigned)px;
    a_voff[i] = dpx * (unsigned)(p.Cout * 2) + (unsigned)(co0 * 2) + (unsigned)((chunk ^ (sw << 2)) * 16);
  }
  // patch: unit u = wave + 4*k of 1 KB: slot q = u*64 + lane: cell q / 8, chunk q % 8
  int x_seg[G::XU], x_pc[G::XU];
  unsigned x_chunk[G::XU];
  bool x_cell_ok[G::XU];
#pragma unroll
  for (int k = 0; k < G::XU; ++k) {
    const int q = (wave + 4 * k) * 64 + lane;
    const int cell = q >> 3;
    x_seg[k] = cell / G::PCW;
    x_pc[k] = cell - x_seg[k] * G::PCW;
    x_chunk[k] = (unsigned)(((q & 7) ^ (((cell >> 1) & 1) << 2)) * 16) + (unsigned)(ci0 * 2);
    x_cell_ok[k] = cell < G::PCELLS && x_pc[k] >= 1 && x_pc[k] <= SW + 2;
  }
  // coordinates of the next slab to load (uniform)
  unsigned a_soff = (unsigned)m_begin * (unsigned)(p.Cout * 2);     // (UP2: recomputed from (n, h, w0) per slab)
  int w0 = (int)((unsigned)m_begin % (unsigned)p.Wc);
  int h = (int)(((unsigned)m_begin / (unsigned)p.Wc) % (unsigned)p.Hc);
  int n = (int)((unsigned)m_begin / ((unsigned)p.Wc * (unsigned)p.Hc));
  const unsigned cin_bytes = (unsigned)(p.Cin * 2);
#define WGRAD3_DMA(STG)                                                                                      \
  {                                                                                                          \
    char* const da = smem + (STG) * G::STAGE + wave * 1024;                                                  \
    if (UP2) a_soff = (((unsigned)n * (unsigned)(2 * p.Hc) + (unsigned)(2 * h + par_a)) * (unsigned)(2 * p.Wc) + (unsigned)(2 * w0 + par_b)) * (unsigned)(p.Cout * 2); \
    _Pragma("unroll") for (int i = 0; i < G::A_PASSES; ++i)                                                  \
        dma_load16s(rDY, da + i * 4096, a_voff[i], a_soff);                                                  \
    _Pragma("unroll") for (int k = 0; k < G::XU; ++k) {                                                      \
      if (wave + 4 * k < G::X_UNITS) {                                                                       \
        const int row = h + x_seg[k] + (UP2 ? par_u + par_a - 1 : r - 1), col = w0 + x_pc[k] - 2;            \
        const bool ok = x_cell_ok[k] && row >= 0 && row < p.Hc && col >= 0 && col < p.Wc;                    \
        const unsigned pix = UP2 ? ((unsigned)n * (unsigned)Hin + (unsigned)row) * (unsigned)Win + (unsigned)col        \
                                 : ((unsigned)n * (unsigned)Hin + (unsigned)(row >> p.up)) * (unsigned)Win + (unsigned)(col >> p.up); \
        dma_load16(rX, smem + (STG) * G::STAGE + G::A_BYTES + (wave + 4 * k) * 1024, ok ? pix * cin_bytes + x_chunk[k] : kOob); \
      }                                                                                                      \
    }                                                                                                        \
    if (!UP2) a_soff += (unsigned)(G::BK * p.Cout * 2);                                                      \
    if (SW < 64) { h += G::SR; if (h == p.Hc) { h = 0; ++n; } }                                              \
    else { w0 += 64; if (w0 == p.Wc) { w0 = 0; if (++h == p.Hc) { h = 0; ++n; } } }                          \
  }

  // ---- fragment addresses (per-lane constants).  Transposing read: within 16 lanes, lane 4*j+q
  // addresses 4 channels (4q..) of pixel j; 16-lane group G: channels +16*(G&1), pixels +8*(G>>1)
  const int grp = lane >> 4, sl = lane & 15;
  const int lp = 8 * (grp >> 1) + (sl >> 2);
  const unsigned lds0 = (unsigned)(size_t)(lds_char*)smem;
  const int a_col = G::RBA == 256 ? (2 * wm) : wm;                       // 64-byte column of the wave's first 32 channels
  const int a_sw = G::RBA == 256 ? (lp & 3) : ((lp >> 1) & 1);
  const unsigned a_lane = (unsigned)(lp * G::RBA + ((a_col ^ a_sw) << 6) + 32 * (grp & 1) + 8 * (sl & 3));
  unsigned b_lane;                               // tap 0; tap s is s cells further (tr_run_taps)
  {
    // (UP2: tap v of column parity b reads stored column j + v - (1-b): the view shifted by b + v - 1)
    // (SW = 8: the 16 pixels of a K-step are two segment rows of the patch, PCW cells apart)
    const int lp_cell = SW >= 16 ? lp : (lp / SW) * G::PCW + lp % SW;
    const int cell = 1 + (UP2 ? par_b : 0) + lp_cell;   // + cell_base(ks) (a multiple of 4), + 4 and + 8 for the next pixels
    b_lane = (unsigned)(G::A_BYTES + cell * 128 + ((wn ^ ((cell >> 1) & 1)) << 6) + 32 * (grp & 1) + 8 * (sl & 3));
  }

  floatx16 acc[NTAP][MI];
#pragma unroll
  for (int s_ = 0; s_ < NTAP; ++s_)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[s_][i][e] = 0.0f;

  [[maybe_unused]] TrFrag fa0[MI], fa1[MI];      // (used by the device pass only)
  [[maybe_unused]] TrRun fb0, fb1;
  [[maybe_unused]] constexpr int NR = 2 * MI + 3;                    // LDS reads per K-step
#define WGRAD3_MMA(FA, FB)                                                                                   \
  {                                                                                                          \
    bf16x8 av[MI], bv[NTAP];                                                                                 \
    _Pragma("unroll") for (int i = 0; i < MI; ++i) av[i] = tr_value(FA[i]);                                  \
    tr_run_taps<NTAP>(FB, bv);                                                                               \
    _Pragma("unroll") for (int s_ = 0; s_ < NTAP; ++s_) {                                                    \
      _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                         \
          acc[s_][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[s_], acc[s_][i], 0, 0, 0);          \
    }                                                                                                        \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
  }
  // waits until at most N LDS reads are outstanding and ties the fragments that have arrived to the wait: no MFMA of theirs may move ahead of it
#define LGKM_WAIT(N, FA, FB)                                                                                 \
  {                                                                                                          \
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N));                                                          \
    _Pragma("unroll") for (int i = 0; i < MI; ++i) tr_tie(FA[i]);                                            \
    asm volatile("" : "+v"(FB.lo), "+v"(FB.hi), "+v"(FB.ex));                                                \
  }

  // Three slabs in flight before the loop.  A slab's last fragments are in registers when its last MFMAs have yet to run: there the
  // workgroup waits for the next slab and gives the stage to the slab after the next two, so that a load has two slabs' time.  (Waiting where the
  // slab begins gave it one: a launch of 128 <-> 256 channels over 32 images of 64 x 64 97.9 -> 95.0 us; of a training step under 1 %.)
  const bool full = __builtin_amdgcn_readfirstlane(wave) + 4 * (G::XU - 1) < G::X_UNITS;   // (loads per slab and wave: L, or one less)
  constexpr int L = G::A_PASSES + G::XU;
  auto landed = [&](int behind) {                // all loads but those of the last `behind` slabs
    if (behind >= 2) { if (full) __builtin_amdgcn_s_waitcnt(vm_imm(2 * L)); else __builtin_amdgcn_s_waitcnt(vm_imm(2 * L - 2)); }
    else if (behind == 1) { if (full) __builtin_amdgcn_s_waitcnt(vm_imm(L)); else __builtin_amdgcn_s_waitcnt(vm_imm(L - 1)); }
    else __builtin_amdgcn_s_waitcnt(vm_imm(0));
  };
  WGRAD3_DMA(0);
  if (KT > 1) WGRAD3_DMA(1);
  if (KT > 2) WGRAD3_DMA(2);
  landed(KT - 1);
  __builtin_amdgcn_s_barrier();
  wgrad3_reads<BM, SW, 0>(fa0, fb0, lds0 + a_lane, lds0 + b_lane);
#if defined(__HIP_DEVICE_COMPILE__)
#define WGRAD3_STEPS(CUR)                                                                                    \
  {                                                                                                          \
    const unsigned sa = lds0 + (unsigned)((CUR) * G::STAGE) + a_lane, sb = lds0 + (unsigned)((CUR) * G::STAGE) + b_lane; \
    wgrad3_reads<BM, SW, 1>(fa1, fb1, sa, sb);                                                               \
    LGKM_WAIT(NR, fa0, fb0)                                                                                  \
    WGRAD3_MMA(fa0, fb0)                                                                                     \
    wgrad3_reads<BM, SW, 2>(fa0, fb0, sa, sb);                                                               \
    LGKM_WAIT(NR, fa1, fb1)                                                                                  \
    WGRAD3_MMA(fa1, fb1)                                                                                     \
    wgrad3_reads<BM, SW, 3>(fa1, fb1, sa, sb);                                                               \
    LGKM_WAIT(NR, fa0, fb0)                                                                                  \
    WGRAD3_MMA(fa0, fb0)                                                                                     \
    LGKM_WAIT(0, fa1, fb1)                                                                                   \
  }
  int cur = 0;
  for (int t = 0; t + 1 < KT; ++t) {
    const int nxt = cur == 2 ? 0 : cur + 1;
    WGRAD3_STEPS(cur)
    landed(t + 2 < KT ? 1 : 0);
    __builtin_amdgcn_s_barrier();
    wgrad3_reads<BM, SW, 0>(fa0, fb0, lds0 + (unsigned)(nxt * G::STAGE) + a_lane, lds0 + (unsigned)(nxt * G::STAGE) + b_lane);
    if (t + 3 < KT) WGRAD3_DMA(cur);
    WGRAD3_MMA(fa1, fb1)
    LGKM_WAIT(0, fa0, fb0)                       // (nothing is in flight where the loop turns)
    cur = nxt;
  }
  WGRAD3_STEPS(cur)
  WGRAD3_MMA(fa1, fb1)
#undef WGRAD3_STEPS
#endif
#undef WGRAD3_DMA
#undef WGRAD3_MMA
#undef LGKM_WAIT

  // partial[split][co][(r*3 + s)*Cin + ci]   (UP2: [(r*2 + v)*Cin + ci] with r = (a, b, u), K = 16 Cin)
  float* __restrict__ P = p.partial + (int64_t)split * p.Cout * p.K;
  const int col_lane = lane & 31, row_lane = (lane >> 5) * 4;
  const int ci = ci0 + wn * 32 + col_lane;
#pragma unroll
  for (int s_ = 0; s_ < NTAP; ++s_)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int co = co0 + wm * (BM / 2) + i * 32 + (e >> 2) * 8 + row_lane + (e & 3);
        P[(int64_t)co * p.K + (r * NTAP + s_) * p.Cin + ci] = acc[s_][i][e];
      }
}

// The same for the phase form of an upsampled convolution: dW[co][ci][r][s] = sum over splits and over the four output
// parities (a, b) of partial[split][co][((a, b, u_a(r)), v_b(s))][ci], u_0(r) = (r > 0), u_1(r) = (r > 1), v likewise.
__global__ __launch_bounds__(256) void k_wgrad_reduce_up2(const float* __restrict__ partial, int splits, int Cout, int Cin,
                                                          float* __restrict__ dw) {
  __shared__ float sm[4][64];
  const int64_t total = (int64_t)Cout * 9 * Cin;
  const int64_t stride = (int64_t)Cout * 16 * Cin;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  float acc = 0.0f;
  int ci = 0, tap = 0, co = 0;
  if (i < total) {
    ci = (int)(i % Cin);
    const int64_t q = i / Cin;
    tap = (int)(q % 9);
    co = (int)(q / 9);
    const int r = tap / 3, s_ = tap % 3;
    for (int sp = wave; sp < splits; sp += 4) {
      const float* src = partial + (int64_t)sp * stride + (int64_t)co * 16 * Cin + ci;
      float t = 0.0f;
#pragma unroll
      for (int ab = 0; ab < 4; ++ab) {
        const int a = ab >> 1, b = ab & 1;
        const int u = a == 0 ? (r > 0) : (r > 1), v = b == 0 ? (s_ > 0) : (s_ > 1);
        t += src[((((a << 2) | (b << 1) | u) << 1) | v) * Cin];
      }
      acc += t;
    }
  }
  sm[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && i < total) dw[((int64_t)co * Cin + ci) * 9 + tap] = (sm[0][lane] + sm[1][lane]) + (sm[2][lane] + sm[3][lane]);
}

// dW[co][ci][r][s] = sum over splits of partial[split][co][(r,s,ci)].  A workgroup owns 64
// consecutive outputs; wave v sums splits v, v + W, ... (independent loads, several in flight),
// then the waves are combined in a fixed order.  Sixteen of them where few outputs have many splits (48 x 27 outputs of 512: 6.5 -> 4.9 us).
template <int W>
__global__ __launch_bounds__(W * 64) void k_wgrad_reduce(const float* __restrict__ partial, int splits, int Cout, int Cin,
                                                         int taps, float* __restrict__ dw) {
  __shared__ float sm[W][64];
  const int64_t total = (int64_t)Cout * taps * Cin;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  float acc = 0.0f;
  if (i < total) {
    const float* src = partial + i;
#pragma unroll 8
    for (int sp = wave; sp < splits; sp += W) acc += src[(int64_t)sp * total];
  }
  sm[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && i < total) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < W; w += 4) t += (sm[w][lane] + sm[w + 1][lane]) + (sm[w + 2][lane] + sm[w + 3][lane]);
    const int ci = (int)(i % Cin);
    const int64_t q = i / Cin;
    const int tap = (int)(q % taps);
    const int co = (int)(q / taps);
    dw[((int64_t)co * Cin + ci) * taps + tap] = t;
  }
}

int launch_wgrad_reduce(const float* partial, int splits, int cout, int cin, int taps, float* dw, hipStream_t s) {
  const int64_t g = ((int64_t)cout * cin * taps + 63) / 64;
  if (g < 256 && splits >= 32) hipLaunchKernelGGL(k_wgrad_reduce<16>, dim3((unsigned)g), dim3(1024), 0, s, partial, splits, cout, cin, taps, dw);
  else hipLaunchKernelGGL(k_wgrad_reduce<4>, dim3((unsigned)g), dim3(256), 0, s, partial, splits, cout, cin, taps, dw);
  return launch_status("wgrad_reduce");
}

struct WgradPlan { int bm, bn, bk, tiles_m, tiles_n, splits, rows_per_split, row3; };   // bk = 0: generic kernel; row3: three taps per workgroup

WgradPlan plan_wgrad(int cout, int cin, int k, int64_t rows, int wc, int hc = 0, int up = 0) {
  WgradPlan w;
  w.row3 = 0;
  // an upsampled 3x3 layer in its phase form (row3 = 2): eight groups (a, b, u) of two taps over the stored image
  const int hs = hc >> 1, ws = wc >> 1;
  if (k == 3 && up == 1 && hc > 0 && !(hc & 1) && !(wc & 1) && (ws % 64 == 0 || (ws >= 8 && 64 % ws == 0)) &&
      ((int64_t)hs * ws) % 64 == 0) {
    w.row3 = 2;
    w.bm = cout % 128 == 0 ? 128 : 64;
    w.bn = 64;
    w.bk = 64;
    w.tiles_m = cout / w.bm;
    w.tiles_n = cin / 64;
    const int64_t prow = rows / 4;                       // pixels of one phase = pixels of the stored image
    const int64_t groups = (int64_t)w.tiles_m * w.tiles_n * 8;
    int64_t splits = (512 + groups - 1) / groups;
    const int64_t max_splits = (prow + 511) / 512;
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    int64_t rps = (prow + splits - 1) / splits;
    rps = (rps + 63) / 64 * 64;
    w.rows_per_split = (int)rps;
    w.splits = (int)((prow + rps - 1) / rps);
    return w;
  }
  if (k == 3 && hc > 0 && (wc % 64 == 0 || (wc >= 16 && 64 % wc == 0)) && ((int64_t)hc * wc) % 64 == 0) {
    w.row3 = 1;
    w.bm = cout % 128 == 0 ? 128 : 64;
    w.bn = 64;
    w.bk = 64;
    w.tiles_m = cout / w.bm;
    w.tiles_n = cin / 64;
    const int64_t groups = (int64_t)w.tiles_m * w.tiles_n * 3;
    int64_t splits = (512 + groups - 1) / groups;       // two workgroups per compute unit fit: one round
    const int64_t max_splits = (rows + 511) / 512;
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    int64_t rps = (rows + splits - 1) / splits;
    rps = (rps + 63) / 64 * 64;
    w.rows_per_split = (int)rps;
    w.splits = (int)((rows + rps - 1) / rps);
    return w;
  }
  w.bm = cout % 128 == 0 ? 128 : 64;
  w.bn = cin % 128 == 0 ? 128 : 64;
  if (w.bm == 64 && w.bn == 64) w.bn = 64;
  w.tiles_m = cout / w.bm;
  w.tiles_n = cin / w.bn;
  const int64_t tiles = (int64_t)w.tiles_m * w.tiles_n * k * k;
  int64_t splits = (1024 + tiles - 1) / tiles;          // about four workgroups per compute unit
  const int64_t max_splits = (rows + 511) / 512;        // at least 512 pixels per split
  if (splits > max_splits) splits = max_splits;
  if (splits < 1) splits = 1;
  // row-slab kernel: slabs of bk pixels that never straddle an image row
  w.bk = wc % 64 == 0 ? 64 : wc % 32 == 0 ? 32 : 0;
  const int gran = w.bk ? w.bk : 32;
  int64_t rps = (rows + splits - 1) / splits;
  rps = (rps + gran - 1) / gran * gran;
  w.rows_per_split = (int)rps;
  w.splits = (int)((rows + rps - 1) / rps);
  return w;
}

}  // namespace

bool wgrad_mfma_supported(const WgradArgs& a) {
  if (a.dtype != AE_BF16 || a.cin % 64 != 0 || a.cout % 64 != 0) return false;   // (binary32: launch_wgrad_chunks)
  const int64_t es = 2;
  if ((int64_t)a.n * a.hc * a.wc * a.cout * es >= 0x7FFFFFFF) return false;                    // 32-bit buffer offsets
  if ((int64_t)a.n * (a.hc >> a.up) * (a.wc >> a.up) * a.cin * es >= 0x7FFFFFFF) return false;
  const int64_t rows = (int64_t)a.n * a.hc * a.wc;
  return rows < 0x7FFFFFFF;
}

// does launch_wgrad_mfma run this layer in the phase form of an upsampled convolution (4/9 of the multiply-adds)?
bool wgrad_mfma_up_phases(const WgradArgs& a) {
  if (!wgrad_mfma_supported(a)) return false;
  return plan_wgrad(a.cout, a.cin, a.k, (int64_t)a.n * a.hc * a.wc, a.wc, a.hc, a.up).row3 == 2;
}

int64_t wgrad_mfma_workspace_floats(const WgradArgs& a) {
  const int64_t rows = (int64_t)a.n * a.hc * a.wc;
  const WgradPlan w = plan_wgrad(a.cout, a.cin, a.k, rows, a.wc, a.hc, a.up);
  return (int64_t)w.splits * a.cout * a.cin * (w.row3 == 2 ? 16 : a.k * a.k);
}

int launch_wgrad_mfma(const WgradArgs& a, float* workspace, hipStream_t s) {
  if (!wgrad_mfma_supported(a)) return fail(AE_EINVAL, "wgrad_mfma: shape not supported");
  const int64_t rows = (int64_t)a.n * a.hc * a.wc;
  const WgradPlan w = plan_wgrad(a.cout, a.cin, a.k, rows, a.wc, a.hc, a.up);
  WgradParams p;
  // a 1x1 layer that needs no split: the partial layout [co][ci] is the canonical one
  const bool direct = w.splits == 1 && a.k == 1;
  p.x = a.x; p.dy = a.dy; p.partial = direct ? a.dw_canonical : workspace;
  p.M = rows; p.Cout = a.cout; p.Cin = a.cin; p.Hc = a.hc; p.Wc = a.wc; p.ksz = a.k; p.up = a.up;
  p.tiles_m = w.tiles_m; p.tiles_n = w.tiles_n; p.rows_per_split = w.rows_per_split;
  p.K = a.k * a.k * a.cin;
  const int64_t es = (int64_t)dtype_size(a.dtype);
  p.dy_bytes = (unsigned)(rows * a.cout * es);
  p.x_bytes = (unsigned)((int64_t)a.n * (a.hc >> a.up) * (a.wc >> a.up) * a.cin * es);
  const bool pow2 = (a.hc & (a.hc - 1)) == 0 && (a.wc & (a.wc - 1)) == 0;
  p.log_w = p.log_h = 0;
  if (pow2) {
    while ((1 << p.log_w) < a.wc) ++p.log_w;
    while ((1 << p.log_h) < a.hc) ++p.log_h;
  }
  if (w.row3 == 2) {     // phase form: the kernel walks the stored image
    p.M = rows / 4; p.Hc = a.hc / 2; p.Wc = a.wc / 2; p.up = 0; p.K = 16 * a.cin;
  }
  const int64_t blocks = (int64_t)w.splits * w.tiles_m * w.tiles_n * (w.row3 == 2 ? 8 : w.row3 ? 3 : a.k * a.k);
  if (blocks > 0x7FFFFFFF) return fail(AE_EINVAL, "wgrad_mfma: grid too large");
  dim3 grid((unsigned)blocks);
#define WGRAD_LAUNCH(P2)                                                                             \
  do {                                                                                               \
    if (w.bm == 128 && w.bn == 128) hipLaunchKernelGGL((k_wgrad<128, 128, P2>), grid, dim3(256), 0, s, p); \
    else if (w.bm == 128) hipLaunchKernelGGL((k_wgrad<128, 64, P2>), grid, dim3(256), 0, s, p);      \
    else if (w.bn == 128) hipLaunchKernelGGL((k_wgrad<64, 128, P2>), grid, dim3(256), 0, s, p);      \
    else hipLaunchKernelGGL((k_wgrad<64, 64, P2>), grid, dim3(256), 0, s, p);                        \
  } while (0)
#define WGRAD_ROWS(BKV)                                                                              \
  do {                                                                                               \
    if (w.bm == 128 && w.bn == 128) hipLaunchKernelGGL((k_wgrad_rows<128, 128, BKV>), grid, dim3(256), 0, s, p); \
    else if (w.bm == 128) hipLaunchKernelGGL((k_wgrad_rows<128, 64, BKV>), grid, dim3(256), 0, s, p); \
    else if (w.bn == 128) hipLaunchKernelGGL((k_wgrad_rows<64, 128, BKV>), grid, dim3(256), 0, s, p); \
    else hipLaunchKernelGGL((k_wgrad_rows<64, 64, BKV>), grid, dim3(256), 0, s, p);                  \
  } while (0)
  if (w.row3) {
    const int sw = p.Wc < 64 ? p.Wc : 64;
#define WGRAD_ROW3(BMV, UPV)                                                                            \
  do {                                                                                                  \
    if (sw == 64) hipLaunchKernelGGL((k_wgrad_row3<BMV, 64, UPV>), grid, dim3(256), 0, s, p);           \
    else if (sw == 32) hipLaunchKernelGGL((k_wgrad_row3<BMV, 32, UPV>), grid, dim3(256), 0, s, p);      \
    else hipLaunchKernelGGL((k_wgrad_row3<BMV, 16, UPV>), grid, dim3(256), 0, s, p);                    \
  } while (0)
    if (w.row3 == 2 && sw == 8) {      // stored images of 8 x 8: the phase form only
      if (w.bm == 128) hipLaunchKernelGGL((k_wgrad_row3<128, 8, true>), grid, dim3(256), 0, s, p);
      else hipLaunchKernelGGL((k_wgrad_row3<64, 8, true>), grid, dim3(256), 0, s, p);
    }
    else if (w.row3 == 2) { if (w.bm == 128) WGRAD_ROW3(128, true); else WGRAD_ROW3(64, true); }
    else { if (w.bm == 128) WGRAD_ROW3(128, false); else WGRAD_ROW3(64, false); }
#undef WGRAD_ROW3
  }
  else if (w.bk) { if (w.bk == 64) WGRAD_ROWS(64); else WGRAD_ROWS(32); }
  else { if (pow2) WGRAD_LAUNCH(true); else WGRAD_LAUNCH(false); }
#undef WGRAD_ROWS
#undef WGRAD_LAUNCH
  AE_TRY(launch_status("wgrad_mfma"));
  if (direct) return AE_OK;
  if (w.row3 != 2) return launch_wgrad_reduce(workspace, w.splits, a.cout, a.cin, a.k * a.k, a.dw_canonical, s);
  const int64_t g = ((int64_t)a.cout * a.cin * 9 + 63) / 64;
  hipLaunchKernelGGL(k_wgrad_reduce_up2, dim3((unsigned)g), dim3(256), 0, s, workspace, w.splits, a.cout, a.cin, a.dw_canonical);
  return launch_status("wgrad_reduce");
}

// ---- any channel counts -------------------------------------------------------------------------------------------
static FastDiv fast_div(int d) {
  int l = 0;
  while ((int64_t{1} << l) < d) ++l;
  FastDiv f;
  f.mul = (uint32_t)(((uint64_t{1} << (31 + l)) + (uint64_t)d - 1) / (uint64_t)d);
  f.shift = 31 + l;
  return f;
}

// a.x and a.dy hold whole 16-byte chunks per pixel (chan_pad channels, zeros behind the layer's own)
int launch_wgrad_chunks(const WgradArgs& a, float* workspace, hipStream_t s) {
  if (!wgrad_chunks_supported(a)) return fail(AE_EINVAL, "wgrad_chunks: shape not supported");
  const WgradChunksPlan w = plan_wgrad_chunks(a);
  const int64_t rows = (int64_t)a.n * a.hc * a.wc;
  const int es = (int)dtype_size(a.dtype), epc = 16 / es;
  const bool direct = w.splits == 1 && a.k == 1;        // the partial layout [co][ci] is the canonical one
  WgradParams p = {};
  p.x = a.x; p.dy = a.dy; p.partial = direct ? a.dw_canonical : workspace;
  p.M = rows; p.Cout = a.cout; p.Cin = a.cin; p.Hc = a.hc; p.Wc = a.wc; p.ksz = a.k; p.up = a.up;
  p.tiles_m = w.tiles_m; p.tiles_n = w.tiles_n; p.rows_per_split = w.rows_per_split;
  p.K = a.k * a.k * a.cin;
  p.chunks = chan_pad(a.cin, a.dtype) / epc; p.dy_chunks = chan_pad(a.cout, a.dtype) / epc;
  p.dy_bytes = (unsigned)(rows * p.dy_chunks * 16);
  p.x_bytes = (unsigned)((int64_t)a.n * (a.hc >> a.up) * (a.wc >> a.up) * p.chunks * 16);
  p.div_w = fast_div(a.wc); p.div_h = fast_div(a.hc);
  const int64_t blocks = (int64_t)w.splits * w.tiles_m * w.tiles_n;
  if (blocks > 0x7FFFFFFF) return fail(AE_EINVAL, "wgrad_chunks: grid too large");
  const dim3 grid((unsigned)blocks);
  // (bfloat16: k_wgrad_chunks; binary32: k_wgrad_split)
#define WGRAD_CHUNKS(BMV, BNV)                                                                                     \
  do {                                                                                                             \
    if (a.dtype == AE_BF16) hipLaunchKernelGGL((k_wgrad_chunks<BMV, BNV>), grid, dim3(256), 0, s, p);              \
    else hipLaunchKernelGGL((k_wgrad_split<BMV, BNV>), grid, dim3(256), 0, s, p);                                  \
  } while (0)
  if (w.bm == 128 && w.bn == 128) WGRAD_CHUNKS(128, 128);
  else if (w.bm == 128) WGRAD_CHUNKS(128, 64);
  else if (w.bn == 128) WGRAD_CHUNKS(64, 128);
  else WGRAD_CHUNKS(64, 64);
#undef WGRAD_CHUNKS
  AE_TRY(launch_status("wgrad_chunks"));
  if (direct) return AE_OK;
  return launch_wgrad_reduce(workspace, w.splits, a.cout, a.cin, a.k * a.k, a.dw_canonical, s);
}

}  // namespace ae
