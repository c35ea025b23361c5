// ae_fused_small.hip — the whole forward pass of a SMALL-IMAGE autoencoder in three launches.
//
// A network of the shape
//     conv3+bn+relu+pool2, conv3+bn+relu+pool2, flatten, fc, pnorm, awgn, fc, reshape, up2+conv3+relu, up2+conv3+sigmoid
// on images of at most 32 x 32 pixels (the smallest workload: 64 samples of 1 x 28 x 28, 0.29 GFLOP per batch)
// is bound by the launch-to-launch latency of its ~20 layer kernels, not by any roof.  Here one workgroup owns one
// sample and keeps that sample's tensors in LDS; batch-norm with batch statistics is the only coupling between
// samples, so a launch boundary stands exactly where a layer needs the statistics of the whole batch:
//   k_small_conv1   conv 1 of the sample, its output (for the next launch) and per-sample partial statistics;
//   k_small_conv2   statistics of layer 1 finished by every workgroup for itself (fixed order, double), batch-norm +
//                   ReLU + max-pool into LDS, conv 2, its output and partial statistics;
//   k_small_tail    statistics of layer 2, batch-norm + ReLU + max-pool, flatten, fc, power normalisation, noise,
//                   fc, reshape, both upsampled convolutions, sigmoid — all in LDS, y written once.
// Arithmetic is binary32: the first three convolutions on the binary32 matrix instruction (16 pixels x 16 channels x 4 input
// channels, one wavefront per 16 pixels), whose accumulators hold one channel per lane so that the batch statistics are
// a few adds, the rest as fused multiply-adds on the vector ALUs.  Sixteen wavefronts per workgroup, and where samples leave
// compute units idle several workgroups share the pixels of one (bands: launch 3 repeats what all its pixels need, the decoder's
// layers are computed for the band's rows and those around them): what counts is the length of one workgroup's chain of loads, LDS
// reads and MFMAs.  64 samples of 28 x 28: 6 + 11 + 32 us for the three launches with one workgroup per sample, in all 51 and
// now 39; of launch 3: statistics and pooling 4, fc 5, channel 1.7, fc 6, convolutions 3.5 and 1.7 (one workgroup: 7.6 and 7).
// Definitions as in aemodel.h.  No activation is kept for a backward pass: the executor takes this path only for a
// model in inference mode.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ae_device.h"
#include "ae_internal.h"
#include "ae_philox.h"

namespace ae {
namespace {

constexpr int NT_MAX = 1024;   // threads per workgroup (launch_fused_small chooses 1024 or 512)
#define NT ((int)blockDim.x)
constexpr int COB = 16;        // output channels per accumulator block
typedef float floatx4 __attribute__((ext_vector_type(4)));

// v of the lane that a DPP control selects
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
}
// sum over the 4 lanes of a quad / the 16 lanes of a row, in every lane of it
__device__ __forceinline__ float quad_sum(float v) { v += dpp<0xB1>(v); return v + dpp<0x4E>(v); }
__device__ __forceinline__ float row_sum(float v) { v += dpp<0x128>(v); v += dpp<0x124>(v); v += dpp<0x122>(v); return v + dpp<0x121>(v); }

// sum over the workgroup of `v` (every thread contributes), result in thread 0 only; red: NT/64 floats of LDS
__device__ __forceinline__ float block_sum_to0(float v, float* red) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float t = 0.0f;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) t += red[i];
  return t;
}

// Batch-norm vectors of a layer from the per-sample partial sums (taken about the conv bias): every workgroup
// computes them for itself in double, in a fixed order — thread (g, c) adds the samples g, g + G, ... of channel c
// (independent loads, all in flight together), then the G group sums of a channel are added in index order.
// scale[c] = gamma * invstd, shift[c] = beta - mean * scale.  The first BT = 256 threads do this; tmp: 2 * BT doubles.
__device__ __forceinline__ void bn_vectors(const float* __restrict__ partial, int B, int C, double inv_rows,
                                           const float* __restrict__ bias, const float* __restrict__ gamma_beta,
                                           float* scale, float* shift, double* tmp) {
  constexpr int BT = 256;
  const int G = BT / C > 0 ? BT / C : 1;           // sample groups per channel (C <= BT)
  const int c = threadIdx.x % C, g = threadIdx.x / C;
  double s1 = 0.0, s2 = 0.0;
  if (g < G) {
#pragma unroll 8
    for (int b = g; b < B; b += G) {
      s1 += (double)partial[((int64_t)b * 2) * C + c];
      s2 += (double)partial[((int64_t)b * 2 + 1) * C + c];
    }
  }
  if ((int)threadIdx.x < BT) {
    tmp[threadIdx.x] = s1;
    tmp[BT + threadIdx.x] = s2;
  }
  __syncthreads();
  if ((int)threadIdx.x < C) {
    double t1 = 0.0, t2 = 0.0;
    for (int q = 0; q < G; ++q) { t1 += tmp[q * C + c]; t2 += tmp[BT + q * C + c]; }
    const double dm = t1 * inv_rows;
    double var = t2 * inv_rows - dm * dm;
    if (var < 0.0) var = 0.0;
    const double mean = dm + (double)bias[c];
    const double invstd = 1.0 / sqrt(var + 1e-5);
    const double sc = (double)gamma_beta[c] * invstd;
    scale[c] = (float)sc;
    shift[c] = (float)((double)gamma_beta[C + c] - mean * sc);
  }
}

// 16 output pixels x 16 channels of a 3x3 convolution (zero padding) of a planar LDS image src[cin][hs x ws] (planes `plane`
// floats apart), UP: read through a x2 nearest-neighbour upsample.  Lane l multiplies input channel c + l/16 of pixel
// `m0 + l % 16` (v_mfma_f32_16x16x4); results: channel l % 16 of pixels m0 + 4 (l/16) + 0..3.  Pixels from hi on are those of
// pixel lo (nobody stores them).  wl: [tap][cin][16].
template <bool UP>
__device__ __forceinline__ floatx4 conv3_tile(const float* src, int plane, int cin, int hs, int ws, const float* wl, int m0, int lo, int hi) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int hc = UP ? 2 * hs : hs, wc = UP ? 2 * ws : ws, whole = cin & ~3;
  const int px = m0 + (lane & 15) < hi ? m0 + (lane & 15) : lo;
  const int y = px / wc, x = px - y * wc;
  floatx4 even = {0.f, 0.f, 0.f, 0.f}, odd = {0.f, 0.f, 0.f, 0.f};   // two chains: an MFMA waits for the one before the last
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const int yy = y + t / 3 - 1, xx = x + t % 3 - 1;
    const bool ok = yy >= 0 && yy < hc && xx >= 0 && xx < wc;
    const float* sp = src + g * plane + (ok ? (UP ? (yy >> 1) * ws + (xx >> 1) : yy * ws + xx) : 0);
    const float* wp = wl + (t * cin + g) * COB + (lane & 15);
    int c = 0;                                   // this lane's channels: g, g + 4, ...
    for (; c + 32 <= whole; c += 32) {           // all reads of 32 channels ahead of their MFMAs
      float v[8], w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { v[u] = sp[(c + 4 * u) * plane]; w[u] = wp[(c + 4 * u) * COB]; }
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        even = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? v[u] : 0.0f, w[u], even, 0, 0, 0);
        odd = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? v[u + 1] : 0.0f, w[u + 1], odd, 0, 0, 0);
      }
    }
    for (; c + 8 <= whole; c += 8) {
      const float v0 = ok ? sp[c * plane] : 0.0f, v1 = ok ? sp[(c + 4) * plane] : 0.0f;
      even = __builtin_amdgcn_mfma_f32_16x16x4f32(v0, wp[c * COB], even, 0, 0, 0);
      odd = __builtin_amdgcn_mfma_f32_16x16x4f32(v1, wp[(c + 4) * COB], odd, 0, 0, 0);
    }
    if (c < whole) even = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? sp[c * plane] : 0.0f, wp[c * COB], even, 0, 0, 0);
    if (whole < cin) {                           // up to three channels more: what is not there is neither read nor multiplied
      const bool in = whole + g < cin;
      odd = __builtin_amdgcn_mfma_f32_16x16x4f32(in && ok ? sp[whole * plane] : 0.0f, in ? wp[whole * COB] : 0.0f, odd, 0, 0, 0);
    }
  }
  return even + odd;
}
// canonical conv weights W[co][ci][3][3], channels co0 .. co0 + 15 -> wl[tap][cin][16]
__device__ __forceinline__ void stage_tile_weights(const float* __restrict__ w, int cin, int co0, float* wl) {
  const int row = cin * 9;
  const float* src = w + (int64_t)co0 * row;
  for (int i = threadIdx.x; i < COB * row; i += NT) {
    const int co = i / row, r = i - co * row, ci = r / 9, t = r - ci * 9;
    wl[(t * cin + ci) * COB + co] = src[i];
  }
}
// Sum and sum of squares of a channel over the workgroup's tiles, lane l holding channel l % 16: over the four lane groups,
// then the wavefronts in order.  red: [NT / 64][2][COB]; the first 2 COB threads store.
__device__ __forceinline__ void store_channel_sums(float s1, float s2, float* red, float* __restrict__ part, int C, int co0) {
  s1 += __shfl_xor(s1, 16, 64); s1 += __shfl_xor(s1, 32, 64);
  s2 += __shfl_xor(s2, 16, 64); s2 += __shfl_xor(s2, 32, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane < COB) { red[(wave * 2) * COB + lane] = s1; red[(wave * 2 + 1) * COB + lane] = s2; }
  __syncthreads();
  if ((int)threadIdx.x < 2 * COB) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += red[w * 2 * COB + threadIdx.x];
    part[(threadIdx.x / COB) * C + co0 + threadIdx.x % COB] = t;
  }
}

// The 2x2 block of output pixels (rows 2*by, 2*by + 1, columns 2*bx, 2*bx + 1) of a 3x3 convolution behind a x2
// nearest upsample of src[cin][hs][ws]: the block's 36 taps read only the 3x3 source cells around (by, bx), which
// are loaded once per input channel, and a weight serves four pixels.  (One pixel per thread is bound
// by the LDS reads: a value and NCO weights per NCO multiply-adds.)  Each output adds its taps in the order
// (ci, r, s); this call adds the input channels ci0, ci0 + 4, ...
// wl: [ci*9 + tap][NCO].  acc[2*a + b] is pixel (2*by + a, 2*bx + b).
template <int NCO>
__device__ __forceinline__ void conv3_up_block(const float* src, int plane, const float* wl, int ci0, int cin, int hs, int ws,
                                               int by, int bx, float (&acc)[4][NCO]) {
  int off[9];
  bool ok[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int yy = by + q / 3 - 1, xx = bx + q % 3 - 1;
    ok[q] = yy >= 0 && yy < hs && xx >= 0 && xx < ws;
    off[q] = ok[q] ? yy * ws + xx : 0;
  }
  for (int ci = ci0; ci < cin; ci += 4) {
    const float* sp = src + ci * plane;
    const float* wp = wl + ci * 9 * NCO;
    float sv[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) sv[q] = ok[q] ? sp[off[q]] : 0.0f;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      float w[NCO];
      if constexpr (NCO == 4) {
        const float4 w4 = *reinterpret_cast<const float4*>(wp + t * NCO);
        w[0] = w4.x; w[1] = w4.y; w[2] = w4.z; w[3] = w4.w;
      } else {
#pragma unroll
        for (int k = 0; k < NCO; ++k) w[k] = wp[t * NCO + k];
      }
#pragma unroll
      for (int ab = 0; ab < 4; ++ab) {
        // output row 2*by + a under tap row r is upsampled row 2*by + a + r - 1, i.e. source row by + ((a + r - 1) >> 1)
        const int dy = ((ab >> 1) + t / 3 - 1) >> 1, dx = ((ab & 1) + t % 3 - 1) >> 1;
        const float v = sv[(dy + 1) * 3 + dx + 1];
#pragma unroll
        for (int k = 0; k < NCO; ++k) acc[ab][k] = fmaf(v, w[k], acc[ab][k]);
      }
    }
  }
}

// canonical conv weights W[co][ci][3][3] -> wl[(ci*9 + tap)*NCO + k] for co = co0 + k (zero beyond cout)
__device__ __forceinline__ void stage_weights(const float* __restrict__ w, int cout, int cin, int co0, int nco, float* wl) {
  for (int i = threadIdx.x; i < cin * 9 * nco; i += NT) {
    const int k = i % nco, t = i / nco;           // t = ci*9 + tap
    const int co = co0 + k;
    wl[i] = co < cout ? w[(int64_t)co * cin * 9 + t] : 0.0f;
  }
}


struct SmallArgs {
  const float* x; const float* params; float* y;
  float* raw1; float* raw2; float* part1; float* part2;
  int B, c0, h, w, c1, c2, n, cr, c3, c4;       // cr: channels after the reshape (input of the first decoder conv)
  int64_t w1, b1, bn1, w2, b2, bn2, wf1, bf1, wf2, bf2, w3, b3, w4, b4;   // offsets into params
  float sigma; uint64_t seed, first_sample;
  int bands1, bands2, bands;                      // workgroups per sample (launch 2: and block of channels) that share its pixels
  int plane2, plane_d, plane3;                    // plane strides in LDS of conv 2's input, the decoder fc's output, the last conv's input
};

// ---- launch 1: conv 1 (planar input, c0 <= 4 channels) ------------------------------------------------------------
// K = (ci, tap), four of them per MFMA
__global__ __launch_bounds__(NT_MAX) void k_small_conv1(SmallArgs a) {
  extern __shared__ float lds[];
  const int hw = a.h * a.w, K = a.c0 * 9, K4 = (K + 3) & ~3;
  float* img = lds;                               // [c0][h*w]
  float* red = img + a.c0 * hw;                   // [NT/64][2][COB]
  const int b = blockIdx.x, band = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4;
  const float* xb = a.x + (int64_t)b * a.c0 * hw;
  for (int i = threadIdx.x; i < a.c0 * hw; i += NT) img[i] = xb[i];
  for (int co0 = 0; co0 < a.c1; co0 += COB) {
    const int co = co0 + (lane & 15);
    const float bias = a.params[a.b1 + co];
    float wk[9];                                  // this lane's weights: k = 4 s + g
#pragma unroll
    for (int s = 0; s < 9; ++s) wk[s] = 4 * s + g < K ? a.params[a.w1 + (int64_t)co * K + 4 * s + g] : 0.0f;
    __syncthreads();                              // the image is there; the sums of the block before have been read
    float s1 = 0.0f, s2 = 0.0f;
    const int t_hi = (band + 1) * (hw / 16) / a.bands1;
    for (int m0 = (band * (hw / 16) / a.bands1 + wave) * 16; m0 < t_hi * 16; m0 += NT / 64 * 16) {       // (hw is a multiple of 16)
      const int px = m0 + (lane & 15), y = px / a.w, x = px - y * a.w;
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 9; ++s) {
        if (4 * s >= K4) break;
        const int k = 4 * s + g, ci = k / 9, t = k - 9 * ci, yy = y + t / 3 - 1, xx = x + t % 3 - 1;
        const bool ok = k < K && yy >= 0 && yy < a.h && xx >= 0 && xx < a.w;
        const float v = img[ok ? ci * hw + yy * a.w + xx : 0];
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? v : 0.0f, wk[s], acc, 0, 0, 0);
      }
      float* dst = a.raw1 + ((int64_t)b * hw + m0 + 4 * g) * a.c1 + co;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dst[r * a.c1] = acc[r] + bias;
        s1 += acc[r];
        s2 = fmaf(acc[r], acc[r], s2);
      }
    }
    store_channel_sums(s1, s2, red, a.part1 + ((int64_t)b * a.bands1 + band) * 2 * a.c1, a.c1, co0);
  }
}

// batch-norm + ReLU + 2x2 max-pool of a [pixels][C] conv output of one sample into a planar LDS image dst[C][hp*wp], rows lo .. hi - 1 of it
__device__ __forceinline__ void bn_relu_pool_to_lds(const float* __restrict__ raw, int wc, int lo, int hi, int C, const float* scale,
                                                    const float* shift, float* dst, int plane) {
  const int wp = wc / 2;
  for (int i = lo * wp * C + threadIdx.x; i < hi * wp * C; i += NT) {
    const int c = i % C, q = i / C;
    const int yy = q / wp, xx = q % wp;
    const float sc = scale[c], sh = shift[c];
    const float* r0 = raw + ((int64_t)(2 * yy) * wc + 2 * xx) * C + c;
    const float v0 = fmaf(r0[0], sc, sh), v1 = fmaf(r0[C], sc, sh);
    const float v2 = fmaf(r0[(int64_t)wc * C], sc, sh), v3 = fmaf(r0[(int64_t)wc * C + C], sc, sh);
    dst[c * plane + q] = fmaxf(fmaxf(fmaxf(v0, v1), fmaxf(v2, v3)), 0.0f);
  }
}

// ---- launch 2: layer-1 statistics, bn + relu + pool, conv 2 (one workgroup per sample and block of COB channels) ----
__global__ __launch_bounds__(NT_MAX) void k_small_conv2(SmallArgs a) {
  extern __shared__ float lds[];
  const int h2 = a.h / 2, w2 = a.w / 2, hw2 = h2 * w2;
  double* tmp = reinterpret_cast<double*>(lds);   // [2*256] scratch of the statistics
  float* a1 = lds + 1024;                         // [c1][plane2]
  float* wl = a1 + a.c1 * a.plane2;               // [9][c1][COB]
  float* scale = wl + a.c1 * 9 * COB;             // [c1]
  float* shift = scale + a.c1;                    // [c1]
  float* red = shift + a.c1;                      // [NT/64][2][COB]
  const int b = blockIdx.x, co0 = blockIdx.y * COB, band = blockIdx.z, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tiles = (hw2 + 15) / 16, m_lo = band * tiles / a.bands2 * 16, m_hi = min((band + 1) * tiles / a.bands2 * 16, hw2);   // pixels of the band
  stage_tile_weights(a.params + a.w2, a.c1, co0, wl);
  bn_vectors(a.part1, a.B * a.bands1, a.c1, 1.0 / ((double)a.B * a.h * a.w), a.params + a.b1, a.params + a.bn1, scale, shift, tmp);
  __syncthreads();
  bn_relu_pool_to_lds(a.raw1 + (int64_t)b * a.h * a.w * a.c1, a.w, max(m_lo / w2 - 1, 0), min((m_hi - 1) / w2 + 2, h2), a.c1, scale, shift, a1, a.plane2);
  __syncthreads();
  const int co = co0 + (lane & 15);
  const float bias = a.params[a.b2 + co];
  float s1 = 0.0f, s2 = 0.0f;
  for (int m0 = m_lo + wave * 16; m0 < m_hi; m0 += NT / 64 * 16) {
    const floatx4 acc = conv3_tile<false>(a1, a.plane2, a.c1, h2, w2, wl, m0, m_lo, m_hi);
    const int px = m0 + (lane >> 4) * 4;
    if (px < m_hi) {                              // (m_hi is a multiple of 4)
      float* dst = a.raw2 + ((int64_t)b * hw2 + px) * a.c2 + co;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dst[r * a.c2] = acc[r] + bias;
        s1 += acc[r];
        s2 = fmaf(acc[r], acc[r], s2);
      }
    }
  }
  store_channel_sums(s1, s2, red, a.part2 + ((int64_t)b * a.bands2 + band) * 2 * a.c2, a.c2, co0);
}

template <int NCO>
__device__ __forceinline__ void last_conv(const SmallArgs& a, const float* a3, const float* wl, float* __restrict__ yb, int h2, int w2, int y_lo, int y_hi) {
  const int q = threadIdx.x & 3;
  for (int blk = y_lo * w2 + (threadIdx.x >> 2); blk < y_hi * w2; blk += NT / 4) {          // (the lanes of a quad stay together)
    const int by = blk / w2, bx = blk - by * w2;
    float acc[4][NCO];
#pragma unroll
    for (int ab = 0; ab < 4; ++ab)
#pragma unroll
      for (int k = 0; k < NCO; ++k) acc[ab][k] = 0.0f;
    conv3_up_block<NCO>(a3, a.plane3, wl, q, a.c3, h2, w2, by, bx, acc);
#pragma unroll
    for (int k = 0; k < NCO; ++k) {
      float v = 0.0f;
#pragma unroll
      for (int ab = 0; ab < 4; ++ab) {
        const float t = quad_sum(acc[ab][k]);
        v = ab == q ? t : v;
      }
      if (k < a.c4) yb[(int64_t)k * a.h * a.w + (2 * by + (q >> 1)) * a.w + 2 * bx + (q & 1)] = apply_act(v + a.params[a.b4 + k], ACT_SIGMOID);
    }
  }
}

// ---- launch 3: everything from the second batch-norm to y ----------------------------------------------------------
template <int DB>                                 // outputs of the decoder's fc at a time (launch_fused_small)
__global__ __launch_bounds__(NT_MAX) void k_small_tail(SmallArgs a) {
  extern __shared__ float lds[];
  const int h2 = a.h / 2, w2 = a.w / 2, h4 = a.h / 4, w4 = a.w / 4, hw4 = h4 * w4, hw2 = h2 * w2, hw = a.h * a.w;
  const int F = a.c2 * hw4;                       // flattened encoder output
  // A workgroup has the 2x2 blocks of output pixels y_lo .. y_hi - 1 of its sample: the rows c_lo .. c_hi - 1 of the convolution before
  // and d_lo .. d_hi - 1 of the decoder fc's output are what they read.  What lies before is the same in every band.
  const int band = blockIdx.y, y_lo = band * h2 / a.bands, y_hi = (band + 1) * h2 / a.bands;
  const int c_lo = max(y_lo - 1, 0), c_hi = min(y_hi + 1, h2), d_lo = max(c_lo - 1, 0) >> 1, d_hi = (min(c_hi, h2 - 1) >> 1) + 1;
  const int n_d = (d_hi - d_lo) * w4, FD = a.cr * n_d;               // decoder fc outputs of the band: n_d pixels of every channel
  double* tmp = reinterpret_cast<double*>(lds);   // [2*256] scratch of the statistics
  float* a2 = lds + 1024;                         // [c2][hw4]   (flatten order)
  float* lat = a2 + F;                            // [n] z, then the channel output (F is a multiple of 16: read four at a time)
  float* scale = lat + a.n;                       // [c2]
  float* shift = scale + a.c2;
  float* dec = shift + a.c2;                      // [cr][plane_d]   (reshape order)
  float* a3 = dec + a.cr * a.plane_d;             // [c3][plane3]
  float* red = lds;                               // [NT/64 + 1], over the scratch of the statistics
  // weights of the decoder convs, 16-byte aligned: read four at a time.  (Rounded as an offset: a pointer made of an integer is no LDS
  // pointer to the compiler, and its flat loads tripled the time of the convolution.)
  float* wl = lds + ((a3 + a.c3 * a.plane3 - lds + 3) & ~(int64_t)3);
  const int b = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  stage_tile_weights(a.params + a.w3, a.cr, 0, wl);
  bn_vectors(a.part2, a.B * a.bands2, a.c2, 1.0 / ((double)a.B * hw2), a.params + a.b2, a.params + a.bn2, scale, shift, tmp);
  __syncthreads();
  bn_relu_pool_to_lds(a.raw2 + (int64_t)b * hw2 * a.c2, w2, 0, h4, a.c2, scale, shift, a2, hw4);
  // weights of the last conv: over the scratch of the statistics where they fit, else over those of the conv before it once it is done
  const int nco4 = a.c4 == 1 ? 1 : 4;
  const bool w4_early = a.c3 * 9 * nco4 <= 1024 - 32;
  float* wl4 = w4_early ? lds + 32 : wl;
  if (w4_early) stage_weights(a.params + a.w4, a.c4, a.c3, 0, nco4, wl4);
  __syncthreads();
  // fc to the latent: one wavefront per output row, lanes stride over the inputs
  {
    const float* wf = a.params + a.wf1;
    constexpr int RB = 4;                         // rows per wavefront at a time: 4 * RB loads in flight per lane
    const bool vec = (F & 3) == 0 && (((uintptr_t)wf | (uintptr_t)a2) & 15) == 0;   // rows in 16-byte pieces: four times the bytes in flight
    for (int o0 = wave * RB; o0 < a.n; o0 += NT / 64 * RB) {
      float acc[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) acc[r] = 0.0f;
      for (int i0 = 4 * lane; vec && i0 < F; i0 += 256 * 4) {
        float4 wv[RB][4], av[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = i0 + 256 * u;
          av[u] = i < F ? *reinterpret_cast<const float4*>(&a2[i]) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int r = 0; r < RB; ++r)
            wv[r][u] = (i < F && o0 + r < a.n) ? *reinterpret_cast<const float4*>(&wf[(int64_t)(o0 + r) * F + i]) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int r = 0; r < RB; ++r)
            acc[r] = fmaf(wv[r][u].w, av[u].w, fmaf(wv[r][u].z, av[u].z, fmaf(wv[r][u].y, av[u].y, fmaf(wv[r][u].x, av[u].x, acc[r]))));
      }
      for (int i0 = lane; !vec && i0 < F; i0 += 64 * 4) {
        float wv[RB][4], av[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = i0 + 64 * u;
          av[u] = i < F ? a2[i] : 0.0f;
#pragma unroll
          for (int r = 0; r < RB; ++r) wv[r][u] = (i < F && o0 + r < a.n) ? wf[(int64_t)(o0 + r) * F + i] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int r = 0; r < RB; ++r) acc[r] = fmaf(wv[r][u], av[u], acc[r]);
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        float t = row_sum(acc[r]);
        t += __shfl_xor(t, 16, 64);
        t += __shfl_xor(t, 32, 64);
        if (lane == 0 && o0 + r < a.n) lat[o0 + r] = t + a.params[a.bf1 + o0 + r];
      }
    }
  }
  __syncthreads();
  // power normalisation and noise (same operation order as the stand-alone channel kernel)
  {
    float ss = 0.0f;
    for (int i = threadIdx.x; i < a.n; i += NT) ss = fmaf(lat[i], lat[i], ss);
    const float tot = block_sum_to0(ss, red);
    if (threadIdx.x == 0) {
      const float ms = tot / (float)a.n;
      red[NT / 64] = ms > 0.0f ? 1.0f / sqrtf(ms) : 0.0f;
    }
    __syncthreads();
    const float sc = red[NT / 64];
    for (int q = threadIdx.x; q < (a.n + 3) / 4; q += NT) {
      float g[4];
      normal_quad(a.seed, a.first_sample + (uint64_t)b, (uint32_t)q, g);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * q + j < a.n) lat[4 * q + j] = __fadd_rn(__fmul_rn(lat[4 * q + j], sc), __fmul_rn(a.sigma, g[j]));
    }
  }
  __syncthreads();
  // decoder fc: 16 lanes per output read a row in 16-byte pieces and add up over the lanes (one thread per output is bound by
  // the vector cache, where every lane of a load touches a line of its own); one thread per output where rows have no such pieces
  {
    const float* wf = a.params + a.wf2;
    const bool vec = (a.n & 3) == 0 && (((uintptr_t)wf | (uintptr_t)lat) & 15) == 0;
    if (vec) {
      const int j0 = 4 * (threadIdx.x & 15);
      const float inv_nd = 1.0f / (float)n_d;    // (o + 1/2) / n_d rounds down to o / n_d: o < 2^14
      auto channel = [&](int o) { return (int)(((float)o + 0.5f) * inv_nd); };
      auto row_of = [&](int o) { const int c = channel(o); return c * hw4 + d_lo * w4 + o - c * n_d; };
      for (int o0 = threadIdx.x >> 4; o0 < FD; o0 += NT / 16 * DB) {
        float acc[DB];
#pragma unroll
        for (int r = 0; r < DB; ++r) acc[r] = 0.0f;
        for (int j = j0; j < a.n; j += 64) {
          const float4 l4 = *reinterpret_cast<const float4*>(lat + j);
          float4 w4[DB];
#pragma unroll
          for (int r = 0; r < DB; ++r) w4[r] = *reinterpret_cast<const float4*>(wf + (int64_t)row_of(min(o0 + r * (NT / 16), FD - 1)) * a.n + j);
#pragma unroll
          for (int r = 0; r < DB; ++r) acc[r] = fmaf(w4[r].w, l4.w, fmaf(w4[r].z, l4.z, fmaf(w4[r].y, l4.y, fmaf(w4[r].x, l4.x, acc[r]))));
        }
#pragma unroll
        for (int r = 0; r < DB; ++r) {
          const int o = o0 + r * (NT / 16);
          const float t = row_sum(acc[r]);
          const int c = channel(o), w = row_of(o);
          if ((threadIdx.x & 15) == 0 && o < FD) dec[c * a.plane_d + w - c * hw4] = t + a.params[a.bf2 + w];
        }
      }
    } else {
      for (int o1 = threadIdx.x; o1 < FD; o1 += NT) {
        const int o = o1 / n_d * hw4 + d_lo * w4 + o1 % n_d;
        const float* row = wf + (int64_t)o * a.n;
        float acc = a.params[a.bf2 + o];
#pragma unroll 16
        for (int j = 0; j < a.n; ++j) acc = fmaf(row[j], lat[j], acc);
        dec[(o / hw4) * a.plane_d + o % hw4] = acc;
      }
    }
  }
  // first decoder conv: x2 upsample of dec [cr][h4 x w4], 3x3 to c3 channels at h2 x w2, ReLU, planar into a3
  for (int co0 = 0; co0 < a.c3; co0 += COB) {
    if (co0 > 0) {                                // (the first block's weights were staged before the statistics)
      __syncthreads();
      stage_tile_weights(a.params + a.w3, a.cr, co0, wl);
    }
    __syncthreads();
    const float bias = a.params[a.b3 + co0 + (lane & 15)];
    for (int m0 = c_lo * w2 + wave * 16; m0 < c_hi * w2; m0 += NT / 64 * 16) {
      const floatx4 acc = conv3_tile<true>(dec, a.plane_d, a.cr, h4, w4, wl, m0, c_lo * w2, c_hi * w2);
      const int px = m0 + (lane >> 4) * 4;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (px + r < c_hi * w2) a3[(co0 + (lane & 15)) * a.plane3 + px + r] = fmaxf(acc[r] + bias, 0.0f);
    }
  }
  // last conv: x2 upsample of a3, 3x3 to c4 <= 4 channels at h x w, sigmoid, planar output: four lanes per 2x2 block of
  // pixels take every fourth input channel each, add up, and store a pixel each
  __syncthreads();
  if (!w4_early) {
    stage_weights(a.params + a.w4, a.c4, a.c3, 0, nco4, wl4);
    __syncthreads();
  }
  float* yb = a.y + (int64_t)b * a.c4 * hw;
  if (nco4 == 1) last_conv<1>(a, a3, wl4, yb, h2, w2, y_lo, y_hi);
  else last_conv<4>(a, a3, wl4, yb, h2, w2, y_lo, y_hi);
}

// LDS of the three launches in bytes
size_t lds1(const SmallArgs& a) { return sizeof(float) * ((size_t)a.c0 * a.h * a.w + NT_MAX / 64 * 2 * COB); }
size_t lds2(const SmallArgs& a) { return sizeof(float) * (1024 + (size_t)a.c1 * a.plane2 + (size_t)a.c1 * 9 * COB + 2 * a.c1 + NT_MAX / 64 * 2 * COB); }
size_t lds3(const SmallArgs& a) {
  const size_t wmax = (size_t)a.cr * 9 * COB > (size_t)a.c3 * 9 * 4 ? (size_t)a.cr * 9 * COB : (size_t)a.c3 * 9 * 4;
  return sizeof(float) * (1024 + (size_t)a.c2 * (a.h / 4) * (a.w / 4) + (size_t)a.cr * a.plane_d + (size_t)a.c3 * a.plane3 + a.n + 2 * a.c2 + 4 + wmax);
}
constexpr size_t kLds = 65536;
// Plane strides of 16 floats more than a multiple of the 64 banks: the four lane groups of an MFMA read four neighbouring
// planes at the same 16 pixels.  Planes without padding where a launch would not fit its LDS otherwise.
void choose_planes(SmallArgs& a) {
  auto pad = [](int n) { return (n + 47) / 64 * 64 + 16; };
  const int hw2 = (a.h / 2) * (a.w / 2), hw4 = (a.h / 4) * (a.w / 4);
  a.plane2 = pad(hw2);
  if (lds2(a) > kLds) a.plane2 = hw2;
  a.plane_d = pad(hw4); a.plane3 = pad(hw2);
  if (lds3(a) > kLds) a.plane_d = hw4;
  if (lds3(a) > kLds) a.plane3 = hw2;
}

#undef NT
}  // namespace

// Does the plan have the shape and the sizes of the three-launch path?  (binary32, batch statistics, channel
// counts that are multiples of the accumulator block, every per-sample tensor inside 64 KiB of LDS.)
bool fused_small_match(const Plan& P, FusedSmall* f) {
  if (P.dtype != AE_F32 || P.bn_mode != 0) return false;
  const std::vector<Step>& S = P.steps;
  if (S.size() != 9) return false;
  const StepKind kinds[9] = {ST_CONV, ST_CONV, ST_TRANSPOSE, ST_CONV, ST_CHANNEL, ST_CONV, ST_TRANSPOSE, ST_CONV, ST_CONV};
  for (int i = 0; i < 9; ++i)
    if (S[i].kind != kinds[i]) return false;
  auto enc = [](const Step& s) { return s.k == 3 && !s.up && s.has_bn && s.act == ACT_RELU && s.pool; };
  auto fc = [](const Step& s) { return s.k == 1 && !s.up && !s.has_bn && s.act == ACT_NONE && !s.pool && s.hin == 1 && s.win == 1; };
  auto dec = [](const Step& s, int act) { return s.k == 3 && s.up && !s.has_bn && s.act == act && !s.pool; };
  // (nine steps: the planar boundary tensors are read / written by the first / last convolution itself, either
  // through the thin kernels or because a single channel has the same layout either way)
  if (!enc(S[0]) || (S[0].thin != 1 && P.c0 != 1) || !enc(S[1]) || !fc(S[3]) || !S[4].do_pnorm || !S[4].do_awgn || !fc(S[5]) ||
      !dec(S[7], ACT_RELU) || !dec(S[8], ACT_SIGMOID) || (S[8].thin != 2 && P.cl != 1))
    return false;
  SmallArgs a{};
  a.B = P.batch; a.c0 = P.c0; a.h = P.h0; a.w = P.w0;
  a.c1 = S[0].cout; a.c2 = S[1].cout; a.n = S[3].cout; a.cr = S[7].cin; a.c3 = S[7].cout; a.c4 = S[8].cout;
  if (a.h % 4 || a.w % 4 || a.h > 32 || a.w > 32 || a.c0 > 4 || a.c4 > 4) return false;
  if (a.c1 % COB || a.c2 % COB || a.c3 % COB || a.c1 > 64 || a.c2 > 128 || a.c3 > 64 || a.n > 1024) return false;
  // the flatten and the reshape keep the (c,h,w) order of the pooled maps
  if (S[3].cin != a.c2 * (a.h / 4) * (a.w / 4) || S[5].cin != a.n || S[7].hin != a.h / 4 || S[7].win != a.w / 4 ||
      a.cr * (a.h / 4) * (a.w / 4) != S[5].cout || S[8].cin != a.c3 || S[8].hin != a.h / 2)
    return false;
  choose_planes(a);
  if (lds1(a) > kLds || lds2(a) > kLds || lds3(a) > kLds) return false;
  if ((int64_t)P.batch * 2 * (a.c1 + a.c2) > P.max_partial_floats) return false;   // the per-sample statistics live in the partial-sum buffer
  if (f) {
    f->w1 = S[0].w_off; f->b1 = S[0].b_off; f->bn1 = S[0].bn_off; f->w2 = S[1].w_off; f->b2 = S[1].b_off; f->bn2 = S[1].bn_off;
    f->wf1 = S[3].w_off; f->bf1 = S[3].b_off; f->wf2 = S[5].w_off; f->bf2 = S[5].b_off;
    f->w3 = S[7].w_off; f->b3 = S[7].b_off; f->w4 = S[8].w_off; f->b4 = S[8].b_off;
    f->c1 = a.c1; f->c2 = a.c2; f->n = a.n; f->cr = a.cr; f->c3 = a.c3; f->c4 = a.c4;
  }
  return true;
}

int launch_fused_small(const Plan& P, const FusedSmall& f, const float* params, const float* x, float* y, float* raw1,
                       float* raw2, float* partial, float sigma, uint64_t seed, uint64_t first_sample, hipStream_t s) {
  SmallArgs a{};
  a.x = x; a.params = params; a.y = y; a.raw1 = raw1; a.raw2 = raw2;
  a.part1 = partial; a.part2 = partial + (int64_t)P.batch * 2 * f.c1;
  a.B = P.batch; a.c0 = P.c0; a.h = P.h0; a.w = P.w0;
  a.c1 = f.c1; a.c2 = f.c2; a.n = f.n; a.cr = f.cr; a.c3 = f.c3; a.c4 = f.c4;
  a.w1 = f.w1; a.b1 = f.b1; a.bn1 = f.bn1; a.w2 = f.w2; a.b2 = f.b2; a.bn2 = f.bn2;
  a.wf1 = f.wf1; a.bf1 = f.bf1; a.wf2 = f.wf2; a.bf2 = f.bf2; a.w3 = f.w3; a.b3 = f.b3; a.w4 = f.w4; a.b4 = f.b4;
  a.sigma = sigma; a.seed = seed; a.first_sample = first_sample;
  choose_planes(a);
  // Sixteen wavefronts per sample while every sample has a compute unit to itself; beyond that eight, so that two workgroups
  // fit the registers of one (28 x 28, 128 / 256 / 300 / 512 samples: 43 / 65 / 118 / 127 us with sixteen, 49 / 73 / 101 / 108
  // with eight; 16 x 16: 30 / 39 / 68 / 75 and 32 / 36 / 49 / 53)
  const dim3 nt(P.batch <= 256 ? NT_MAX : NT_MAX / 2);
  // Bands: as many workgroups per sample as leave at most one per compute unit.  us in all, 28 x 28, bands of the launches 1 / 1 / 1 and as
  // chosen: 1 sample 48 -> 33, 64 50 -> 40, 128 51 -> 43; more of them than compute units lose (128 samples, 4 / 2 / 2: 56).  Two instead of
  // three: their bounds fall between rows, and two have room (85 samples of 16 x 16 / 20 x 20 / 28 x 28 / 32 x 32: one band 32 / 38 / 52 / 62, three 34 / 37 / 48 /
  // 55, two 31 / 36 / 45 / 53).
  int per = P.batch < 256 ? 256 / P.batch : 1;
  if (per == 3) per = 2;
  a.bands1 = std::min(per, 4);
  a.bands2 = std::min(std::max(per / (f.c2 / COB), 1), 4);
  a.bands = std::min(per, a.h / 4);
  if ((int64_t)P.batch * 2 * (a.bands1 * f.c1 + a.bands2 * f.c2) > P.max_partial_floats) a.bands1 = a.bands2 = 1;
  a.part2 = partial + (int64_t)P.batch * a.bands1 * 2 * f.c1;
  hipLaunchKernelGGL(k_small_conv1, dim3(P.batch, a.bands1), nt, lds1(a), s, a);
  hipLaunchKernelGGL(k_small_conv2, dim3(P.batch, f.c2 / COB, a.bands2), nt, lds2(a), s, a);
  // The decoder's fc: the loads of 6 outputs per 16 threads in flight, of 8 where one workgroup's outputs are whole passes of as many (us in all
  // with 6 / 8: 256 samples of 16 x 16 39.5 / 38.4, 32 x 32 75.0 / 73.8; others as fast or slower with 8: 20 x 20 45.4 / 45.6, 28 x 28 65.6 / 65.5,
  // 64 samples in four bands, 28 x 28, 39.9 / 41.6).
  if (a.bands == 1 && f.cr * (a.h / 4) * (a.w / 4) % (8 * (int)nt.x / 16) == 0) hipLaunchKernelGGL(k_small_tail<8>, dim3(P.batch, 1), nt, lds3(a), s, a);
  else hipLaunchKernelGGL(k_small_tail<6>, dim3(P.batch, a.bands), nt, lds3(a), s, a);
  return launch_status("fused_small");
}

}  // namespace ae
