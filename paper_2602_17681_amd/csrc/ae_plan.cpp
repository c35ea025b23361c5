// ae_plan.cpp — host-only: layer-spec parser, shape inference, fusion of spec
// tokens into executable steps, parameter-blob offsets and workspace sizing.
// No GPU call is made here, so model_describe works on a machine without a device.
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>

#include "ae_internal.h"

namespace ae {

static thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

const char* last_error() { return g_err; }

namespace {

enum TokKind { T_CONV, T_FC, T_BN, T_RELU, T_SIGMOID, T_POOL, T_UP, T_FLATTEN, T_RESHAPE, T_PNORM, T_AWGN };

struct Tok {
  TokKind kind;
  int a = 0, b = 0, c = 0;  // conv: k, cout; fc: cout; reshape: c,h,w
};

// a positive decimal integer of at most 9 digits (so it fits an int with room to spare), nothing else
bool read_int(const std::string& s, int* v) {
  if (s.empty() || s.size() > 9) return false;
  int64_t acc = 0;
  for (char ch : s) {
    if (ch < '0' || ch > '9') return false;
    acc = acc * 10 + (ch - '0');
  }
  *v = (int)acc;
  return acc > 0;
}

// "CxHxW": three such integers
bool read_dims(const std::string& s, int* c, int* h, int* w) {
  const size_t p1 = s.find('x');
  if (p1 == std::string::npos) return false;
  const size_t p2 = s.find('x', p1 + 1);
  if (p2 == std::string::npos) return false;
  return read_int(s.substr(0, p1), c) && read_int(s.substr(p1 + 1, p2 - p1 - 1), h) && read_int(s.substr(p2 + 1), w);
}

// Every tensor of a model (activations of the whole batch, weights of a layer) must stay below 2 GiB in
// binary32: the kernels index elements with 32-bit integers and address memory through 32-bit buffer ranges.
constexpr int64_t kMaxTensorElems = ((int64_t)1 << 29) - 1;
bool tensor_fits(int64_t batch, int64_t c, int64_t h, int64_t w) {
  if (c > kMaxTensorElems || h > kMaxTensorElems || w > kMaxTensorElems) return false;
  const int64_t hw = h * w;                       // < 2^58
  if (hw > kMaxTensorElems) return false;
  const int64_t chw = c * hw;                     // < 2^58
  if (chw > kMaxTensorElems) return false;
  return batch * chw <= kMaxTensorElems;          // batch < 2^31: < 2^60
}

int tokenize(const char* spec, int* c0, int* h0, int* w0, std::vector<Tok>* toks) {
  if (!spec) return fail(AE_EINVAL, "layer_spec is null");
  std::vector<std::string> parts;
  std::string cur;
  for (const char* p = spec;; ++p) {
    if (*p == ',' || *p == 0) {
      size_t a = cur.find_first_not_of(" \t\r\n");
      size_t b = cur.find_last_not_of(" \t\r\n");
      if (a == std::string::npos) return fail(AE_ESPEC, "empty token in layer spec");
      parts.push_back(cur.substr(a, b - a + 1));
      cur.clear();
      if (*p == 0) break;
    } else {
      cur.push_back(*p);
    }
  }
  if (parts.empty() || parts[0].compare(0, 3, "in:") != 0 || !read_dims(parts[0].substr(3), c0, h0, w0))
    return fail(AE_ESPEC, "layer spec must start with in:CxHxW");
  for (size_t i = 1; i < parts.size(); ++i) {
    const std::string& t = parts[i];
    Tok k;
    if (t.compare(0, 6, "conv3:") == 0 || t.compare(0, 6, "conv1:") == 0) {
      k.kind = T_CONV;
      k.a = t[4] - '0';
      if (!read_int(t.substr(6), &k.b)) return fail(AE_ESPEC, "bad channel count in '%s'", t.c_str());
    } else if (t.compare(0, 3, "fc:") == 0) {
      k.kind = T_FC;
      if (!read_int(t.substr(3), &k.b)) return fail(AE_ESPEC, "bad width in '%s'", t.c_str());
    } else if (t.compare(0, 8, "reshape:") == 0) {
      k.kind = T_RESHAPE;
      if (!read_dims(t.substr(8), &k.a, &k.b, &k.c)) return fail(AE_ESPEC, "bad shape in '%s'", t.c_str());
    } else if (t == "bn") k.kind = T_BN;
    else if (t == "relu") k.kind = T_RELU;
    else if (t == "sigmoid") k.kind = T_SIGMOID;
    else if (t == "pool2") k.kind = T_POOL;
    else if (t == "up2") k.kind = T_UP;
    else if (t == "flatten") k.kind = T_FLATTEN;
    else if (t == "pnorm") k.kind = T_PNORM;
    else if (t == "awgn") k.kind = T_AWGN;
    else return fail(AE_ESPEC, "unknown token '%s'", t.c_str());
    toks->push_back(k);
  }
  return AE_OK;
}

int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

}  // namespace

// The GEMM behind the two forms of an upsampled convolution: rows are pixels of the STORED
// (half-size) grid, 2x2 taps per phase or 4x4 taps with stride 2.
ConvArgs conv_effective(const ConvArgs& a) {
  ConvArgs e = a;
  if (a.geom == CONV_PLAIN) return e;
  e.hc = a.hc / 2; e.wc = a.wc / 2; e.up = 0;
  e.k = a.geom == CONV_UP_PHASES ? 2 : 4;
  e.geom = CONV_PLAIN;                      // (applying this twice must not halve twice)
  return e;
}

bool conv_mfma_supported(const ConvArgs& a0) {
  const ConvArgs a = conv_effective(a0);
  const int es = (int)dtype_size(a.dtype);
  if ((a.cin * es) % 64 != 0 || a.cout < 32) return false;
  const int64_t M = (int64_t)a.n * a.hc * a.wc;
  const int64_t x_bytes = a0.geom == CONV_UP_DGRAD ? (int64_t)a0.n * a0.hc * a0.wc * a.cin * es
                                                   : (int64_t)a.n * (a.hc >> a.up) * (a.wc >> a.up) * a.cin * es;
  const int64_t w_bytes = (int64_t)a.cout * a.k * a.k * a.cin * es * (a0.geom == CONV_UP_PHASES ? 4 : 1);
  if (x_bytes >= 0x7FFFFFFF || w_bytes >= 0x7FFFFFFF) return false;   // 32-bit buffer offsets
  return M * ((a.cout + 63) / 64) / 128 < 0x7FFFFFFF && M < 0x7FFFFFFF;
}

// ---- any channel counts (the chunk walk of k_igemm, k_wgrad_chunks) ----------------------------------------------
ConvChunksPlan plan_conv_chunks(const ConvArgs& a) {
  ConvChunksPlan c;
  const int epc = 16 / (int)dtype_size(a.dtype);
  const ConvArgs e = conv_effective(a);
  c.M = (int64_t)e.n * e.hc * e.wc;
  c.chunks = chan_pad(a.cin, a.dtype) / epc;
  c.KT = (e.k * e.k * c.chunks + 3) / 4;
  // Column tiles of 32 and 64 for few channels (a latent, an image), 64 where 128 would leave a whole 64 empty; 256-row
  // tiles only while they are about two per compute unit.
  c.bn = a.cout <= 32 ? 32 : ((a.cout + 63) / 64) % 2 == 1 ? 64 : 128;
  const int64_t tiles_n = (a.cout + c.bn - 1) / c.bn;
  const bool tall = c.bn == 32 || (c.bn == 64 && a.dtype == AE_BF16);
  c.bm = tall && (c.M + 255) / 256 * tiles_n >= 512 ? 256 : 128;
  // ... and 64-row ones while 128 rows would leave compute units idle (12 960 pixels, 80 channels: 102 workgroups 9.2 us, 203 7.7; with K
  // split, 612 14.4, 609 12.0).
  if (c.bn == 128 && a.dtype == AE_BF16 && (c.M + 127) / 128 * tiles_n < 256) c.bm = 64;
  c.tiles = (c.M + c.bm - 1) / c.bm * tiles_n;
  c.splits = 1;
  if (!a.partial && a.geom != CONV_UP_PHASES && c.tiles < 256 && c.KT >= 16)   // fewer than one workgroup per compute unit and a long K
    c.splits = (int)std::max<int64_t>(1, std::min<int64_t>((512 + c.tiles - 1) / c.tiles, c.KT / 4));
  return c;
}

bool conv_chunks_supported(const ConvArgs& a) {
  if (a.epi != CONV_EPI_NONE || a.tri != 0 || a.comp_mode != 0) return false;
  const int64_t es = (int64_t)dtype_size(a.dtype), cin_p = chan_pad(a.cin, a.dtype);
  const int64_t x_px = (int64_t)a.n * (a.hc >> a.up) * (a.wc >> a.up);
  const int64_t taps = a.geom != CONV_PLAIN ? 16 : a.k * a.k;
  const int64_t M = (int64_t)a.n * a.hc * a.wc;
  return x_px * cin_p * es < 0x7FFFFFFF && (int64_t)a.cout * taps * cin_p * es < 0x7FFFFFFF && M < 0x7FFFFFFF &&
         M / 128 * ((a.cout + 31) / 32) < 0xFFFFFFF;           // 32-bit buffer offsets and grids
}

int64_t conv_chunks_splitk_floats(const ConvArgs& a) {
  const ConvChunksPlan c = plan_conv_chunks(a);
  return c.splits > 1 ? (int64_t)c.splits * c.M * a.cout : 0;
}

WgradChunksPlan plan_wgrad_chunks(const WgradArgs& a) {
  WgradChunksPlan w;
  const int64_t rows = (int64_t)a.n * a.hc * a.wc;
  const int cols = a.k * a.k * chan_pad(a.cin, a.dtype);
  // Tiles of 64 where 128 would leave a whole 64 empty, of the columns only up to five 64s: beyond, the empty half is a sixth of the
  // tiles at most and the wider tile reads dY half as often.  3x3 weights, wide tiles against tiles of 64: 72 -> 160 channels over
  // 32,768 pixels 36 and 44 us, 120 -> 160 50 and 62; with few pixels, where the compute units are not full, 48 -> 80 over 18,432
  // 20.4 and 18.2, 48 -> 40 over 2,304 12.2 and 11; binary32 16 -> 80 over 18,432 28 and 22, 64 -> 160 over 32,768 79 and 84.
  w.bm = ((a.cout + 63) / 64) % 2 == 0 ? 128 : 64;
  w.bn = ((cols + 63) / 64) % 2 == 0 || cols > 320 ? 128 : 64;
  // Where even the most splits leave compute units without a workgroup, tiles of 64: a workgroup's time is then the launch's.
  // Binary32, 3x3, 64 -> 64 over 256 pixels 19.8 -> 15.5 us (14.7 with a tile per tap and the binary32 MFMA), 64 -> 256 26.7 -> 16.9
  // (21.0), 128 -> 128 over 1,024 27 -> 17 (53), 1x1 256 -> 256 over 4,096 28 -> 18 (50); bfloat16 80 -> 40 over 2,304 12.5 -> 11.1;
  // no difference from 256 workgroups on (256 -> 256 over 4,096 53 and 52).
  if ((int64_t)((a.cout + w.bm - 1) / w.bm) * ((cols + w.bn - 1) / w.bn) * ((rows + 255) / 256) < 256) w.bm = w.bn = 64;
  w.tiles_m = (a.cout + w.bm - 1) / w.bm;
  w.tiles_n = (cols + w.bn - 1) / w.bn;
  const int64_t tiles = (int64_t)w.tiles_m * w.tiles_n;
  int64_t splits = 512 / tiles;                         // two workgroups per compute unit fit: one full round and none behind it
  const int64_t max_splits = (rows + 255) / 256;        // at least 256 pixels per split
  if (splits > max_splits) splits = max_splits;
  if (splits < 1) splits = 1;
  int64_t rps = (rows + splits - 1) / splits;
  rps = (rps + 31) / 32 * 32;
  w.rows_per_split = (int)rps;
  w.splits = (int)((rows + rps - 1) / rps);
  return w;
}

bool wgrad_chunks_supported(const WgradArgs& a) {
  const int64_t es = (int64_t)dtype_size(a.dtype), rows = (int64_t)a.n * a.hc * a.wc;
  const int64_t cin_p = chan_pad(a.cin, a.dtype), cout_p = chan_pad(a.cout, a.dtype);
  if (rows * cout_p * es >= 0x7FFFFFFF || (int64_t)a.n * (a.hc >> a.up) * (a.wc >> a.up) * cin_p * es >= 0x7FFFFFFF) return false;
  return rows < 0x7FFFFFFF - 64 && (int64_t)a.k * a.k * cin_p < 0x3FFFFFFF;
}

int64_t wgrad_chunks_workspace_floats(const WgradArgs& a) {
  return (int64_t)plan_wgrad_chunks(a).splits * a.cout * a.cin * a.k * a.k;
}

namespace {
// A layer whose channel counts the tiled matrix-core kernels do not take runs on the kernel for any channel counts,
// except for small 1x1 layers, whose few launches are their time: the direct kernel needs no padded input and, in
// binary32, no packed weights.  Measured on two such layers forward, direct against chunks: 100 -> 50 -> 100 channels x 64
// rows 19.5 against 33.4 us, 1 -> 8 -> 1 x 32768 rows 15.5 against 18.9; on the other side 16 -> 12 -> 16 x 32768 rows 28.4
// against 20.4, 24 -> 20 -> 24 x 32768 rows 63 against 22, 1000 -> 10 -> 1000 x 32 rows 117 against 25 (a thread of the
// direct kernel walks K alone, so a long K is slow at any size).  3x3 layers gain from 4 x 4 images on (8 -> 8 channels:
// 24.6 against 21.4 us).
bool conv_chunks_worthwhile(const ConvArgs& a) {
  return a.k != 1 || a.cin > 128 || (int64_t)a.n * a.hc * a.wc * a.cin * a.cout > (1 << 21);
}
// (a small weight gradient over a handful of pixels: the direct kernel's serial walk over them is shorter than a slab's way
// through LDS, and nothing is padded: 100 -> 50 -> 100 channels x 1 row, forward and backward, 48 against 53 us; 16 rows of
// 48 -> 80 -> 48 channels 69 against 57, 64 rows of 100 -> 50 -> 100 channels 114 against 63.  Its threads divide 64-bit indices
// for every product, so a large one is slow at any number of rows; backward pass of c -> c -> c channels in binary32, direct
// against chunks: 1024 x 1 row 91 and 94 us, 2048 x 1 row 111 and 97, 1024 x 8 105 and 92, 4096 x 8 673 and 160)
bool wgrad_chunks_worthwhile(const WgradArgs& a) {
  const int64_t rows = (int64_t)a.n * a.hc * a.wc;
  return rows > 8 || rows * a.cout * a.cin * a.k * a.k > (1 << 20);
}
ConvArgs chunks_form(ConvArgs a, int geom) {
  if (geom == CONV_UP_PHASES) a.up = 1;
  a.geom = geom;
  return a;
}
int64_t wgrad_floats(const Step& st, const WgradArgs& wa) {
  return wgrad_mfma_supported(wa) ? wgrad_mfma_workspace_floats(wa)
         : st.chunks_w ? wgrad_chunks_workspace_floats(wa) : wgrad_direct_workspace_floats(wa);
}
}  // namespace

int build_plan(const char* spec, int batch, int dtype, int bn_mode, Plan* plan) {
  if (batch <= 0) return fail(AE_EINVAL, "batch must be positive");
  if (dtype != AE_F32 && dtype != AE_BF16) return fail(AE_EINVAL, "dtype must be AE_F32 or AE_BF16");
  if (bn_mode != 0 && bn_mode != 1) return fail(AE_EINVAL, "bn_mode must be 0 or 1");
  std::vector<Tok> toks;
  int c, h, w;
  AE_TRY(tokenize(spec, &c, &h, &w, &toks));
  if (toks.empty()) return fail(AE_ESPEC, "layer spec has no layers");
  plan->batch = batch; plan->dtype = dtype; plan->bn_mode = bn_mode;
  if (!tensor_fits(batch, c, h, w)) return fail(AE_ESHAPE, "the input tensor of the batch exceeds 2 GiB");
  plan->c0 = c; plan->h0 = h; plan->w0 = w;
  plan->steps.clear();
  int64_t off = 0;
  const int64_t B = batch;

  auto add_transpose = [&](int rows, int cols, int last_token, int oc, int oh, int ow) {
    Step st;
    st.kind = ST_TRANSPOSE;
    st.last_token = last_token;
    st.cin = c; st.hin = h; st.win = w;
    st.cout = oc; st.hout = oh; st.wout = ow;
    st.t_rows = rows; st.t_cols = cols;
    plan->steps.push_back(st);
  };

  // boundary NCHW -> stored NHWC
  if (c > 1 && h * w > 1) add_transpose(c, h * w, -1, c, h, w);

  bool seen_param_step = false;
  size_t i = 0;
  while (i < toks.size()) {
    const Tok& t = toks[i];
    if (t.kind == T_UP || t.kind == T_CONV || t.kind == T_FC) {
      Step st;
      st.kind = ST_CONV;
      st.cin = c; st.hin = h; st.win = w;
      size_t j = i;
      if (t.kind == T_UP) {
        st.up = 1;
        ++j;
        if (j >= toks.size() || toks[j].kind != T_CONV)
          return fail(AE_ESPEC, "up2 must be followed by conv1/conv3");
      }
      const Tok& cv = toks[j];
      if (cv.kind == T_FC) {
        if (h != 1 || w != 1) return fail(AE_ESHAPE, "fc needs a flattened input (use flatten first)");
        st.k = 1;
      } else {
        if (cv.a != 1 && cv.a != 3) return fail(AE_ESPEC, "only conv1 and conv3 exist");
        st.k = cv.a;
      }
      st.cout = cv.b;
      if (!tensor_fits(batch, std::max(st.cin, st.cout), (int64_t)h << st.up, (int64_t)w << st.up) ||
          !tensor_fits(1, st.cout, st.cin, st.k * st.k))
        return fail(AE_ESHAPE, "token %d: an activation or weight tensor of this layer exceeds 2 GiB", (int)j);
      st.hc = h << st.up; st.wc = w << st.up;
      st.w_off = off;
      off += (int64_t)st.cout * st.cin * st.k * st.k;
      st.b_off = off;
      off += st.cout;
      ++j;
      if (j < toks.size() && toks[j].kind == T_BN) {
        st.has_bn = 1;
        st.bn_off = off;
        off += (int64_t)(bn_mode == 1 ? 4 : 2) * st.cout;
        ++j;
      }
      if (j < toks.size() && (toks[j].kind == T_RELU || toks[j].kind == T_SIGMOID)) {
        st.act = toks[j].kind == T_RELU ? ACT_RELU : ACT_SIGMOID;
        ++j;
      }
      if (j < toks.size() && toks[j].kind == T_POOL) {
        if ((st.hc & 1) || (st.wc & 1)) return fail(AE_ESHAPE, "pool2 needs even height and width");
        st.pool = 1;
        ++j;
      }
      st.hout = st.hc >> st.pool; st.wout = st.wc >> st.pool;
      st.last_token = (int)j - 1;
      st.needs_dx = seen_param_step;
      seen_param_step = true;
      c = st.cout; h = st.hout; w = st.wout;
      plan->steps.push_back(st);
      i = j;
    } else if (t.kind == T_FLATTEN) {
      if (c > 1 && h * w > 1) add_transpose(h * w, c, (int)i, c * h * w, 1, 1);
      else if (!plan->steps.empty()) plan->steps.back().last_token = (int)i;
      c = c * h * w; h = 1; w = 1;
      ++i;
    } else if (t.kind == T_RESHAPE) {
      if (h != 1 || w != 1) return fail(AE_ESPEC, "reshape needs a flattened input");
      if (!tensor_fits(batch, t.a, t.b, t.c) || (int64_t)t.a * t.b * t.c != (int64_t)c)
        return fail(AE_ESHAPE, "reshape changes the element count");
      if (t.a > 1 && t.b * t.c > 1) add_transpose(t.a, t.b * t.c, (int)i, t.a, t.b, t.c);
      else if (!plan->steps.empty()) plan->steps.back().last_token = (int)i;
      c = t.a; h = t.b; w = t.c;
      ++i;
    } else if (t.kind == T_PNORM || t.kind == T_AWGN) {
      Step st;
      st.kind = ST_CHANNEL;
      st.cin = st.cout = c; st.hin = st.hout = h; st.win = st.wout = w;
      size_t j = i;
      if (toks[j].kind == T_PNORM) { st.do_pnorm = 1; ++j; }
      if (j < toks.size() && toks[j].kind == T_AWGN) { st.do_awgn = 1; ++j; }
      st.last_token = (int)j - 1;
      plan->latent_n = (int64_t)c * h * w;
      plan->steps.push_back(st);
      i = j;
    } else {
      return fail(AE_ESPEC, "token %d (bn/relu/sigmoid/pool2) must follow a conv or fc", (int)i);
    }
  }
  if (plan->steps.empty()) return fail(AE_ESPEC, "layer spec has no layers");
  plan->cl = c; plan->hl = h; plan->wl = w;
  // stored NHWC -> boundary NCHW
  if (c > 1 && h * w > 1) add_transpose(h * w, c, (int)toks.size() - 1, c, h, w);
  plan->n_params = off;

  // ---- thin first / last layer: the planar boundary tensor is read / written by the conv itself
  {
    std::vector<Step>& S = plan->steps;
    int fc = -1, lc = -1;
    for (size_t q = 0; q < S.size(); ++q)
      if (S[q].kind == ST_CONV) { if (fc < 0) fc = (int)q; lc = (int)q; }
    if (fc >= 0 && (fc == 0 || (fc == 1 && S[0].kind == ST_TRANSPOSE && S[0].last_token == -1))) {
      Step& st = S[fc];
      // (the thin kernels write no binary32 copy of a sigmoid output, which the backward pass of a bfloat16 model reads)
      const bool needs_aux = dtype == AE_BF16 && st.act == ACT_SIGMOID && !st.has_bn && !st.pool;
      if (st.cin <= 4 && !needs_aux && thin_in_supported(st.cin, st.cout, st.k, st.up)) {
        st.thin = 1;
        if (fc == 1) { S.erase(S.begin()); --lc; }
      }
    }
    if (lc >= 0) {
      const bool tail_ok = lc == (int)S.size() - 1 || (lc == (int)S.size() - 2 && S.back().kind == ST_TRANSPOSE);
      Step& st = S[lc];
      if (tail_ok && st.thin == 0 && !st.has_bn && !st.pool && st.cout <= 4 && thin_out_supported(st.cout, st.cin, st.k, dtype) &&
          thin_in_supported(st.cout, st.cin, st.k, 0)) {
        st.thin = 2;
        st.out_planar = true;
        if (lc == (int)S.size() - 2) { st.last_token = S.back().last_token; S.pop_back(); }
      }
    }
  }

  // ---- workspace layout ---------------------------------------------------
  const int64_t es = (int64_t)dtype_size(dtype);
  int64_t total = 0;
  auto take = [&](int64_t bytes) {
    int64_t at = total;
    total += align_up(bytes > 0 ? bytes : 4, 256);
    return at;
  };
  plan->max_act_elems = B * plan->c0 * plan->h0 * plan->w0;
  plan->max_raw_elems = plan->max_full_elems = plan->max_partial_floats = plan->max_wgrad_floats = plan->max_splitk_floats = 0;
  plan->max_wgrad_inorder_floats = plan->max_dypad_bytes = 0;
  for (Step& st : plan->steps) {
    int64_t out_elems = B * st.cout * st.hout * st.wout;
    int64_t in_elems = B * st.cin * st.hin * st.win;
    plan->max_act_elems = std::max(plan->max_act_elems, std::max(out_elems, in_elems));
    st.off_out = take(out_elems * es);
    if (st.kind == ST_CONV) {
      int64_t rows = B * st.hc * st.wc;
      int64_t raw_elems = rows * st.cout;
      plan->max_raw_elems = std::max(plan->max_raw_elems, raw_elems);
      if (st.has_bn || st.pool) st.off_raw = take(raw_elems * es);
      else if (st.act == ACT_SIGMOID && dtype == AE_BF16) st.off_aux = take(raw_elems * 4);
      plan->max_full_elems = std::max(plan->max_full_elems, rows * st.cin);
      const int cin_p = chan_pad(st.cin, dtype), cout_p = chan_pad(st.cout, dtype);
      // (both packings; the matrix-core kernels for any channel counts read whole 16-byte chunks per tap)
      int64_t wel = std::max((int64_t)st.cout * cin_p, (int64_t)st.cin * cout_p) * st.k * st.k;
      // thin layers keep their weights repacked as MFMA operand rows of the wide side
      // (the summed-weight forms of an upsampled 3x3 conv hold 16 taps instead of 9)
      const int64_t wpk = (st.up && st.k == 3 ? wel / 9 * 16 : wel) * es;
      st.off_wpack = take(std::max(wpk, st.thin == 1 ? thin_wfrag_bytes(st.cout)
                                        : st.thin == 2 ? thin_out_wz_bytes(st.cout, st.cin) : (int64_t)0));
      st.off_wpack_d = take(std::max(wpk, st.thin == 2 ? thin_wfrag_bytes(st.cin) : (int64_t)0));
      if (st.has_bn) st.off_bn = take(6 * (int64_t)st.cout * 4);
      int64_t blocks = std::max<int64_t>((rows + 63) / 64, reduce_blocks_bound(rows));  // finest partial-sum granularity
      if (st.thin == 1) blocks = std::max<int64_t>(blocks, thin_in_mfma_blocks(batch, st.hc, st.wc));
      plan->max_partial_floats = std::max(plan->max_partial_floats, blocks * 2 * std::max(st.cout, st.cin));
      WgradArgs wa;
      wa.x = wa.dy = nullptr; wa.dw_canonical = nullptr;
      wa.n = batch; wa.hc = st.hc; wa.wc = st.wc; wa.cin = st.cin; wa.cout = st.cout; wa.k = st.k; wa.up = st.up;
      wa.dtype = dtype;
      if (st.thin == 0) {
        // split-K scratch of the forward conv and of the conv that yields the input gradient
        ConvArgs ca;
        ca.x = ca.w = nullptr; ca.bias = nullptr; ca.y = nullptr; ca.partial = nullptr; ca.y_aux = nullptr;
        ca.n = batch; ca.hc = st.hc; ca.wc = st.wc; ca.cin = st.cin; ca.cout = st.cout; ca.k = st.k; ca.up = st.up;
        ca.act = ACT_NONE; ca.dtype = dtype;
        st.chunks = !conv_mfma_supported(ca) && conv_chunks_worthwhile(ca) && conv_chunks_supported(chunks_form(ca, st.up && st.k == 3 ? CONV_UP_PHASES : CONV_PLAIN));
        if (st.chunks && !st.has_bn)
          plan->max_splitk_floats = std::max(plan->max_splitk_floats, conv_chunks_splitk_floats(chunks_form(ca, st.up && st.k == 3 ? CONV_UP_PHASES : CONV_PLAIN)));
        if (!st.has_bn) plan->max_splitk_floats = std::max(plan->max_splitk_floats, conv_mfma_splitk_floats(ca));
        ca.cin = st.cout; ca.cout = st.cin; ca.up = 0;
        plan->max_splitk_floats = std::max(plan->max_splitk_floats, conv_mfma_splitk_floats(ca));
        if (st.up && conv_up_dgrad_usable(ca)) {
          ca.geom = CONV_UP_DGRAD;
          plan->max_splitk_floats = std::max(plan->max_splitk_floats, conv_mfma_splitk_floats(ca));
        }
        if (st.needs_dx) {
          ca.geom = CONV_PLAIN;
          const ConvArgs cd = chunks_form(ca, st.up && st.k == 3 ? CONV_UP_DGRAD : CONV_PLAIN);
          st.chunks_d = !conv_mfma_supported(ca) && conv_chunks_worthwhile(ca) && conv_chunks_supported(cd);
          if (st.chunks_d) plan->max_splitk_floats = std::max(plan->max_splitk_floats, conv_chunks_splitk_floats(cd));
        }
        st.chunks_w = !wgrad_mfma_supported(wa) && wgrad_chunks_worthwhile(wa) && wgrad_chunks_supported(wa);
        // (the caller's own x and dy may lie anywhere: copied into whole aligned chunks if need be, see chunk_copy)
        // (noise alone hands its incoming gradient on: dy may reach a layer that is not the last)
        const bool reads_x = &st == &plan->steps[0], reads_dy = !st.has_bn && !st.pool && st.act == ACT_NONE;
        if ((st.chunks || st.chunks_w) && (cin_p != st.cin || reads_x)) st.off_xpad = take(in_elems / st.cin * cin_p * es);
        if ((st.chunks_d || st.chunks_w) && (cout_p != st.cout || reads_dy))
          plan->max_dypad_bytes = std::max(plan->max_dypad_bytes, rows * cout_p * es);
      }
      if (st.thin == 1) {
        plan->max_wgrad_floats = std::max(plan->max_wgrad_floats, thin_wgrad_workspace_floats(rows, st.cin, st.cout));
        if (thin_wgrad_mfma_supported(st.cin, st.cout, st.wc, dtype))
          plan->max_wgrad_floats = std::max(plan->max_wgrad_floats,
                                            thin_wgrad_mfma_workspace_floats(batch, st.hc, st.wc, st.cout));
      }
      else if (st.thin == 2) {
        plan->max_wgrad_floats = std::max(plan->max_wgrad_floats,
                                          thin_wgrad_workspace_floats(B * st.hin * st.win, st.cout, st.cin));
        if (thin_wgrad_mfma_supported(st.cout, st.cin, st.win, dtype))
          plan->max_wgrad_floats = std::max(plan->max_wgrad_floats,
                                            thin_wgrad_mfma_workspace_floats(batch, st.hin, st.win, st.cin));
      }
      else
        plan->max_wgrad_floats = std::max(plan->max_wgrad_floats, wgrad_floats(st, wa));
      // a layer without batch-norm, activation or pooling has no conv-output gradient buffer of its own: its
      // weight gradient runs in order on the caller's stream, with scratch apart from the side stream's
      if (!st.has_bn && !st.pool && st.act == ACT_NONE && st.thin == 0)
        plan->max_wgrad_inorder_floats = std::max(plan->max_wgrad_inorder_floats, wgrad_floats(st, wa));
      if (st.thin == 2)
        plan->max_partial_floats = std::max(plan->max_partial_floats,
                                            B * plane_sums_split((int64_t)st.hc * st.wc) * 2 * (int64_t)st.cout);
    }
  }
  plan->off_grad_a = take(plan->max_act_elems * es);      // gradient ping-pong
  plan->off_grad_b = take(plan->max_act_elems * es);
  plan->off_draw = take(plan->max_raw_elems * es);        // gradient at conv resolution (two buffers: consecutive
  plan->off_draw2 = take(plan->max_raw_elems * es);       // layers alternate, see the side stream of the backward pass)
  plan->off_dfull = take(plan->max_full_elems * es);      // input gradient before the 2x2 sum of an upsampled conv
  plan->off_partial = take(plan->max_partial_floats * 4);
  plan->off_wgrad = take(plan->max_wgrad_floats * 4);
  plan->off_wgrad_inorder = take(plan->max_wgrad_inorder_floats * 4);
  plan->off_splitk = take(plan->max_splitk_floats * 4);
  plan->off_dypad = take(3 * plan->max_dypad_bytes);
  plan->ws_bytes = total;
  return AE_OK;
}

}  // namespace ae
