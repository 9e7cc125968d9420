// nx_device.hpp -- the fused per-pixel routine shared by every kernel that
// evaluates the model: causal gather, masked first layer, 1x1 residual blocks,
// head, mixture parameters, quantised CDF point evaluation, channel posterior.
//
// Determinism contract: the encoder's full-image pass and the decoder's
// wavefront/raster passes call exactly these functions, so their CDFs agree
// bit for bit. Everything is FP32 with a fixed operation order: the library is
// built with -ffp-contract=off, FMAs are written out where wanted, sums over
// mixture components use one fixed tree, and the exp/log/sigmoid used here are
// this file's own (hardware exp2/log2/rcp plus explicit range reduction).
//
// Wave layout ("transposed tile"): a wave evaluates 16 pixels at once. Lane
// l = p + 16 g holds pixel p (0..15) and lane group g (0..3). The network runs
// on v_mfma_f32_16x16x4f32 with A = weights (16 output rows x 4 inputs) and
// B = activations (4 inputs x 16 pixels), so the result D (16 output rows x
// 16 pixels) leaves row 16 mt + 4 g + v of pixel p in VGPR v of lane (p, g).
// Read as a B operand, VGPR q of tile ct supplies input channel 16 ct + 4 g + q
// of pixel p: layer outputs feed the next layer without any data movement.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nx_layout.hpp"
#include "nx_window.hpp"

namespace nx {

typedef float f4 __attribute__((ext_vector_type(4)));

#define NXD __device__ __forceinline__

// ------------------------------------------------------------------ math
constexpr float kLog2e = 1.44269504088896341f;
constexpr float kLn2 = 0.693147180559945309f;
// exp(x) from the hardware exp2: rounding x log2(e) costs a relative error
// of at most |x| 2^-24 ln 2 (below 5e-6 for the |x| < 100 the model meets);
// exp(-inf) = 0, exp(+big) = +inf
NXD float xexp(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }

// natural log of x > 0 from the hardware log2
NXD float xlog(float x) { return __builtin_amdgcn_logf(x) * kLn2; }

// log(1 + u) for u >= 0, with the rounding of 1 + u compensated
// (log(v) * u / (v - 1), v = fl(1 + u); Goldberg 1991, Theorem 4), the
// quotient through the hardware reciprocal; no branch
NXD float xlog1p(float u) {
  const float v = 1.0f + u;
  const float d = v - 1.0f;
  const float r = xlog(v) * (u * __builtin_amdgcn_rcpf(d));
  return d == 0.0f ? u : r;
}

// exp(x) - 1: Taylor polynomial through x^9/9! for |x| < ln2/2, else
// exp - 1 (both evaluated, one selected: no branch)
NXD float xexpm1(float x) {
  float q = 2.75573192e-06f;                  // 1/9!
  q = __builtin_fmaf(q, x, 2.48015873e-05f);  // 1/8!
  q = __builtin_fmaf(q, x, 1.98412698e-04f);  // 1/7!
  q = __builtin_fmaf(q, x, 1.38888889e-03f);  // 1/6!
  q = __builtin_fmaf(q, x, 8.33333333e-03f);  // 1/5!
  q = __builtin_fmaf(q, x, 4.16666667e-02f);  // 1/4!
  q = __builtin_fmaf(q, x, 1.66666667e-01f);  // 1/3!
  q = __builtin_fmaf(q, x, 0.5f);             // 1/2!
  const float taylor = __builtin_fmaf(x * x, q, x);
  const float direct = xexp(x) - 1.0f;
  return __builtin_fabsf(x) < 0.34657359f ? taylor : direct;
}

NXD float xtanh(float x) {
  const float e = xexpm1(-2.0f * __builtin_fabsf(x));  // in (-1, 0]
  const float t = -e * __builtin_amdgcn_rcpf(e + 2.0f);
  return __builtin_copysignf(t, x);
}

// The larger of a and b, the other one where one is NaN (as fmaxf): their
// median with infinity (a value the compiler does not see: it would make it a
// maximum, prefaced with a quieting v_max of each operand that comes from a
// lane exchange, a load or a matrix instruction; about 30 of the 1,250 vector
// instructions of a tile of the pass: 64 images of 64 to 320 wide, model C,
// encoded in 942 -> 929 us, their code lengths, model B, in 1.36 -> 1.347 ms).
NXD float xmax(float a, float b) {
  float inf = INFINITY;
  asm("" : "+s"(inf));
  return __builtin_amdgcn_fmed3f(a, b, inf);
}

// ELU with exp(x) - 1 from the hardware exp2 for x <= 0: the rounding of
// x log2(e) costs a relative error of at most |x| 2^-24 ln2 in exp(x), i.e.
// an absolute error below 3e-8 in the activation. 1 - exp(x), clamped to
// [0, 1] by the subtraction's output modifier, is 0 for x > 0 and its negative
// is the activation for x <= 0, where exp(x) - 1 >= x; so the larger of x and
// that is the activation (x itself where rounding put it above, |x| < 2^-23).
// 4 instructions where min, max and their quieting took 6.
NXD float xelu(float x) {
  const float c = __builtin_amdgcn_fmed3f(1.0f - __builtin_amdgcn_exp2f(x * kLog2e), 0.0f, 1.0f);
  return xmax(x, -c);
}

// logistic sigmoid: monotone non-decreasing in z because the hardware exp2
// and reciprocal are monotone (nellox_debug_check_monotone scans every finite
// FP32 input of both on the device)
NXD float xsigmoid(float z) {
  float e = __builtin_amdgcn_exp2f(-z * kLog2e);
  return __builtin_amdgcn_rcpf(1.0f + e);
}

// log sigmoid(z) = min(z, 0) - log1p(exp(-|z|))
NXD float xlogsigmoid(float z) {
  return fminf(z, 0.0f) - xlog1p(xexp(-__builtin_fabsf(z)));
}

// normalised pixel value v/127.5 - 1 (exact numerator, rounded reciprocal)
NXD float normalise(int v) { return (float)(2 * v - 255) * (1.0f / 255.0f); }

// lower edge of bin k (1..255): (2k - 256)/255
NXD float bin_edge(int k) { return (float)(2 * k - 256) * (1.0f / 255.0f); }

// ------------------------------------------------------------------ lane group reductions
// A pixel's mixture is spread over its four lanes p + 16 g; these combine one
// value per lane group with a fixed tree (v0 + v1) + (v2 + v3). The exchanges
// use the gfx950 row swaps (VALU, no LDS round trip): permlane16_swap of a
// value with itself leaves every lane holding its own value and that of its
// partner row (0<->1, 2<->3), permlane32_swap that of its partner half (rows
// 0,1 <-> 2,3); the pair is combined in either order, and IEEE addition and
// max are commutative, so every lane of the pixel obtains the same bits.
NXD float grp_sum(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float s = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const uint32_t w = __float_as_uint(s);
  const auto q = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
NXD float grp_max(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float s = xmax(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const uint32_t w = __float_as_uint(s);
  const auto q = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return xmax(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
// ------------------------------------------------------------------ gather
// Causal context of pixel (i, j) of a lane (a rect of Hl x Wl pixels at (y0, x0)
// of an image with row length W): input index k = 3 tap + ch over the taps in
// raster order (h rows of 2h+1, then h to the left in row i); lane group g
// gathers k = 4 kc + g for K-chunk kc. Outside the lane reads as 0.
// A lane's tap offsets are packed, one byte per K-chunk (dy | dx << 2 | ch << 5),
// into TapCodes once; unpacking them per pixel keeps them out of the register
// budget of the persistent loops.
template <int H_>
struct TapCodes {
  static constexpr int NW = (conv_chunks(H_) + 3) / 4;
  uint32_t w[NW];
  NXD void init(int g) {
    constexpr int K = 2 * H_ + 1;
#pragma unroll
    for (int t = 0; t < NW; ++t) w[t] = 0;
#pragma unroll
    for (int kc = 0; kc < conv_chunks(H_); ++kc) {
      const int k = 4 * kc + g;
      const int tap = k / 3, ch = k - 3 * (k / 3);
      const int dy = tap < H_ * K ? tap / K : H_;
      const int dx = tap < H_ * K ? tap - K * (tap / K) : tap - H_ * K;
      w[kc >> 2] |= (uint32_t)(dy | (dx << 2) | (ch << 5)) << (8 * (kc & 3));
    }
  }
  // an opaque copy per use: the unpacked offsets are not hoisted out of loops
  NXD void refresh() {
#pragma unroll
    for (int t = 0; t < NW; ++t) asm volatile("" : "+v"(w[t]));
  }
};

NXD int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }

// global-memory view of a byte pointer (lets the compiler use global loads)
typedef const __attribute__((address_space(1))) uint8_t* gbytes;
NXD gbytes as_global(const uint8_t* p) { return (gbytes)p; }

// Which of a lane group's taps lie inside the lane (bit kc: the tap of
// K-chunk kc), by what is cut off around the pixel: n columns of the window
// at its left, n at its right, n rows at its top (n = 0 .. H_).
struct TapMasks {
  uint32_t cut[3][4][4];  // [left, right, top][n][lane group]
};
template <int H_>
constexpr TapMasks tap_masks() {
  TapMasks M{};
  constexpr int K = 2 * H_ + 1;
  for (int n = 0; n <= H_; ++n)
    for (int g = 0; g < 4; ++g)
      for (int kc = 0; kc < conv_chunks(H_); ++kc) {
        const int tap = (4 * kc + g) / 3;
        const int dy = tap < H_ * K ? tap / K : H_, dx = tap - K * dy;
        if (dx >= n) M.cut[0][n][g] |= 1u << kc;
        if (dx <= 2 * H_ - n) M.cut[1][n][g] |= 1u << kc;
        if (dy >= n) M.cut[2][n][g] |= 1u << kc;
      }
  return M;
}
template <int H_>
__device__ const TapMasks tap_masks_of = tap_masks<H_>();

// Every tap is loaded from a position clamped into the lane (always in
// bounds), then taps outside the lane are replaced by 0: no branch around the
// loads, so all of them are in flight together.
template <int H_>
NXD void gather_clamped(float (&ctx)[conv_chunks(H_)], const TapCodes<H_>& tc, const uint8_t* img, int W, int y0,
                        int x0, int Hl, int Wl, int i, int j) {
  const gbytes gimg = as_global(img);
  uint32_t raw[conv_chunks(H_)];
#pragma unroll
  for (int kc = 0; kc < conv_chunks(H_); ++kc) {
    const uint32_t code = (tc.w[kc >> 2] >> (8 * (kc & 3))) & 0xffu;
    const int dy = (int)(code & 3u), dx = (int)((code >> 2) & 7u), ch = (int)(code >> 5);
    const int y = min(max(i - H_ + dy, 0), Hl - 1), x = min(max(j - H_ + dx, 0), Wl - 1);
    raw[kc] = gimg[((int64_t)(y0 + y) * W + (x0 + x)) * 3 + ch];
  }
#pragma unroll
  for (int kc = 0; kc < conv_chunks(H_); ++kc) {
    const uint32_t code = (tc.w[kc >> 2] >> (8 * (kc & 3))) & 0xffu;
    const int dy = (int)(code & 3u), dx = (int)((code >> 2) & 7u);
    const int y = i - H_ + dy, x = j - H_ + dx;
    // inside the lane, as a bit mask (no short-circuit, no branch)
    const int ok = -(int)(((unsigned)y < (unsigned)Hl) & ((unsigned)x < (unsigned)Wl));
    // normalise() of the tap, with the numerator masked: padding is exactly 0
    const int num = (2 * (int)raw[kc] - 255) & ok;
    ctx[kc] = (float)num * (1.0f / 255.0f);
  }
}

// The same contexts with an address per row of the window instead of one per
// tap. The bytes of a window row are contiguous and are the inputs k = R dy
// .. R dy + R - 1 in order (R = 3 (2 H_ + 1)), so the tap of K-chunk kc sits
// at the lane's row address plus a constant (the instruction's offset); a
// chunk that straddles two rows picks one of two addresses by lane group.
// Bytes outside the lane but inside the image are read and dropped (rows
// above the image: row 0 is read). In an image of at least H_ columns the
// only window positions outside its memory are those left of its first row
// and, with one row, right of it; a wave with such a pixel takes the clamped
// form. ytop: a row of the image (wave-uniform) at or above every pixel's, by
// fewer than 64 rows. The context of a pixel outside the lane (a tile's or
// group's unused rows) is that of a pixel in it. A tap costs 3 instructions here (a border pixel's 5), 28 in
// the clamped form: 504 of the about 2,200 of a tile of the full-image pass.
template <int H_>
NXD void gather(float (&ctx)[conv_chunks(H_)], const TapCodes<H_>& tc, const uint8_t* img, int W, int y0, int x0,
                int Hl, int Wl, int i, int j, int ytop) {
  constexpr int R = 3 * (2 * H_ + 1);
  const int ic = min(i, Hl - 1), jc = min(max(j, 0), Wl - 1);
  const int Y = y0 + ic, X = x0 + jc;
  if (__ballot((Y <= H_ && X < H_) || (Y == 0 && X + H_ >= W) || W < H_) != 0ull) {
    gather_clamped<H_>(ctx, tc, img, W, y0, x0, Hl, Wl, ic, jc);
    return;
  }
  const int g = (threadIdx.x >> 4) & 3;
  const int top = __builtin_amdgcn_readfirstlane(max(ytop - H_, 0));
  const gbytes base = as_global(img + (int64_t)top * W * 3);
  const uint32_t col = 3u * (uint32_t)X + (uint32_t)g;
  uint32_t row[H_ + 1];
#pragma unroll
  for (int dy = 0; dy <= H_; ++dy)
    row[dy] = __umul24((uint32_t)(max(Y - H_ + dy, 0) - top), 3u * (uint32_t)W) + col;
  uint32_t raw[conv_chunks(H_)];
#pragma unroll
  for (int kc = 0; kc < conv_chunks(H_); ++kc) {
    const int d0 = min(4 * kc / R, H_), d1 = min((4 * kc + 3) / R, H_);
    const int c0 = 4 * kc - R * d0 - 3 * H_, c1 = 4 * kc - R * d1 - 3 * H_;
    if (d0 == d1)
      raw[kc] = (base + c0)[row[d0]];
    else
      raw[kc] = (base + c1)[4 * kc + g >= R * d1 ? row[d1] : row[d0] + (uint32_t)(c0 - c1)];
  }
  const int nl = max(H_ - jc, 0), nr = max(jc + H_ - (Wl - 1), 0), nt = max(H_ - ic, 0);
  if (__ballot((nl | nr | nt) != 0) == 0ull) {
#pragma unroll
    for (int kc = 0; kc < conv_chunks(H_); ++kc)
      ctx[kc] = __builtin_fmaf(2.0f, (float)raw[kc], -255.0f) * (1.0f / 255.0f);
  } else {
    const TapMasks& M = tap_masks_of<H_>;
    const uint32_t m = M.cut[0][min(nl, H_)][g] & M.cut[1][min(nr, H_)][g] & M.cut[2][min(nt, H_)][g];
#pragma unroll
    for (int kc = 0; kc < conv_chunks(H_); ++kc) {
      const float v = __builtin_fmaf(2.0f, (float)raw[kc], -255.0f) * (1.0f / 255.0f);
      ctx[kc] = __int_as_float(__float_as_int(v) & __builtin_amdgcn_sbfe((int)m, kc, 1));
    }
  }
}

// Context of pixel (i, t) of a lane from its sheared canvas window (Sec. 3.1,
// Algorithm 2): tap (dy, dx) of the causal kernel is row i - h + dy, sheared
// column t - h(h+2) + (h+1) dy + dx, always a column before t. The window
// holds the int16 numerators 2x - 255 with 0 off the lane, so no bounds test
// is needed and the value is the unsheared gather's, bit for bit. i must be
// a row of the lane (callers clamp inactive rows, whose contexts go unused).
// Input k is plane 3 (t - Q) + k - 3 h dy (mod 48): the four lane groups' inputs
// of a K-chunk are four planes in a row, whose first is the same for the whole
// wave; groups past plane 47 go back to 0, and a chunk that straddles two window
// rows picks one of two firsts. 3 vector instructions a tap, where finding
// each tap's own column took 13.
NXD int ring_at(const int16_t* ring, int64_t base, uint32_t at) {
  return *(const __attribute__((address_space(1))) int16_t*)(as_global((const uint8_t*)ring) + base + at);
}
template <int H_>
NXD void gather_ring(float (&ctx)[conv_chunks(H_)], const int16_t* ring, int rows, int t, int i) {
  constexpr int Q = H_ * (H_ + 2), R = 3 * (2 * H_ + 1), PLANES = 3 * RING_COLS;
  const int g = (threadIdx.x >> 4) & 3;
  const int s = 3 * ((t - Q) & (RING_COLS - 1));
  // bytes; a place that isn't wrapped is the larger, over a base 48 planes low
  const uint32_t at = (uint32_t)(2 * (g * rows + i)), unwrapped = at + (uint32_t)(2 * PLANES * rows);
  int raw[conv_chunks(H_)];
#pragma unroll
  for (int kc = 0; kc < conv_chunks(H_); ++kc) {
    const int d0 = min(4 * kc / R, H_), d1 = min((4 * kc + 3) / R, H_);
    auto first = [&](int dy) {
      const int p = s + 4 * kc - 3 * H_ * dy;
      return uniform_int(p >= PLANES ? p - PLANES : p);
    };
    const int f0 = first(d0), f1 = first(d1);
    if (d0 == d1) {
      raw[kc] = ring_at(ring, 2 * ((int64_t)(f0 - PLANES) * rows + d0), g >= PLANES - f0 ? at : unwrapped);
    } else {
      const bool upper = 4 * kc + g >= R * d1;
      const int f = upper ? f1 : f0;
      const uint32_t row = (uint32_t)(upper ? 2 * (f1 * rows + d1) : 2 * (f0 * rows + d0));
      raw[kc] = ring_at(ring, 0, row + at - (g >= PLANES - f ? (uint32_t)(2 * PLANES * rows) : 0u));
    }
  }
#pragma unroll
  for (int kc = 0; kc < conv_chunks(H_); ++kc) ctx[kc] = (float)raw[kc] * (1.0f / 255.0f);
}

// ------------------------------------------------------------------ network
// The weight image is never written after it is staged in LDS, so the
// compiler would hoist every weight read out of the persistent loops and try
// to keep the whole network in registers. An offset it cannot see through
// (always 0) keeps the reads next to their MFMAs.
NXD const float* lds_weights(const float* w) {
  int zero = 0;
  asm volatile("" : "+s"(zero));
  return w + zero;
}

// One 1x1 layer: out[mt] (pre-initialised with the bias) += W in, K-chunks in
// the order (ct, q) = (0,0), (0,1), ..., (C/16-1, 3).
template <int MT_OUT, int CT_IN>
NXD void layer_mm(const float* __restrict__ w, const f4 (&in)[CT_IN], f4 (&out)[MT_OUT], int lane) {
#pragma unroll
  for (int ct = 0; ct < CT_IN; ++ct) {
    f4 wv[MT_OUT];
#pragma unroll
    for (int mt = 0; mt < MT_OUT; ++mt) wv[mt] = *(const f4*)(w + (((int64_t)mt * CT_IN + ct) * 64 + lane) * 4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int mt = 0; mt < MT_OUT; ++mt)
        out[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[mt][q], in[ct][q], out[mt], 0, 0, 0);
  }
}

template <int N>
NXD void bias_init(f4 (&a)[N], const float* __restrict__ b, int g) {
#pragma unroll
  for (int mt = 0; mt < N; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) a[mt][v] = b[16 * mt + 4 * g + v];
}

// Receives each post-activation tensor of the network (for the backward
// pass); the default discards them.
struct NoSink {
  template <int N>
  NXD void operator()(int, const f4 (&)[N]) const {}
};

// Network of a 16-pixel tile: head[7] receives the 112 (permuted) head rows.
// w points at the weight image (LDS). ctx is this lane's conv B operand.
// sink(l, u) sees the layer inputs u = elu(.) in order: l = 2b is the input of
// block b's first 1x1 layer, 2b + 1 of its second, 2 nb of the head.
template <int H_, int C_, class Sink = NoSink>
NXD void net_forward(const float* __restrict__ w, int nb, const float (&ctx)[conv_chunks(H_)], f4 (&head)[HEAD_TILES],
                     int lane, const Sink& sink = Sink()) {
  constexpr int MT = C_ / 16;
  constexpr int KC = conv_chunks(H_), KQ = conv_quads(H_);
  const WeightLayout L = weight_layout(H_, C_, 0);
  const int g = lane >> 4;
  const int64_t layer_stride = (int64_t)MT * MT * 256;
  const float* bias_conv = w + L.head + (int64_t)HEAD_TILES * MT * 256 + 2 * (int64_t)nb * layer_stride;
  const float* bias_blk = bias_conv + C_;
  const float* bias_head = bias_blk + 2 * (int64_t)nb * C_;
  const float* w_head = w + L.layer0 + 2 * (int64_t)nb * layer_stride;

  f4 a[MT];
  bias_init(a, bias_conv, g);
#pragma unroll
  for (int kq = 0; kq < KQ; ++kq) {
    f4 wv[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) wv[mt] = *(const f4*)(w + (((int64_t)mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (4 * kq + q < KC) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          a[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[mt][q], ctx[4 * kq + q], a[mt], 0, 0, 0);
      }
    }
  }
  for (int b = 0; b < nb; ++b) {
    f4 u[MT], z[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) u[mt][v] = xelu(a[mt][v]);
    sink(2 * b, u);
    bias_init(z, bias_blk + (int64_t)(2 * b) * C_, g);
    layer_mm<MT, MT>(w + L.layer0 + (int64_t)(2 * b) * layer_stride, u, z, lane);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) u[mt][v] = xelu(z[mt][v]);
    sink(2 * b + 1, u);
    bias_init(z, bias_blk + (int64_t)(2 * b + 1) * C_, g);
    layer_mm<MT, MT>(w + L.layer0 + (int64_t)(2 * b + 1) * layer_stride, u, z, lane);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) a[mt] = a[mt] + z[mt];
  }
  f4 u[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) u[mt][v] = xelu(a[mt][v]);
  sink(2 * nb, u);
  bias_init(head, bias_head, g);
  layer_mm<HEAD_TILES, MT>(w_head, u, head, lane);
}

// ------------------------------------------------------------------ network, four pixels at a time
// The network of NQ times four pixels on one wave. v_mfma_f32_4x4x1f32 adds 16
// outer products (blocks) of 4 x 4; with the activations as its A operand, one
// block's four pixels broadcast to all (cbsz 4, block abid), and the weights
// as B, it is one input k of 64 outputs: lane l has output l, register v pixel
// v, and A's block abid has input k of pixel r in lane 4 abid + r. Inputs are
// added one by one in the order of the 16x16x4 form, which rounds the same
// (each is a chain of fused multiply-adds). A layer's outputs become the next
// one's A operand by a 4 x 4 transpose within each four lanes. (C < 64: the
// lanes past C repeat the others.)
// It does the work of its pixels alone: net_forward's tile takes 32 cycles an
// instruction for 16 pixels, this 8 for four, or 12.5 where the wave is alone
// on its SIMD and NQ is 1 (each waits for the last). Used where a group has few
// pixels, and by teams, whose waves take four pixels each: split by output
// tiles instead, a team's layers cost six exchanges through LDS a group, 600
// cycles each (model B's network 7.3 thousand cycles a group so, about 6 as
// here; one 1024 x 1024 image with a stream per row, with the link wave:
// 34.6 -> 29.9 ms, 28.6 now).
constexpr int quad_inputs(int h) { return (4 * conv_chunks(h) + 15) / 16; }
constexpr int HB_STRIDE = 132;  // floats per pixel of a head table
template <int A>
NXD f4 quad_mfma(float act, float w, f4 d) { return __builtin_amdgcn_mfma_f32_4x4x1f32(act, w, d, 4, A, 0); }

template <int CTRL>
NXD float quad_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// x[j] of lane 4 a + r = u[r] of lane 4 a + j
NXD f4 quad_transpose(const f4& u, int lane) {
  const bool o0 = lane & 1, o1 = lane & 2;
  // (all lanes exchange, then each picks: no branch around an exchange)
  f4 e, y, x;
#pragma unroll
  for (int c = 0; c < 4; ++c) e[c] = quad_dpp<0xB1>(u[c ^ 1]);
#pragma unroll
  for (int c = 0; c < 4; ++c) y[c] = o0 == ((c & 1) != 0) ? u[c] : e[c];
#pragma unroll
  for (int c = 0; c < 4; ++c) e[c] = quad_dpp<0x4E>(y[c ^ 2]);
#pragma unroll
  for (int c = 0; c < 4; ++c) x[c] = o1 == ((c & 2) != 0) ? y[c] : e[c];
  return x;
}
template <int NQ>
NXD void quad_act(const f4 (&a)[NQ], f4 (&x)[NQ], int lane) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    f4 u;
#pragma unroll
    for (int v = 0; v < 4; ++v) u[v] = xelu(a[q][v]);
    x[q] = quad_transpose(u, lane);
  }
}
template <int NQ>
NXD void quad_splat(f4 (&a)[NQ], float b) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) a[q] = f4{b, b, b, b};
}

// The weights of 16 inputs, N outputs a lane (rows `stride` floats apart): four
// 16-byte reads of LDS each. They are issued a chunk of 16 inputs ahead of
// their use (the barrier to scheduling keeps them there): read where they are
// used, they cost a wait of about 130 cycles in every chunk of 200.
template <int N>
struct QuadW {
  f4 v[4][N];
  NXD void load(const float* w, int stride) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int n = 0; n < N; ++n) v[g][n] = *(const f4*)(w + n * stride + 64 * g);
    __builtin_amdgcn_sched_barrier(0);
  }
};
// 16 inputs of block 4 CT's lanes on: chunk (ct, q) of the 16x16x4 form holds
// inputs 16 ct + 4 g + q, g = 0 .. 3, and their order is the order here
template <int CT, int N, int NQ, int Q = 0, int G = 0>
NXD void quad_chunk(const QuadW<N>& w, const f4 (&x)[NQ], f4 (&d)[N][NQ]) {
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int q = 0; q < NQ; ++q) d[n][q] = quad_mfma<4 * CT + G>(x[q][Q], w.v[G][n][Q], d[n][q]);
  if constexpr (G < 3) quad_chunk<CT, N, NQ, Q, G + 1>(w, x, d);
  else if constexpr (Q < 3) quad_chunk<CT, N, NQ, Q + 1, 0>(w, x, d);
}
// a layer of 16 CTS inputs; w[0] holds its first chunk, and in the end what
// `next` points at
template <int CTS, int N, int NQ, int CT = 0>
NXD void quad_layer(const float* wl, int stride, const float* next, const f4 (&x)[NQ], QuadW<N> (&w)[2],
                    f4 (&d)[N][NQ]) {
  w[(CT + 1) & 1].load(CT + 1 < CTS ? wl + (CT + 1) * 256 : next, stride);
  quad_chunk<CT, N, NQ>(w[CT & 1], x, d);
  if constexpr (CT + 1 < CTS) quad_layer<CTS, N, NQ, CT + 1>(wl, stride, next, x, w, d);
  else if constexpr (CTS & 1) w[0] = w[1];
}
// inputs 16 kq .. of the first layer (there in ascending order)
template <int H_, int KQ_, int NQ, int Q = 0, int G = 0>
NXD void quad_first_chunk(const QuadW<1>& w, const float (&cx)[NQ][quad_inputs(H_)], f4 (&d)[NQ]) {
  if constexpr (4 * KQ_ + Q < conv_chunks(H_)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) d[q] = quad_mfma<4 * Q + G>(cx[q][KQ_], w.v[G][0][Q], d[q]);
    if constexpr (G < 3) quad_first_chunk<H_, KQ_, NQ, Q, G + 1>(w, cx, d);
    else if constexpr (Q < 3) quad_first_chunk<H_, KQ_, NQ, Q + 1, 0>(w, cx, d);
  }
}
template <int H_, int NQ, int KQ_ = 0>
NXD void quad_first(const float* wl, const float* next, const float (&cx)[NQ][quad_inputs(H_)], QuadW<1> (&w)[2],
                    f4 (&d)[NQ]) {
  constexpr int KQ = conv_quads(H_), P = (KQ_ + KQ) & 1;  // the last chunk in w[1]
  w[P ^ 1].load(KQ_ + 1 < KQ ? wl + (KQ_ + 1) * 256 : next, 0);
  quad_first_chunk<H_, KQ_, NQ>(w[P], cx, d);
  if constexpr (KQ_ + 1 < KQ) quad_first<H_, NQ, KQ_ + 1>(wl, next, cx, w, d);
}

// cx[q][j]: lane 4 a + r has input 16 j + a of pixel 4 q + r. Head row R of
// pixel P goes to hb[P HB_STRIDE + R], readable by the wave on return.
template <int H_, int C_, int NQ>
NXD void net_quad(const float* __restrict__ w, int nb, const float (&cx)[NQ][quad_inputs(H_)], float* hb, int lane) {
  constexpr int MT = C_ / 16;
  const WeightLayout L = weight_layout(H_, C_, 0);
  const int l = lane & (C_ - 1), r16 = lane & 15;
  const int layer_stride = MT * MT * 256;
  const float* bias_conv = w + L.head + HEAD_TILES * MT * 256 + 2 * nb * layer_stride;
  const float* bias_head = bias_conv + C_ + 2 * nb * C_;
  const float* wl = w + L.layer0 + ((l >> 4) * MT * 64 + r16) * 4;
  const float* bl = bias_conv + C_ + l;
  const float* wc = w + ((l >> 4) * conv_quads(H_) * 64 + r16) * 4;
  QuadW<1> q[2];
  q[conv_quads(H_) & 1].load(wc, 0);
  f4 a[NQ], x[NQ], z[1][NQ];
  quad_splat(a, bias_conv[l]);
  quad_first<H_, NQ>(wc, wl, cx, q, a);
  for (int b = 0; b < nb; ++b) {
    quad_splat(z[0], bl[0]);
    quad_act(a, x, lane);
    quad_layer<MT, 1, NQ>(wl, 0, wl + layer_stride, x, q, z);
    quad_act(z[0], x, lane);
    quad_splat(z[0], bl[C_]);
    wl += layer_stride;
    quad_layer<MT, 1, NQ>(wl, 0, wl + layer_stride, x, q, z);
#pragma unroll
    for (int k = 0; k < NQ; ++k) a[k] = a[k] + z[0][k];
    wl += layer_stride;
    bl += 2 * C_;
  }
  f4 h[2][NQ];
  quad_splat(h[0], bias_head[lane]);
  quad_splat(h[1], bias_head[64 + min(lane, 47)]);
  // (row 64 + lane of the head; it has 112, and lanes 48 on repeat their first)
  const float* w_head = w + L.layer0 + 2 * nb * layer_stride + ((lane >> 4) * MT * 64 + r16) * 4;
  const int second = lane < 48 ? 4 * MT * 256 : 0;
  QuadW<2> qh[2];
  qh[0].load(w_head, second);
  quad_act(a, x, lane);
  quad_layer<MT, 2, NQ>(w_head, second, w_head, x, qh, h);
#pragma unroll
  for (int k = 0; k < NQ; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      hb[(4 * k + v) * HB_STRIDE + lane] = h[0][k][v];
      hb[(4 * k + v) * HB_STRIDE + 64 + lane] = h[1][k][v];
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Contexts for net_quad of a pixel per lane 4 a + r: each lane loads its
// inputs k = 16 j + a, clamped into the lane's pixels and masked as
// gather_clamped does, or from the sheared window as gather_ring does.
template <int H_>
NXD void quad_gather_image(float (&cx)[quad_inputs(H_)], const uint8_t* img, int W, int y0, int x0, int Hl, int Wl, int i,
                           int j, int lane) {
  const gbytes g = as_global(img);
  int raw[quad_inputs(H_)], ok[quad_inputs(H_)];
#pragma unroll
  for (int n = 0; n < quad_inputs(H_); ++n) {
    int k, dy;
    quad_tap<H_>(n, lane, k, dy);
    const int e = k - 3 * (2 * H_ + 1) * dy, dx = e / 3, ch = e - 3 * dx;
    const int y = i - H_ + dy, x = j - H_ + dx;
    ok[n] = -(int)(((unsigned)y < (unsigned)Hl) & ((unsigned)x < (unsigned)Wl));
    raw[n] = g[((int64_t)(y0 + min(max(y, 0), Hl - 1)) * W + (x0 + min(max(x, 0), Wl - 1))) * 3 + ch];
  }
#pragma unroll
  for (int n = 0; n < quad_inputs(H_); ++n) cx[n] = (float)((2 * raw[n] - 255) & ok[n]) * (1.0f / 255.0f);
}
template <int H_>
NXD void quad_gather_ring(float (&cx)[quad_inputs(H_)], const int16_t* ring, int rows, int t, int i, int lane) {
  constexpr int Q = H_ * (H_ + 2), PLANES = 3 * RING_COLS;
  const int s = 3 * ((t - Q) & (RING_COLS - 1));
  int raw[quad_inputs(H_)];
#pragma unroll
  for (int n = 0; n < quad_inputs(H_); ++n) {
    int k, dy;
    quad_tap<H_>(n, lane, k, dy);
    // tap (dy, dx), channel ch is plane 3 ((t - Q) + (h + 1) dy + dx) + ch = 3 (t - Q) + k - 3 h dy
    uint32_t plane = (uint32_t)(s + k - 3 * H_ * dy);
    plane = min(plane, plane - (uint32_t)PLANES);
    raw[n] = ring_at(ring, 0, 2u * (plane * (uint32_t)rows + (uint32_t)(i + dy)));
  }
#pragma unroll
  for (int n = 0; n < quad_inputs(H_); ++n) cx[n] = (float)raw[n] * (1.0f / 255.0f);
}

// ------------------------------------------------------------------ mixture
// Head slot s = 4 mt + v of lane group g holds parameter s % 10 of component
// m = g + 4 (s / 10) (s < 30, m < 10): 0 logit, 1..3 means R,G,B,
// 4..6 raw log-scales R,G,B, 7..9 pre-tanh coefficients G|R, B|R, B|G.
// Lane groups 0,1 own three components, groups 2,3 own two (slot 2 unused).
struct Mix {
  float logw[3];       // current (posterior) log weights
  float mu[3][3];      // [channel][slot] base means
  float invs[3][3];    // [channel][slot] inverse scales
  float co[3][3];      // [coef][slot] tanh'd coefficients alpha, beta, gamma
};

// The lane group's slots (see head_row_src) from its values. The swap
// exchanges its first operand's lanes 32 .. 63 with its second's 0 .. 31, so
// against zeros it brings groups 0 and 1 their slots 28 and 29 and leaves
// zeros in the others'. head_values is the reverse.
constexpr int HEAD_SLOTS = 8;  // slots / 4
NXD void swap_halves(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// a's lane rows 1 and 3 with b's 0 and 2
NXD void swap_rows(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
NXD void head_slots(const f4 (&hd)[HEAD_TILES], f4 (&s)[HEAD_SLOTS]) {
#pragma unroll
  for (int t = 0; t < HEAD_TILES; ++t) s[t] = hd[t];
  s[7] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    float a = s[5][v], b = 0.0f;
    swap_halves(a, b);
    s[5][v] = a;
    s[7][v] = b;
  }
}
NXD void head_values(const f4 (&s)[HEAD_SLOTS], f4 (&hd)[HEAD_TILES]) {
#pragma unroll
  for (int t = 0; t < HEAD_TILES; ++t) hd[t] = s[t];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    float a = s[5][v], b = s[7][v];
    swap_halves(a, b);
    hd[5][v] = a;
  }
}
NXD float head_slot(const f4 (&s)[HEAD_SLOTS], int k) { return s[k >> 2][k & 3]; }

// log-sum-exp over the ten components of one pixel (own slots, fixed tree;
// -infinity in a slot without a component)
NXD float lse10(const float (&t)[3]) {
  float m = xmax(t[0], t[1]);
  m = grp_max(xmax(m, t[2]));
  float s = xexp(t[0] - m) + xexp(t[1] - m);
  s = s + xexp(t[2] - m);
  s = grp_sum(s);
  return m + xlog(s);
}

NXD void mix_prep(const f4 (&rows)[HEAD_TILES], Mix& M, bool has2) {
  f4 hd[HEAD_SLOTS];
  head_slots(rows, hd);
  float lam[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) lam[j] = head_slot(hd, 10 * j);
  if (!has2) lam[2] = -INFINITY;
  const float lse = lse10(lam);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    M.logw[j] = lam[j] - lse;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      M.mu[c][j] = head_slot(hd, 10 * j + 1 + c);
      M.invs[c][j] = xexp(-xmax(head_slot(hd, 10 * j + 4 + c), -7.0f));
      M.co[c][j] = xtanh(head_slot(hd, 10 * j + 7 + c));
    }
  }
}

// Mixture of channel c given the normalised values of the earlier channels:
// weights, shifted means, inverse scales of this lane's slots, and the
// sigmoid coefficients a = s log2(e), b = mu a used by cdf_eval. (c may be a
// runtime value: the channel rows are selected, not indexed, so the mixture
// stays in registers.)
struct Chan {
  float w[3], mu[3], is[3], a[3], b[3];
};

NXD void chan_params(const Mix& M, int c, float xr, float xg, Chan& K) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    K.w[j] = xexp(M.logw[j]);
    const float is = c == 0 ? M.invs[0][j] : (c == 1 ? M.invs[1][j] : M.invs[2][j]);
    float m;
    if (c == 0) {
      m = M.mu[0][j];
    } else if (c == 1) {
      m = M.mu[1][j] + M.co[0][j] * xr;
    } else {
      const float t1 = M.co[1][j] * xr;
      const float t2 = M.co[2][j] * xg;
      m = (M.mu[2][j] + t1) + t2;
    }
    K.mu[j] = m;
    K.is[j] = is;
    K.a[j] = is * kLog2e;
    K.b[j] = m * K.a[j];
  }
}

// Mixture CDF at bin edge k (1..255):
//   F = sum_m w_m / (1 + 2^(b_m - B_k a_m)),  i.e. sum_m w_m sigmoid((B_k - mu_m) s_m),
// the sum taken per lane group over its slots in order, then across groups.
// The exponent is one fused multiply-add, monotone decreasing in k (a >= 0),
// and the hardware exp2 and reciprocal are monotone, so F is monotone in k.
// Every lane of a pixel must call this with the same k (lane-group swaps).
NXD float cdf_eval(int k, const float (&w)[3], const float (&a)[3], const float (&b)[3]) {
  const float e = bin_edge(k);
  float t[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(-e, a[j], b[j]));
    t[j] = w[j] * __builtin_amdgcn_rcpf(1.0f + x);
  }
  const float s = (t[0] + t[1]) + t[2];
  return grp_sum(s);
}

// Quantised CDF value: k + floor(clamp(F, 0, 1) * (2^16 - 256)). Monotone in
// k whenever F is, with a step of at least 1 between consecutive symbols.
NXD uint32_t cdf_quant(int k, float F) {
  const float c = __builtin_amdgcn_fmed3f(F, 0.0f, 1.0f);
  return (uint32_t)k + (uint32_t)(c * 65280.0f);
}

// log probability of bin x under this lane's slots (Q: stable difference of
// logistic CDFs: log sig(z_hi) + log sig(-z_lo) + log(1 - exp(-(z_hi - z_lo))),
// with z_hi - z_lo = (2/255) s exactly in real arithmetic).
NXD float log_bin(int x, float mu, float is) {
  // both edge forms and the interior form, then a select (no branch)
  const float zlo = (bin_edge(min(max(x, 1), 255)) - mu) * is;
  const float zhi = (bin_edge(min(max(x + 1, 1), 255)) - mu) * is;
  const float d = is * (2.0f / 255.0f);
  const float lhi = xlogsigmoid(zhi), llo = xlogsigmoid(-zlo);
  const float mid = (lhi + llo) + xlog(-xexpm1(-d));
  return x <= 0 ? lhi : (x >= 255 ? llo : mid);
}

// Condition the weights on the coded value x of channel c (posterior for the
// next channel); returns the channel's natural-log probability.
NXD float posterior(Mix& M, int x, const float (&mu)[3], const float (&is)[3], bool has2) {
  float t[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) t[j] = M.logw[j] + log_bin(x, mu[j], is[j]);
  if (!has2) t[2] = -INFINITY;
  const float lse = lse10(t);
#pragma unroll
  for (int j = 0; j < 3; ++j) M.logw[j] = t[j] - lse;
  return lse;
}

// ------------------------------------------------------------------ mixture, 16 lanes per pixel
// The row decoder's mixture phase gives each pixel a row of 16 lanes: lane m
// holds component m (m < 10; lanes 10..15 hold none and add nothing). The
// arithmetic of a component is the lane-group form's, and sums over the
// components take the same tree: lane g < 4 adds (t_g + t_{g+4}) + t_{g+8},
// then (s_0 + s_1) + (s_2 + s_3), so every value is bitwise the one the
// encoder and the other decoders compute. The tree runs on DPP row shifts
// (lane i reads lane i + n of its row; only lanes 0..3 use the sums), and
// row_newbcast hands lane 0's result to the whole row.
template <int CTRL>
NXD float dpp_row(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int DPP_SHL1 = 0x101, DPP_SHL2 = 0x102, DPP_SHL4 = 0x104, DPP_SHL8 = 0x108, DPP_BCAST0 = 0x150;
NXD float row_bcast0(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), DPP_BCAST0, 0xf, 0xf, true));
}
NXD float row16_sum(float t) {
  const float s = (t + dpp_row<DPP_SHL4>(t)) + dpp_row<DPP_SHL8>(t);
  const float u = s + dpp_row<DPP_SHL1>(s);
  return row_bcast0(u + dpp_row<DPP_SHL2>(u));
}
NXD float row16_max(float v) {
  v = fmaxf(v, dpp_row<DPP_SHL8>(v));
  v = fmaxf(v, dpp_row<DPP_SHL4>(v));
  v = fmaxf(v, dpp_row<DPP_SHL2>(v));
  v = fmaxf(v, dpp_row<DPP_SHL1>(v));
  return row_bcast0(v);
}
// lse10 over the row's live components (t of a lane without one is ignored)
NXD float lse16(float t, bool live) {
  const float m = row16_max(live ? t : -INFINITY);
  const float e = live ? xexp(t - m) : 0.0f;
  return m + xlog(row16_sum(e));
}

struct Mix16 {
  float logw;                  // posterior log weight of this lane's component
  float mu[3], invs[3], co[3];
};
// mix_prep for component m of the pixel whose head rows are at hp
NXD void mix_prep16(const float* hp, int m, Mix16& M) {
  const bool live = m < 10;
  const int mm = live ? m : 0;
  const float lam = live ? hp[head_row(mm, 0)] : -INFINITY;
  M.logw = lam - lse16(lam, live);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    M.mu[c] = hp[head_row(mm, 1 + c)];
    M.invs[c] = xexp(-xmax(hp[head_row(mm, 4 + c)], -7.0f));
    M.co[c] = xtanh(hp[head_row(mm, 7 + c)]);
  }
}
struct Chan16 {
  float w, mu, is, a, b;
};
NXD void chan_params16(const Mix16& M, int c, float xr, float xg, Chan16& Q) {
  Q.w = xexp(M.logw);
  Q.is = c == 0 ? M.invs[0] : (c == 1 ? M.invs[1] : M.invs[2]);
  float m;
  if (c == 0) {
    m = M.mu[0];
  } else if (c == 1) {
    m = M.mu[1] + M.co[0] * xr;
  } else {
    const float t1 = M.co[1] * xr;
    const float t2 = M.co[2] * xg;
    m = (M.mu[2] + t1) + t2;
  }
  Q.mu = m;
  Q.a = Q.is * kLog2e;
  Q.b = m * Q.a;
}
NXD float posterior16(Mix16& M, int x, const Chan16& Q, bool live) {
  const float t = live ? M.logw + log_bin(x, Q.mu, Q.is) : -INFINITY;
  const float lse = lse16(t, live);
  M.logw = t - lse;
  return lse;
}

// ------------------------------------------------------------------ sampling
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): a counter-based
// generator of ten rounds; each round multiplies words 0 and 2 by two odd
// constants (full 128-bit products) and mixes the halves with words 1 and 3
// and the key, which steps by two Weyl increments between rounds. Here the
// counter is (n, 0, 0, 0) and the key (seed, 0).
NXD void philox4x64(uint64_t n, uint64_t seed, uint64_t (&o)[4]) {
  uint64_t x0 = n, x1 = 0, x2 = 0, x3 = 0, k0 = seed, k1 = 0;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t a = 0xD2E7470EE14C6C93ull, b = 0xCA5A826395121157ull;
    const uint64_t hi0 = __umul64hi(a, x0), lo0 = a * x0;
    const uint64_t hi1 = __umul64hi(b, x2), lo1 = b * x2;
    x0 = hi1 ^ x1 ^ k0;
    x1 = lo1;
    x2 = hi0 ^ x3 ^ k1;
    x3 = lo0;
    k0 += 0x9E3779B97F4A7C15ull;
    k1 += 0xBB67AE8584CAA73Bull;
  }
  o[0] = x0; o[1] = x1; o[2] = x2; o[3] = x3;
}

// the 16-bit uniform slots of the three channels of pixel (y, x) of a W-wide
// image: top 16 bits of words 0, 1, 2 of the block with counter y W + x
NXD void sample_slots(uint64_t seed, int W, int y, int x, uint32_t (&sl)[3]) {
  uint64_t o[4];
  philox4x64((uint64_t)y * (uint64_t)W + (uint64_t)x, seed, o);
  sl[0] = (uint32_t)(o[0] >> 48);
  sl[1] = (uint32_t)(o[1] >> 48);
  sl[2] = (uint32_t)(o[2] >> 48);
}

}  // namespace nx
