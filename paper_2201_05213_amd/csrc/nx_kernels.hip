// nx_kernels.hip -- HIP kernels for gfx950 (MI355X):
//   k_pass      full-image pass: every pixel's quantised CDF at its own value
//               (encoder symbols), or its continuous code length (NLL), or a
//               full CDF row (debug), 16 pixels per wave on MFMA
//   k_rans_*    rANS encoder: symbols laid out in coding order, then a wave
//               or a thread per stream
//   k_lane_scan / k_img_scan / k_pack   container assembly
//   k_decode    persistent decoder: waves pop lanes from a queue and decode
//               them step by step (wavefront) or pixel by pixel (raster)
// (with few lanes, or a stream per row: nx_team.hip)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "nx_coder.hpp"

namespace nx {

constexpr int NWAVES = 16;      // waves per full-image-pass workgroup (all share the LDS weights)
constexpr int NWAVES_DEC = DECODE_WAVES;  // waves per decoder workgroup
constexpr int PIV_WORDS = 256;            // per decoder wave: 16 pixels x 16 pivot CDF values
constexpr int PRM_STRIDE = 36;            // floats per pixel: (w, a, b) of 12 component slots
constexpr int PRM_WORDS = 16 * PRM_STRIDE;  // per decoder wave: one channel's mixtures of 16 pixels
constexpr int WAVE_LDS_WORDS = PIV_WORDS + PRM_WORDS;
static_assert(DECODE_LDS_EXTRA == NWAVES_DEC * WAVE_LDS_WORDS * 4, "decoder LDS budget");

// the image holding global stream `key` (by its first stream)
NXD int find_img_stream(const ImgDesc* __restrict__ d, int n, int64_t key) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (d[mid].stream_base <= key) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Where stream e of an image (its stream table entry) lies: its lane (q, and
// the patch row and column ly, lx), the lane's rows and columns, its index
// among the lane's streams (kk, K streams) or its row (r, row streams), the
// pixels of the lanes before it in lane order, and the end of its byte slot
// in the encoder's slot buffer (slots are laid out in entry order: with K
// streams, K slots of 6 B per lane pixel + 8 B per lane; with row streams,
// 6 B per row pixel + 8 B per row).
struct StreamAt {
  int q, ly, lx, Hl, Wl, kk, r;
  int64_t lane_px_off, slot_end;
};
NXD StreamAt stream_at(const ImgDesc& D, int K, int64_t e) {
  StreamAt S;
  if (K == ROW_STREAMS) {
    const int64_t per_prow = (int64_t)D.nlx * D.ph;  // entries of a full patch row
    S.ly = (int)(e / per_prow);
    S.Hl = min(D.ph, D.H - S.ly * D.ph);
    const int64_t rem = e - (int64_t)S.ly * per_prow;
    S.lx = (int)(rem / S.Hl);
    S.r = (int)(rem - (int64_t)S.lx * S.Hl);
    S.kk = 0;
  } else {
    const int q = (int)(e / K);
    S.kk = (int)(e - (int64_t)q * K);
    S.ly = q / D.nlx;
    S.lx = q - S.ly * D.nlx;
    S.Hl = min(D.ph, D.H - S.ly * D.ph);
    S.r = 0;
  }
  S.q = S.ly * D.nlx + S.lx;
  S.Wl = min(D.pw, D.W - S.lx * D.pw);
  S.lane_px_off = (int64_t)S.ly * D.ph * D.W + (int64_t)S.lx * D.pw * S.Hl;
  if (K == ROW_STREAMS)
    S.slot_end = D.slot_base + 6 * (S.lane_px_off + (int64_t)(S.r + 1) * S.Wl) + 8 * (e + 1);
  else
    S.slot_end = D.slot_base + K * (6 * S.lane_px_off + 8 * (int64_t)S.q) +
                 (S.kk + 1) * lane_slot_bytes((int64_t)S.Hl * S.Wl);
  return S;
}


// ------------------------------------------------------------------ full-image pass
template <int H_, int C_>
__global__ void __launch_bounds__(NWAVES * 64) k_pass(PassArgs A) {
  extern __shared__ float4 smem_f4[];
  float* w = (float*)smem_f4;
  load_weights(w, A.w, A.wfloats);
  const int lane = threadIdx.x & 63, p = lane & 15, g = lane >> 4;
  const bool has2 = g < 2;
  // a batch of at most a tile per wave is dealt to the workgroups first, so
  // that it spreads over the CUs; else a workgroup takes tiles side by side
  const int64_t nwv = (int64_t)gridDim.x * NWAVES;
  const int wv = uniform((int)(threadIdx.x >> 6));
  const int64_t gw = A.n_tiles <= nwv ? (int64_t)wv * gridDim.x + blockIdx.x : (int64_t)blockIdx.x * NWAVES + wv;
  TapCodes<H_> tc;
  tc.init(g);
  for (int64_t t = gw; t < A.n_tiles; t += nwv) {
    tc.refresh();
    const int n = find_img_uniform(A.desc, A.n_img, t, false);
    const ImgDesc D = uniform_desc(A.desc + n);
    const uint32_t tt = (uint32_t)(t - D.tile_base);  // < 65535 x 4096
    const int y = uniform((int)(tt / (uint32_t)D.ntx));
    const int xraw = (int)(tt - (uint32_t)y * (uint32_t)D.ntx) * 16 + p;
    const bool active = xraw < D.W;
    const int x = active ? xraw : D.W - 1;
    // y / ph and x / pw by float quotients: (v + 0.5) / d is at least 0.5 / d
    // from an integer, the error below 2^-22 v / d with v < 2^16
    const int ly = uniform((int)(((float)y + 0.5f) * __builtin_amdgcn_rcpf((float)D.ph)));
    const int lx = (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)D.pw));
    const int y0 = ly * D.ph, x0 = lx * D.pw;
    const int Hl = min(D.ph, D.H - y0), Wl = min(D.pw, D.W - x0);
    float ctx[conv_chunks(H_)];
    gather<H_>(ctx, tc, D.px, D.W, y0, x0, Hl, Wl, y - y0, x - x0, y);
    f4 head[HEAD_TILES];
    net_forward<H_, C_>(lds_weights(w), A.nb, ctx, head, lane);
    Mix M;
    mix_prep(head, M, has2);
    const int64_t pix = (int64_t)y * D.W + x;
    int xv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) xv[c] = D.px[pix * 3 + c];
    const float xr = normalise(xv[0]), xg = normalise(xv[1]);
    float bits = 0.0f;
    const int64_t gpix = D.px_base + pix;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      Chan K;
      chan_params(M, c, xr, xg, K);
      if (A.mode == 0) {
        const float Flo = cdf_eval(max(xv[c], 1), K.w, K.a, K.b);
        const float Fhi = cdf_eval(min(xv[c] + 1, 255), K.w, K.a, K.b);
        const uint32_t lo = xv[c] == 0 ? 0u : cdf_quant(xv[c], Flo);
        const uint32_t hi = xv[c] == 255 ? CDF_TOTAL : cdf_quant(xv[c] + 1, Fhi);
        if (active && g == 0) A.sym[gpix * 3 + c] = lo | ((hi - lo) << 16);
        bits += (float)CDF_BITS - __builtin_amdgcn_logf((float)(hi - lo));
        if (c < 2) posterior(M, xv[c], K.mu, K.is, has2);
      } else if (A.mode == 1) {
        const float lp = posterior(M, xv[c], K.mu, K.is, has2);
        bits += -lp * kLog2e;
      } else {
        for (int k = 1; k < 256; ++k) {
          const uint32_t v = cdf_quant(k, cdf_eval(k, K.w, K.a, K.b));
          if (active && g == 0) A.cdf[(gpix * 3 + c) * 257 + k] = (int32_t)v;
        }
        if (active && g == 0) {
          A.cdf[(gpix * 3 + c) * 257] = 0;
          A.cdf[(gpix * 3 + c) * 257 + 256] = (int32_t)CDF_TOTAL;
        }
        if (c < 2) posterior(M, xv[c], K.mu, K.is, has2);
      }
    }
    if (A.bits && active && g == 0) A.bits[gpix] = bits;
  }
}

// ------------------------------------------------------------------ rANS encoder
// A stream's state is one serial chain, so what bounds the coder is the
// instructions of that chain, run by a wave that has its SIMD to itself (6 to
// 8 cycles each). Everything that does not depend on the state comes out of
// it: k_rans_counts and k_rans_scatter lay every stream's symbols out
// contiguously in coding order, reading the symbol buffer in pixel order, and
// with few streams a wave codes each: its lanes prepare 64 symbols at a time,
// the quotient by a symbol's frequency becoming a multiplication by its
// reciprocal (k_rans_enc_wave). With many, a thread codes a stream
// (k_rans_enc).

// lane geometry of stream SL = L K + kk, and where its encoder scratch lies
struct StreamGeom {
  ImgDesc D;
  int kk, q, y0, x0, Hl, Wl;
  int64_t lane_px_off;
  int64_t rev_cap, rev_off;      // words of the stream's coding-order buffer, and its first
  int64_t after_cap, after_off;  // entries of its per-step offsets, and its first
};
NXD StreamGeom stream_geom(const RansEncArgs& A, int64_t SL) {
  StreamGeom G;
  const int64_t L = SL / A.K;
  G.kk = (int)(SL - L * A.K);
  const int n = find_img(A.desc, A.n_img, L, true);
  G.D = A.desc[n];
  G.q = (int)(L - G.D.lane_base);
  const int64_t rel = SL - G.D.lane_base * A.K;  // the stream's index within its image
  G.rev_cap = stream_rev_words(G.D.ph, G.D.pw, A.K);
  G.after_cap = stream_after_entries(G.D.ph, G.D.pw);
  G.rev_off = G.D.rev_base + rel * G.rev_cap;
  G.after_off = G.D.after_base + rel * G.after_cap;
  const int ly = G.q / G.D.nlx, lx = G.q - ly * G.D.nlx;
  G.y0 = ly * G.D.ph;
  G.x0 = lx * G.D.pw;
  G.Hl = min(G.D.ph, G.D.H - G.y0);
  G.Wl = min(G.D.pw, G.D.W - G.x0);
  G.lane_px_off = (int64_t)ly * G.D.ph * G.D.W + (int64_t)lx * G.D.pw * G.Hl;
  return G;
}

// One wave per stream. Each lane counts the stream's symbols in a range of
// wavefront steps (stream_rows_at); a suffix sum across the wave gives the
// symbols after each range; the lane then writes, per step t of its range,
// how many of the stream's symbols come in steps after t (in coding order
// the later steps come first). Lane 0's inclusive sum is the stream's
// length. Raster order: the length only.
template <int O, int K>
__global__ void __launch_bounds__(64) k_rans_counts(RansEncArgs A) {
  const int64_t SL = blockIdx.x;
  const int lane = (int)threadIdx.x;
  const StreamGeom G = stream_geom(A, SL);
  if (A.order == 0) {
    if (lane == 0) A.lane_len[SL] = (uint32_t)min<int64_t>(3LL * G.Hl * G.Wl, G.rev_cap);
    return;
  }
  const int T = G.Wl + O * (G.Hl - 1);
  const int tlo = (int)((int64_t)T * lane / 64), thi = (int)((int64_t)T * (lane + 1) / 64);
  int cnt = 0;
  for (int t = tlo; t < thi; ++t) cnt += 3 * stream_rows_at(t, G.Hl, G.Wl, O, K, G.kk);
  int suf = cnt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_down(suf, d, 64);
    if (lane + d < 64) suf += v;
  }
  int32_t* tab = A.after + G.after_off;
  int S = suf - cnt;
  for (int t = thi - 1; t >= tlo; --t) {
    if (t < G.after_cap) tab[t] = S;
    S += 3 * stream_rows_at(t, G.Hl, G.Wl, O, K, G.kk);
  }
  if (lane == 0) A.lane_len[SL] = (uint32_t)min<int64_t>(suf, G.rev_cap);
}

// What coding a symbol (s, f) needs besides the state (a table entry per symbol
// with a reciprocal for the division, a bias that makes good the reciprocal of
// f = 1, and the factor 2^16 - f: the method of F. Giesen's public-domain rANS coder
// (rans_byte.h), whose exact reciprocals are those of R. Alverson, "Integer
// division using reciprocals", 1991): y / f is the high
// word of y M, shifted right by sh, exactly, for every y < 2^31 (M =
// ceil(2^(32 + sh) / f), 2^sh < f <= 2^(sh + 1), so M f exceeds the power of
// two by e < f <= 2^(sh + 1) and y e < 2^(32 + sh)). For f = 1, M would be
// 2^32: M = 2^32 - 1 gives y - 1, which 65535 more in the sum makes good.
//   y -> (y / f) 2^16 + y mod f + s = y + (y / f) (2^16 - f) + s
struct alignas(16) PutSym {
  uint32_t M, xm;   // reciprocal; f 2^15, the state from which a byte is shed first
  uint32_t bias;    // xm + s (f = 1: xm + s + 65535)
  uint32_t mult;    // 2^16 - f, and sh from bit 24 up (24-bit multiplies do not see it)
};
NXD PutSym put_sym(uint32_t w) {
  const uint32_t s = w & 0xffffu, f = w >> 16;
  const uint32_t sh = 31u - (uint32_t)__builtin_clz((f - 1u) | 1u);
  // M from a float quotient (within 2^-22 of it) corrected by its remainder:
  // e = 2^(32 + sh) - M f modulo 2^32 is small enough to be read as signed
  const float r = __builtin_amdgcn_rcpf((float)f);
  uint32_t M = (uint32_t)(r * __uint_as_float((127u + 32u + sh) << 23));
  int32_t e = -(int32_t)(M * f);
  M += (uint32_t)(int32_t)floorf((float)e * r);
  e = -(int32_t)(M * f);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const bool up = e > 0, dn = e <= -(int32_t)f;
    M += up ? 1u : dn ? 0xffffffffu : 0u;
    e += up ? -(int32_t)f : dn ? (int32_t)f : 0;
  }
  PutSym P;
  P.M = f == 1u ? 0xffffffffu : M;
  P.xm = f << 15;
  P.bias = P.xm + s + (f == 1u ? 65535u : 0u);
  P.mult = ((CDF_TOTAL - f) & 0xffffffu) | (sh << 24);
  return P;
}

constexpr int SCATTER_PX = 2048;  // pixels of a lane per k_rans_scatter workgroup

// Workgroup (lane, chunk) reads a chunk of the lane's symbols in pixel order
// (coalesced) and puts each at its place in its stream's coding order
// (coding_slot plus the stream's symbols of later steps); raster order
// reverses the raster index. The writes of a workgroup stay within its
// lane's K streams.
template <int O, int K>
__global__ void __launch_bounds__(256) k_rans_scatter(RansEncArgs A) {
  const int64_t L = blockIdx.x;
  const StreamGeom G = stream_geom(A, L * K);
  const int64_t npx = (int64_t)G.Hl * G.Wl;
  for (int64_t q0 = (int64_t)blockIdx.y * SCATTER_PX; q0 < npx; q0 += (int64_t)gridDim.y * SCATTER_PX) {
    const int64_t q1 = min<int64_t>(npx, q0 + SCATTER_PX);
    const uint32_t* sym = A.sym + G.D.px_base * 3;
    for (int64_t q = q0 + threadIdx.x; q < q1; q += 256) {
      const int i = (int)((uint32_t)q / (uint32_t)G.Wl), j = (int)((uint32_t)q - (uint32_t)i * (uint32_t)G.Wl);
      const uint32_t* sp = sym + ((int64_t)(G.y0 + i) * G.D.W + (G.x0 + j)) * 3;
      const uint32_t v[3] = {sp[0], sp[1], sp[2]};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        int kk = 0;
        int64_t p;
        if (A.order == 0) {
          p = 3 * npx - 1 - (3 * q + c);
        } else {
          int t, off;
          coding_slot(i, j, c, G.Hl, G.Wl, O, K, kk, t, off);
          p = (int64_t)A.after[G.after_off + kk * G.after_cap + t] + off;
        }
        if (p >= 0 && p < G.rev_cap) A.rev[G.rev_off + kk * G.rev_cap + p] = v[c];
      }
    }
  }
}

// A push on a state x >= f first sheds low bytes while the state is at least
// xm = f 2^15 (two at most, the state being below 2^31): of x, x >> 8 and
// x >> 16, the largest below xm is left. Less xm, modulo 2^32, the values
// below xm are the large ones, in order: a maximum finds it without a
// compare and its hazards. Returns it less xm.
NXD uint32_t put_renorm(uint32_t x, uint32_t xm) {
  const uint32_t a = x - xm, b = (x >> 8) - xm, c = (x >> 16) - xm;
  return max(max(a, b), c);
}
// the state after pushing symbol e on x >= f
NXD uint32_t put_state(uint32_t x, const PutSym& e) {
  const uint32_t m = put_renorm(x, e.xm);
  const uint32_t q = __umulhi(m + e.xm, e.M) >> (e.mult >> 24);
  return __umul24(q, e.mult) + (m + e.bias);
}

// The bytes a thread sheds over PUT_BATCH symbols gather in its window in LDS,
// downwards from the window's end, and go to memory as whole words: a store
// of each symbol's bytes is a transaction of its own at the L2, which bounded
// the coder of a large batch.
constexpr int PUT_BATCH = 16;
constexpr int PUT_WINDOW = 2 * PUT_BATCH;  // two bytes a symbol at most
constexpr int PUT_STRIDE = PUT_WINDOW + 16;
struct PutWindow {
  uint8_t* end;  // LDS, 16-byte aligned
  uint32_t o;    // bytes held: end - o .. end - 1
  // to memory below `out`, the last word with up to 3 bytes below them, which
  // the next batch overwrites (or which lie below the stream's first byte,
  // inside its slot)
  NXD void flush(uint8_t*& out) {
    uint32_t w[PUT_WINDOW / 4];
#pragma unroll
    for (int k = 0; k < PUT_WINDOW / 16; ++k) {
      const uint4 v = *(const uint4*)(end - 16 * (k + 1));
      w[4 * k] = v.w;
      w[4 * k + 1] = v.z;
      w[4 * k + 2] = v.y;
      w[4 * k + 3] = v.x;
    }
    struct __attribute__((packed)) Word {
      uint32_t v;
    };
#pragma unroll
    for (int k = 0; k < PUT_WINDOW / 4; ++k)
      if (4u * k < o) ((Word*)(out - 4 * (k + 1)))->v = w[k];
    out -= o;
    o = 0;
  }
};

// Codes symbol w (s | f << 16) into a state; the bytes it sheds go to the
// window, the one shed first on top. Both candidates are always written: what
// is not shed is overwritten by the symbols that follow. A state below f (the
// first pushes of a stream) takes the symbol's spread slot and sheds nothing.
// y / f: a float quotient made a little too small (the reciprocal times
// 1 - 2^-21, so between the quotient less 2^-5 and the quotient, which is
// below 2^15), and one step up if the remainder asks for it.
NXD void put_write(uint32_t& x, uint32_t w, PutWindow& win, bool small) {
  const uint32_t s = w & 0xffffu, f = w >> 16;
  if (small && x < f) {
    x = spread_select(x, s, f);
    return;
  }
  const uint32_t xm = f << 15;
  const float rf = __builtin_amdgcn_rcpf((float)f) * (1.0f - 0x1p-21f);
  uint8_t* at = win.end - win.o;
  at[-1] = (uint8_t)x;
  at[-2] = (uint8_t)(x >> 8);
  const uint32_t y = put_renorm(x, xm) + xm;
  win.o += (x >= xm ? 1u : 0u) + ((x >> 8) >= xm ? 1u : 0u);
  const uint32_t q = (uint32_t)((float)y * rf);
  const uint32_t r = y - __umul24(q, f);
  const bool up = r >= f;
  x = ((q + (up ? 1u : 0u)) << CDF_BITS) + (r - (up ? f : 0u)) + s;
}

// the final state's significant bytes (x >= 1), most significant first
NXD uint8_t* put_end(uint32_t x, uint8_t* out) {
  do {
    *--out = (uint8_t)x;
    x >>= 8;
  } while (x != 0u);
  return out;
}

// One wave per stream (row streams: a lane row, its symbols read in place,
// backwards), 64 symbols at a time: the lanes work out what the coding of a
// symbol each needs, the first lane runs the chain (11 instructions a
// symbol: its symbols come from LDS 8 ahead, and the states go back there),
// and the lanes write the bytes their symbols shed, placed by counting the
// lanes before them. Chosen while the waves of a SIMD are few (rans_wave).
// 196,608 symbols in one stream: 36.7 ms (448 cycles a symbol) with a chain
// that divided by a float quotient and moved its own bytes, 7.3 ms (89) so.
template <bool ROWS>
__global__ void __launch_bounds__(64) k_rans_enc_wave(RansEncArgs A) {
  __shared__ PutSym ent[64 + 16];  // the last 16 are read ahead, never coded
  __shared__ uint32_t xs[64];      // the state each symbol was pushed on
  const int64_t SL = blockIdx.x;
  const int lane = threadIdx.x;
  const uint32_t* src;
  int64_t n, slot_end, step;
  if constexpr (ROWS) {
    const int im = find_img_stream(A.desc, A.n_img, SL);
    const ImgDesc D = A.desc[im];
    const StreamAt S = stream_at(D, ROW_STREAMS, SL - D.stream_base);
    n = 3 * (int64_t)S.Wl;
    slot_end = S.slot_end;
    src = A.sym + (D.px_base + (int64_t)(S.ly * D.ph + S.r) * D.W + (int64_t)S.lx * D.pw) * 3 + (n - 1);
    step = -1;
  } else {
    const StreamGeom G = stream_geom(A, SL);
    slot_end = G.D.slot_base + A.K * (6 * G.lane_px_off + 8 * (int64_t)G.q) +
               (G.kk + 1) * lane_slot_bytes((int64_t)G.Hl * G.Wl);
    src = A.rev + G.rev_off;
    n = A.lane_len[SL];
    step = 1;
  }
  uint8_t* out = A.slots + slot_end;  // the same in every lane
  uint32_t x = RANS_X0;               // lane 0's is the stream's
  uint32_t w = lane < n ? src[step * lane] : 0x10000u;
  for (int64_t p0 = 0; p0 < n; p0 += 64) {
    const PutSym mine = put_sym(w);
    ent[lane] = mine;
    const int64_t pn = p0 + 64 + lane;
    w = pn < n ? src[step * pn] : 0x10000u;
    const int cnt = n - p0 < 64 ? (int)(n - p0) : 64;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane == 0) {
      int k = 0;
      // a state from 2^23 up stays there, and above every f
      for (; k < cnt && x < RANS_L; ++k) {
        const PutSym e = ent[k];
        xs[k] = x;
        const uint32_t f = e.xm >> 15;  // where x < f, f > 1: the bias is xm + s
        x = x < f ? spread_select(x, e.bias - e.xm, f) : put_state(x, e);
      }
      if (k + 8 <= cnt) {
        PutSym ea[8], eb[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) ea[u] = ent[k + u];
        do {
#pragma unroll
          for (int u = 0; u < 8; ++u) eb[u] = ent[k + 8 + u];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            xs[k + u] = x;
            x = put_state(x, ea[u]);
          }
          k += 8;
          if (k + 8 > cnt) break;
#pragma unroll
          for (int u = 0; u < 8; ++u) ea[u] = ent[k + 8 + u];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            xs[k + u] = x;
            x = put_state(x, eb[u]);
          }
          k += 8;
        } while (k + 8 <= cnt);
      }
      for (; k < cnt; ++k) {
        xs[k] = x;
        x = put_state(x, ent[k]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint32_t xl = xs[lane];
    const bool b1 = lane < cnt && xl >= mine.xm, b2 = lane < cnt && (xl >> 8) >= mine.xm;
    const uint64_t m1 = __ballot(b1), m2 = __ballot(b2);
    const uint64_t below = (1ull << lane) - 1ull;
    uint8_t* at = out - (__popcll(m1 & below) + __popcll(m2 & below));
    if (b1) at[-1] = (uint8_t)xl;
    if (b2) at[-2] = (uint8_t)(xl >> 8);
    out -= __popcll(m1) + __popcll(m2);
  }
  if (lane == 0) A.lane_len[SL] = (uint32_t)((A.slots + slot_end) - put_end(x, out));
}

// One thread per stream (lane L, stream k: index L K + k), PUT_BATCH symbols
// at a time, the next in flight: a wave waits for a line of 32 symbols from
// HBM once in two rounds, and a round is longer than that takes. Bound by
// the 29 instructions of a symbol on a wave alone on its SIMD: 133 us for
// 32,512 streams of 968 symbols on average (226 us with a branch and up to two
// byte stores a symbol).
__global__ void __launch_bounds__(64) k_rans_enc(RansEncArgs A) {
  __shared__ __align__(16) uint8_t shed[64 * PUT_STRIDE];
  const int64_t SL = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (SL >= A.n_streams) return;
  const StreamGeom G = stream_geom(A, SL);
  const int64_t slot_end = G.D.slot_base + A.K * (6 * G.lane_px_off + 8 * (int64_t)G.q) +
                           (G.kk + 1) * lane_slot_bytes((int64_t)G.Hl * G.Wl);
  uint8_t* out = A.slots + slot_end;
  PutWindow win{shed + (threadIdx.x + 1) * PUT_STRIDE, 0u};
  const uint4* src = (const uint4*)(A.rev + G.rev_off);
  const int64_t n = A.lane_len[SL];
  uint32_t x = RANS_X0;
  constexpr int B = PUT_BATCH;
  uint4 nxt[B / 4];
#pragma unroll
  for (int u = 0; u < B / 4; ++u) nxt[u] = n > 0 ? src[u] : make_uint4(0u, 0u, 0u, 0u);
  for (int64_t p0 = 0; p0 < n; p0 += B) {
    uint32_t cur[B];
#pragma unroll
    for (int u = 0; u < B / 4; ++u) {
      cur[4 * u] = nxt[u].x;
      cur[4 * u + 1] = nxt[u].y;
      cur[4 * u + 2] = nxt[u].z;
      cur[4 * u + 3] = nxt[u].w;
    }
    if (p0 + B < n) {
#pragma unroll
      for (int u = 0; u < B / 4; ++u) nxt[u] = src[(p0 + B) / 4 + u];
    }
    // a state from 2^23 up stays there, and above every f; streams of a wave
    // end in different batches
    const bool grown = x >= RANS_L, whole = p0 + B <= n;
    if (__ballot(!(grown && whole)) == 0ull) {
#pragma unroll
      for (int u = 0; u < B; ++u) put_write(x, cur[u], win, false);
    } else if (__ballot(!grown) == 0ull) {
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (p0 + u < n) put_write(x, cur[u], win, false);
    } else {
      for (int u = 0; u < B; ++u) {
        // (the symbols move down one place a round: no indexed registers)
        if (p0 + u < n) put_write(x, cur[0], win, true);
#pragma unroll
        for (int v = 0; v + 1 < B; ++v) cur[v] = cur[v + 1];
      }
    }
    win.flush(out);
  }
  A.lane_len[SL] = (uint32_t)((A.slots + slot_end) - put_end(x, out));
}

// Row streams too many for a wave each: one thread per stream, its symbols
// read in place from the symbol buffer, backwards
__global__ void __launch_bounds__(64) k_rans_enc_rows(RansEncArgs A) {
  __shared__ __align__(16) uint8_t shed[64 * PUT_STRIDE];
  const int64_t SL = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (SL >= A.n_streams) return;
  const int n = find_img_stream(A.desc, A.n_img, SL);
  const ImgDesc D = A.desc[n];
  const int64_t e = SL - D.stream_base;
  const StreamAt S = stream_at(D, ROW_STREAMS, e);
  uint8_t* out = A.slots + S.slot_end;
  PutWindow win{shed + (threadIdx.x + 1) * PUT_STRIDE, 0u};
  const uint32_t* row = A.sym + (D.px_base + (int64_t)(S.ly * D.ph + S.r) * D.W + (int64_t)S.lx * D.pw) * 3;
  uint32_t x = RANS_X0;
  constexpr int B = PUT_BATCH;
  uint32_t v[B];
  for (int k = 3 * S.Wl - 1; k >= 0; k -= B) {
    const int nb = min(B, k + 1);
#pragma unroll
    for (int m = 0; m < B; ++m) v[m] = m < nb ? row[k - m] : 0u;
#pragma unroll
    for (int m = 0; m < B; ++m)
      if (m < nb) put_write(x, v[m], win, true);
    win.flush(out);
  }
  A.lane_len[SL] = (uint32_t)((A.slots + S.slot_end) - put_end(x, out));
}

// ------------------------------------------------------------------ container assembly
// inclusive sum over the wave's lanes
NXD uint64_t wave_scan(uint64_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// per image: lane_end (inclusive prefix of lane lengths), container bytes.
// SCAN_THREADS streams a round: sums within each wave by lane shuffles, then
// over the waves through LDS (two barriers a round; 32,512 streams of 6 images
// took 43 us with 256 threads and a barrier a doubling, 12 us so)
constexpr int SCAN_THREADS = 1024;
__global__ void __launch_bounds__(SCAN_THREADS) k_lane_scan(PackArgs A) {
  __shared__ uint32_t part[SCAN_THREADS / 64];
  const int n = blockIdx.x;
  const ImgDesc D = A.desc[n];
  const int64_t nl = image_streams(A.K, D.H, D.nlx, D.nly);  // streams of this image
  const int64_t sbase = D.stream_base;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (int64_t b0 = 0; b0 < nl; b0 += SCAN_THREADS) {
    const int64_t q = b0 + threadIdx.x;
    const uint32_t s = (uint32_t)wave_scan(q < nl ? A.lane_len[sbase + q] : 0u, lane);
    if (lane == 63) part[wv] = s;
    __syncthreads();
    uint32_t before = carry, all = 0;
#pragma unroll
    for (int w = 0; w < SCAN_THREADS / 64; ++w) {
      before += w < wv ? part[w] : 0u;
      all += part[w];
    }
    if (q < nl) A.lane_end[sbase + q] = before + s;
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) A.img_bytes[n] = (uint64_t)HDR_BYTES + 4ull * (uint64_t)nl + carry;  // nl = streams
}

// the containers' offsets, one wave
__global__ void __launch_bounds__(64) k_img_scan(PackArgs A) {
  const int lane = threadIdx.x;
  uint64_t acc = 0;
  for (int n0 = 0; n0 < A.n_img; n0 += 64) {
    const int n = n0 + lane;
    const uint64_t v = n < A.n_img ? A.img_bytes[n] : 0ull;
    const uint64_t s = wave_scan(v, lane);
    if (n < A.n_img) A.out_offsets[n] = acc + s - v;
    acc += __shfl(s, 63, 64);
  }
  if (lane == 0) {
    A.out_offsets[A.n_img] = acc;
    *A.overflow = acc > A.out_cap ? 1 : 0;
  }
}

// 16 bytes at any address (byte alignment: the hardware splits what it must)
struct __attribute__((packed)) Bytes16 {
  uint32_t w[4];
};

// 64-thread blocks (stream, part): payload copy, 16 bytes a lane, parts of
// PACK_PART bytes; the stream's first block writes its table entry, the
// image's first the header
constexpr uint32_t PACK_PART = 8192;
__global__ void __launch_bounds__(64) k_pack(PackArgs A) {
  if (*A.overflow) return;
  const int64_t SL = blockIdx.x;
  const int n = find_img_stream(A.desc, A.n_img, SL);
  const ImgDesc D = A.desc[n];
  const int64_t entry = SL - D.stream_base;
  const int64_t ns = image_streams(A.K, D.H, D.nlx, D.nly);
  const int nl = D.nlx * D.nly;
  const StreamAt S = stream_at(D, A.K, entry);
  const int64_t slot_end = S.slot_end;
  const uint32_t len = A.lane_len[SL];
  const uint32_t end = A.lane_end[SL];
  uint8_t* C = A.out + A.out_offsets[n];
  uint8_t* dst = C + HDR_BYTES + 4 * ns + (end - len);
  const uint8_t* src = A.slots + slot_end - len;
  for (uint64_t p0 = (uint64_t)blockIdx.y * PACK_PART; p0 < len; p0 += (uint64_t)gridDim.y * PACK_PART) {
    const uint64_t p1 = p0 + PACK_PART < len ? p0 + PACK_PART : len;
    uint64_t k = p0 + 16 * threadIdx.x;
    for (; k + 16 <= p1; k += 16 * 64) *(Bytes16*)(dst + k) = *(const Bytes16*)(src + k);
    for (; k < p1; ++k) dst[k] = src[k];
  }
  if (blockIdx.y != 0) return;
  if (threadIdx.x < 4) C[HDR_BYTES + 4 * entry + threadIdx.x] = (uint8_t)(end >> (8 * threadIdx.x));
  if (entry == 0 && threadIdx.x == 0) {
    uint8_t h[HDR_BYTES];
    for (int k = 0; k < HDR_BYTES; ++k) h[k] = 0;
    h[0] = 'N'; h[1] = 'L'; h[2] = 'X'; h[3] = 'C';
    h[4] = CONTAINER_VERSION;
    h[5] = (uint8_t)A.order;
    h[6] = (uint8_t)A.h;
    h[7] = (uint8_t)A.K;
    for (int k = 0; k < 4; ++k) h[8 + k] = (uint8_t)((uint32_t)D.H >> (8 * k));
    for (int k = 0; k < 4; ++k) h[12 + k] = (uint8_t)((uint32_t)D.W >> (8 * k));
    const uint32_t ph = D.ph == D.H ? 0u : (uint32_t)D.ph, pw = D.pw == D.W ? 0u : (uint32_t)D.pw;
    h[16] = (uint8_t)ph; h[17] = (uint8_t)(ph >> 8);
    h[18] = (uint8_t)pw; h[19] = (uint8_t)(pw >> 8);
    for (int k = 0; k < 8; ++k) h[20 + k] = (uint8_t)(A.model_hash >> (8 * k));
    for (int k = 0; k < 4; ++k) h[28 + k] = (uint8_t)((uint32_t)nl >> (8 * k));
    for (int k = 0; k < HDR_BYTES; ++k) C[k] = h[k];
  }
}

// ------------------------------------------------------------------ decoder
// ------------------------------------------------------------------ four-row decoding
// With four streams per lane, the wave's 16-lane rows work independently:
// row g searches the symbol of stream g while every lane evaluates all ten
// mixture components at its own point, so no cross-row reduction is needed.
// A pixel's mixture for the channel is staged in LDS as (w, a, b) of
// component m at floats 3m..3m+2 of the pixel's row of the table.
NXD void load_mix10(Mix10& P, const float* prm, int pix) {
  const float4* s = (const float4*)(prm + pix * PRM_STRIDE);
  float v[32];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float4 t = s[i];
    v[4 * i] = t.x; v[4 * i + 1] = t.y; v[4 * i + 2] = t.z; v[4 * i + 3] = t.w;
  }
#pragma unroll
  for (int m = 0; m < 10; ++m) {
    P.w[m] = v[3 * m];
    P.a[m] = v[3 * m + 1];
    P.b[m] = v[3 * m + 2];
  }
}

// One stream per row: state, position and a 64-byte window of its bytes,
// 4 bytes per lane of the row (every value uniform within the row).
struct RowStream {
  const uint8_t* S;
  uint32_t len, base, pos, x, word;
  // lanes of the row load the window [at, at + 64) (clamped, unconditional loads)
  NXD void fill(uint32_t at, int p) {
    base = at;
    const gbytes gs = as_global(S);
    uint32_t v = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t o = at + 4 * (uint32_t)p + b;
      const uint32_t byte = gs[o < len ? o : len - 1];
      v |= (o < len ? byte : 0u) << (8 * b);
    }
    word = v;
  }
  // renormalisation after a pop of this row (as ByteStage::renorm): the window
  // is moved first where it would not hold pos + 1
  NXD void renorm(bool act, int p, int g) {
    const bool need = pos + 2u > base + 64u && pos < len;
    if (__ballot(need) != 0ull) {
      if (need) fill(pos & ~3u, p);
    }
    // bytes pos and pos + 1 (off <= 62 here): the two window words from
    // off / 4 on, then the byte pair at off % 4 of their concatenation
    const uint32_t off = pos - base;
    const uint32_t wi = off >> 2;
    const uint32_t w0 = (uint32_t)__shfl((int)word, (g << 4) | (int)(wi & 15u));
    const uint32_t w1 = (uint32_t)__shfl((int)word, (g << 4) | (int)((wi + 1u) & 15u));
    const uint32_t two = __builtin_amdgcn_alignbyte(w1, w0, off & 3u);
    const uint32_t b0 = two & 255u, b1 = (two >> 8) & 255u;
    const bool r0 = act && x < RANS_L && pos < len;
    x = r0 ? ((x << 8) | b0) : x;
    pos += r0 ? 1u : 0u;
    const bool r1 = act && x < RANS_L && pos < len;
    x = r1 ? ((x << 8) | b1) : x;
    pos += r1 ? 1u : 0u;
  }
};

// One symbol of every pixel of a 16-row group, each from the pixel's own
// stream, all pixels at once: eight halvings of [0, 256], each the encoder's
// evaluation of the quantised CDF (cdf_eval, all lanes of a pixel in step),
// keeping the bracket's CDF values, so (start, freq) are bitwise the
// encoder's. Pixels with act pop (state and position updated); the stream's
// next two bytes are loaded before the search (clamped into the stream,
// used only while bytes remain). Every lane must call it (lane-group sums).
NXD int pop_own(const Chan& Q, PixStream& P, bool act, uint32_t& start, uint32_t& freq) {
  const uint32_t lm = P.len - 1u;
  const uint32_t nb0 = P.S[min(P.pos, lm)];
  const uint32_t nb1 = P.S[min(P.pos + 1u, lm)];
  // a state below 2^16 (the end of the stream) holds a spread slot
  const bool small = P.x < CDF_TOTAL;
  const uint32_t slot = small ? rev16(P.x) : (P.x & 0xffffu);
  // the bracket [lo, lo + 2^(8 - it)) halves at every step: its midpoint is
  // lo plus a constant, and only its CDF values need keeping
  int lo = 0;
  uint32_t clo = 0u, chi = CDF_TOTAL;
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int mid = lo + (128 >> it);
    const uint32_t v = cdf_quant(mid, cdf_eval(mid, Q.w, Q.a, Q.b));
    const bool le = v <= slot;
    lo = le ? mid : lo;
    clo = le ? v : clo;
    chi = le ? chi : v;
  }
  freq = chi - clo;
  start = clo;
  uint32_t xn = freq * (P.x >> 16) + slot - clo;
  if (__ballot(small && act) != 0ull) {  // rare: a stream's last few pops
    const uint32_t xr = spread_rank(P.x, clo, freq);
    xn = small ? xr : xn;
  }
  uint32_t pn = P.pos;
  const bool r0 = xn < RANS_L && pn < P.len;
  xn = r0 ? ((xn << 8) | nb0) : xn;
  pn += r0 ? 1u : 0u;
  const bool r1 = xn < RANS_L && pn < P.len;
  xn = r1 ? ((xn << 8) | nb1) : xn;
  pn += r1 ? 1u : 0u;
  P.x = act ? xn : P.x;
  P.pos = act ? pn : P.pos;
  return lo;
}

// K: rANS streams of the lane; the chain pops K symbols (rows ts + q0 + k,
// streams k) per iteration, their searches independent of each other;
// K >= 8: every row of a group pops from its own stream at once, found by a
// bisection of the quantised CDF over the whole group.
// SAMPLE: ancestral sampling instead of decoding (no container): each
// symbol is the inverse quantised CDF at its Philox slot, found by bisection
// for all rows of a group at once (their slots do not depend on each other).
// SHEAR: the sheared layout (order 2): contexts from the wave's window of the
// lane's sheared canvas instead of the output image.
template <int H_, int C_, int K, bool SAMPLE, bool SHEAR>
__device__ void decode_lane(const DecArgs& A, const float* w, uint32_t* piv, int64_t L, int lane) {
  static_assert(!SAMPLE || K == 4, "sampling is instantiated once, as K = 4");
  const int p = lane & 15, g = lane >> 4;
  const bool has2 = g < 2;
  const int n = find_img_uniform(A.desc, A.n_img, L);
  const ImgDesc D = uniform_desc(A.desc + n);
  const int q = (int)(L - D.lane_base);
  const int nl = D.nlx * D.nly;
  const int ly = q / D.nlx, lx = q - ly * D.nlx;
  const int y0 = ly * D.ph, x0 = lx * D.pw;
  const int Hl = min(D.ph, D.H - y0), Wl = min(D.pw, D.W - x0);
  const uint8_t* C = nullptr;
  int64_t clen = 0, pay = 0;
  // header and stream table checks (every lane reads the same bytes; the
  // verdicts are made wave-uniform, and status is stored by every lane)
  bool ok = true;
  bool mismatch = false;
  if constexpr (!SAMPLE) {
  C = A.in + uniform64((int64_t)A.in_off[n]);
  clen = uniform64((int64_t)(A.in_off[n + 1] - A.in_off[n]));
  pay = HDR_BYTES + 4 * (int64_t)nl * K;
  ok = clen >= pay;
  if (ok) {
    const uint32_t ph = D.ph == D.H ? 0u : (uint32_t)D.ph, pw = D.pw == D.W ? 0u : (uint32_t)D.pw;
    ok = C[0] == 'N' && C[1] == 'L' && C[2] == 'X' && C[3] == 'C' && C[4] == CONTAINER_VERSION &&
         C[5] == (uint8_t)(A.order == 0 ? 0 : 1) && C[6] == (uint8_t)H_ && C[7] == (uint8_t)K && rd_u32(C + 8) == (uint32_t)D.H &&
         rd_u32(C + 12) == (uint32_t)D.W && (uint32_t)(C[16] | (C[17] << 8)) == ph &&
         (uint32_t)(C[18] | (C[19] << 8)) == pw && rd_u32(C + 28) == (uint32_t)nl;
    // the streams fill the container exactly: the last end is its payload
    ok = ok && pay + (int64_t)rd_u32(C + HDR_BYTES + 4 * ((int64_t)nl * K - 1)) == clen;
    ok = uniform(ok ? 1 : 0) != 0;
    if (ok) {
      const uint64_t hsh = (uint64_t)rd_u32(C + 20) | ((uint64_t)rd_u32(C + 24) << 32);
      mismatch = uniform(hsh != A.model_hash ? 1 : 0) != 0;
    }
  }
  }  // !SAMPLE
  if (mismatch) {
    A.status[n] = ST_MISMATCH;
    return;
  }
  // K <= 2: the streams' states are scalar (one search after another);
  // K = 4: one stream per 16-lane row, its state held by the row;
  // K >= 8: one stream per pixel (per pair of pixels for K = 8)
  constexpr int KS = K <= 2 ? K : 1;
  ByteStage R[KS];
  uint32_t x[KS], pos[KS];
  RowStream RS;
  PixStream PS;
  if constexpr (SAMPLE) {
  } else if constexpr (K >= 8) {
    const int64_t e = (int64_t)q * K + (p & (K - 1));  // stream table entry of this pixel row
    uint32_t lend = 0, lstart = 0;
    bool okr = ok;
    if (ok) {
      lend = rd_u32(C + HDR_BYTES + 4 * e);
      lstart = e > 0 ? rd_u32(C + HDR_BYTES + 4 * (e - 1)) : 0u;
      okr = lstart <= lend && pay + (int64_t)lend <= clen && lend - lstart >= 1;
    }
    ok = __ballot(okr) == ~0ull;
    PS.S = as_global(C + pay + lstart);
    PS.len = lend - lstart;
  } else if constexpr (K == 4) {
    const int64_t e = (int64_t)q * K + g;  // stream table entry of this row
    uint32_t lend = 0, lstart = 0;
    bool okr = ok;
    if (ok) {
      lend = rd_u32(C + HDR_BYTES + 4 * e);
      lstart = e > 0 ? rd_u32(C + HDR_BYTES + 4 * (e - 1)) : 0u;
      okr = lstart <= lend && pay + (int64_t)lend <= clen && lend - lstart >= 1;
    }
    ok = __ballot(okr) == ~0ull;
    RS.S = C + pay + lstart;
    RS.len = lend - lstart;
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t e = (int64_t)q * K + k;  // stream table entry
      uint32_t lend = 0, lstart = 0;
      if (ok) {
        lend = (uint32_t)uniform((int)rd_u32(C + HDR_BYTES + 4 * e));
        lstart = e > 0 ? (uint32_t)uniform((int)rd_u32(C + HDR_BYTES + 4 * (e - 1))) : 0u;
        ok = lstart <= lend && pay + (int64_t)lend <= clen && lend - lstart >= 1;
      }
      R[k].S = C + pay + lstart;
      R[k].len = lend - lstart;
    }
  }
  if (!ok) {
    A.status[n] = ST_CORRUPT;
    return;
  }
  if constexpr (SAMPLE) {
  } else if constexpr (K >= 8) {
    stream_begin(PS);
  } else if constexpr (K == 4) {
    // the initial state: the stream's first bytes, most significant first,
    // read while x < L (at most four)
    RS.fill(0, p);
    const uint32_t w0 = (uint32_t)__shfl((int)RS.word, g << 4);  // bytes 0..3
    uint32_t xs = 0u, ps = 0u;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const bool rd = xs < RANS_L && ps < RS.len;
      xs = rd ? ((xs << 8) | ((w0 >> (8 * b)) & 255u)) : xs;
      ps += rd ? 1u : 0u;
    }
    RS.x = xs;
    RS.pos = ps;
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      R[k].fill(0, lane);
      uint32_t xs = 0u, ps = 0u;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const bool rd = xs < RANS_L && ps < R[k].len;
        xs = rd ? ((xs << 8) | R[k].byte_at((uint32_t)b)) : xs;
        ps += rd ? 1u : 0u;
      }
      x[k] = xs;
      pos[k] = ps;
    }
  }
  float* prm = (float*)(piv + PIV_WORDS);
  uint8_t* img = D.px;
  const int o = H_ + 1;
  const bool raster = A.order == 0;
  // sheared layout: this wave's window of the lane's sheared canvas, cleared
  // (its h top rows stay 0: the padding above the lane)
  constexpr bool shear = SHEAR;
  const int rows = A.ring_rows;
  int16_t* ring = nullptr;
  if constexpr (shear) {
    // workgroups are dealt to the XCDs in turn: the windows of one XCD's
    // waves are kept contiguous, so they spread over its L2 sets
    const int nwv = (int)(blockDim.x >> 6);
    const int xcd_blocks = (int)((gridDim.x + RING_XCDS - 1) / RING_XCDS);
    const int slot = (int)(blockIdx.x % RING_XCDS) * xcd_blocks + (int)(blockIdx.x / RING_XCDS);
    const int wave = uniform(slot * nwv + (int)(threadIdx.x >> 6));
    ring = (int16_t*)(A.ring + (int64_t)wave * ring_wave_bytes(rows));
    uint32_t* r32 = (uint32_t*)ring;
    const int nw = (int)(ring_wave_bytes(rows) >> 2);
    for (int k = lane; k < nw; k += 64) r32[k] = 0u;
    __threadfence_block();
  }
  const int64_t ngroups = raster ? (int64_t)Hl * Wl : (int64_t)Wl + (int64_t)o * (Hl - 1);
  uint32_t* dump = A.sym_dump ? A.sym_dump + D.px_base * 3 : nullptr;
  TapCodes<H_> tc;
  tc.init(g);

  for (int64_t gi = 0; gi < ngroups; ++gi) {
    int ilo, ihi;
    if (raster) {
      ilo = ihi = (int)(gi / Wl);
    } else {
      step_rows((int)gi, Hl, Wl, o, ilo, ihi);
    }
    if constexpr (shear) {
      // column gi of the window: the step's rows [ilo, ihi] are written as
      // they decode; of the other rows (no pixel at this column) only those
      // a later read can reach are cleared: a pixel of step t' in (gi, gi +
      // h(h+2)] reads rows i - h .. i with ilo(gi) <= ilo(t') <= i <=
      // ihi(t') <= ihi(gi) + h + 1, so rows [ilo - h, ihi + h + 1] (at most
      // 2h + 1 of them besides the step's); the rest are never read before
      // the column is rewritten 16 steps later
      int16_t* cb = ring + (int64_t)(gi & (RING_COLS - 1)) * 3 * rows + H_;
      const int r = (ilo <= ihi ? (lane < H_ ? ilo - H_ + lane : ihi + 1 + (lane - H_))
                                : ilo - H_ + lane);
      const int nz = ilo <= ihi ? 2 * H_ + 1 : 2 * H_ + 1 + (ihi + 1 - ilo);
      if (lane < nz && r >= 0 && r < Hl) {
        cb[r] = 0;
        cb[rows + r] = 0;
        cb[2 * rows + r] = 0;
      }
      __threadfence_block();
    }
    for (int ts = ilo; ts <= ihi; ts += 16) {
      const int na = min(16, ihi - ts + 1);
      const int i = ts + p;
      const bool active = p < na;
      const int j = raster ? (int)(gi - (int64_t)ilo * Wl) : (int)gi - o * i;
      // sampling: the slots of pixel p (every lane group draws the same)
      uint32_t sl[3] = {0u, 0u, 0u};
      if constexpr (SAMPLE) sample_slots(D.seed, D.W, y0 + i, x0 + j, sl);
      f4 head[HEAD_TILES];
      if (na <= A.quad_px) {
        // few pixels: eight, then four at a time (see net_quad), through a
        // head table in the wave's LDS
        float* hb = (float*)piv;
        int ql = lane;
        asm("" : "+v"(ql));  // (what follows from it is found here: kept through the loop, it would spill)
        auto quads = [&](auto nq, int q0) {
          constexpr int NQ = decltype(nq)::value;
          float cx[NQ][quad_inputs(H_)];
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            const int qi = min(ts + q0 + 4 * q + (ql & 3), Hl - 1);
            if constexpr (shear)
              quad_gather_ring<H_>(cx[q], ring, rows, (int)gi, qi, ql);
            else
              quad_gather_image<H_>(cx[q], img, D.W, y0, x0, Hl, Wl, qi, raster ? j : (int)gi - o * qi, ql);
          }
          net_quad<H_, C_, NQ>(lds_weights(w), A.nb, cx, hb + q0 * HB_STRIDE, ql);
        };
        int q0 = 0;
        for (; na - q0 > 4; q0 += 8) quads(std::integral_constant<int, 2>(), q0);
        if (q0 < na) quads(std::integral_constant<int, 1>(), q0);
        const float* hp = hb + min(p, na - 1) * HB_STRIDE + 4 * g;
#pragma unroll
        for (int mt = 0; mt < HEAD_TILES; ++mt) head[mt] = *(const f4*)(hp + 16 * mt);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
      } else {
        float ctx[conv_chunks(H_)];
        tc.refresh();
        if constexpr (shear)
          gather_ring<H_>(ctx, ring, rows, (int)gi, min(i, Hl - 1));
        else
          gather<H_>(ctx, tc, img, D.W, y0, x0, Hl, Wl, i, j, y0 + ts);
        net_forward<H_, C_>(lds_weights(w), A.nb, ctx, head, lane);
      }
      Mix M;
      mix_prep(head, M, has2);
      int xv[3] = {0, 0, 0};
      float xr = 0.0f, xg = 0.0f;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        Chan Q;
        chan_params(M, c, xr, xg, Q);
        if constexpr (SAMPLE) {
          // the v with cdf(v) <= slot < cdf(v + 1): eight halvings of
          // [0, 256] with cdf(0) = 0 <= slot < cdf(256) = 2^16 kept; the
          // evaluations are the encoder's (cdf_eval), so the draw is the
          // inverse of the coder's own row
          int lo = 0;
#pragma unroll
          for (int it = 0; it < 8; ++it) {
            const int mid = lo + (128 >> it);
            const bool le = cdf_quant(mid, cdf_eval(mid, Q.w, Q.a, Q.b)) <= sl[c];
            lo = le ? mid : lo;
          }
          if (c == 0) xv[0] = lo;
          else if (c == 1) xv[1] = lo;
          else xv[2] = lo;
        } else if constexpr (K >= 8) {
          // every pixel's symbol from its own stream (pop_own); K = 8 pops
          // rows 0..7, then rows 8..15
#pragma unroll
          for (int half = 0; half < 16 / K; ++half) {
            const int q0 = half * K;
            if (q0 >= na) break;
            const bool act = p >= q0 && p < q0 + K && p < na;
            uint32_t start, freq;
            const int sy = pop_own(Q, PS, act, start, freq);
            if (act) {
              if (c == 0) xv[0] = sy;
              else if (c == 1) xv[1] = sy;
              else xv[2] = sy;
            }
            if (dump && act && g == 0)
              dump[((int64_t)(y0 + i) * D.W + (x0 + j)) * 3 + c] = start | (freq << 16);
            if constexpr (K == 8) {
              // rows p and p + 8 share a stream: the other half takes the new state
              const uint32_t ox = (uint32_t)__shfl_xor((int)PS.x, 8);
              const uint32_t op = (uint32_t)__shfl_xor((int)PS.pos, 8);
              const bool mine = p >= q0 && p < q0 + K;
              PS.x = mine ? PS.x : ox;
              PS.pos = mine ? PS.pos : op;
            }
          }
        } else if constexpr (K == 4) {
          // stage the channel's mixtures: lane (p, g) holds components g + 4 j
          float* mine = prm + p * PRM_STRIDE;
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const int m = g + 4 * j;
            mine[3 * m] = Q.w[j];
            mine[3 * m + 1] = Q.a[j];
            mine[3 * m + 2] = Q.b[j];
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          // pops: row g takes row ts + q0 + g of the group (stream g); lane p
          // of the row first evaluates pivot p of that pixel, the cdf at
          // k = 16 (p + 1) (p = 15 stands for k = 256): it does not depend on
          // the coder state, and only the rows that are popped are evaluated
          for (int q0 = 0; q0 < na; q0 += 4) {
            const int pr = q0 + g;
            const bool act = pr < na;
            const int prc = min(pr, 15);
            Mix10 P;
            load_mix10(P, prm, prc);
            const int kp = min(16 * (p + 1), 255);
            const uint32_t pq = cdf_quant(kp, cdf_eval10(kp, P));
            const uint32_t pv = p < 15 ? pq : CDF_TOTAL;
            // a state below 2^16 (the end of the stream) holds a spread slot:
            // the symbol is searched with its reversal
            const bool small = RS.x < CDF_TOTAL;
            const uint32_t slot = small ? rev16(RS.x) : (RS.x & 0xffffu);
            const int b = row_count(__ballot(pv <= slot), g);
            const int k2 = 16 * b + p;
            const uint32_t c2 = cdf_quant(k2, cdf_eval10(max(k2, 1), P));
            const int cnt = row_count(__ballot(c2 <= slot) & 0xfffefffefffefffeull, g);
            const int sy = 16 * b + cnt;
            const int rb = g << 4;
            // start = cdf(16 b + cnt): lane cnt's value, lane 0's being the
            // bucket's lower edge cdf(16 b) (the same evaluation as pivot
            // b - 1), except cdf(0) = 0; end = cdf(16 b + cnt + 1): lane
            // cnt + 1's value, or the bucket's upper edge, pivot b
            const uint32_t st_r = (uint32_t)__shfl((int)c2, rb | cnt);
            const uint32_t nc_r = (uint32_t)__shfl((int)c2, rb | ((cnt + 1) & 15));
            const uint32_t np_r = (uint32_t)__shfl((int)pv, rb | b);
            const uint32_t start = (b == 0 && cnt == 0) ? 0u : st_r;
            const uint32_t freq = (cnt < 15 ? nc_r : np_r) - start;
            uint32_t xn = freq * (RS.x >> 16) + slot - start;
            if (__ballot(small && act) != 0ull) {  // rare: a stream's last few pops
              const uint32_t xr = spread_rank(RS.x, start, freq);
              xn = small ? xr : xn;
            }
            RS.x = act ? xn : RS.x;
            RS.renorm(act, p, g);
            // the symbol of pixel p (decoded by row p - q0) to all its lanes
            const int src = p - q0;
            const int sv = __shfl(sy, (src & 3) << 4);
            if (src >= 0 && src < 4) {
              if (c == 0) xv[0] = sv;
              else if (c == 1) xv[1] = sv;
              else xv[2] = sv;
            }
            if (dump && act && p == 0) {
              const int ii = ts + pr;
              const int jj = raster ? (int)(gi - (int64_t)ilo * Wl) : (int)gi - o * ii;
              dump[((int64_t)(y0 + ii) * D.W + (x0 + jj)) * 3 + c] = start | (freq << 16);
            }
          }
        } else {
        // pivot CDF values of every pixel of the group: cdf at k = 16 (j + 1),
        // j = 0..14, and 2^16 for k = 256 (independent evaluations)
#pragma unroll 5
        for (int jp = 0; jp < 15; ++jp) {
          const uint32_t v = cdf_quant(16 * (jp + 1), cdf_eval(16 * (jp + 1), Q.w, Q.a, Q.b));
          if (g == 0) piv[p * 16 + jp] = v;
        }
        if (g == 0) piv[p * 16 + 15] = CDF_TOTAL;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // pops, K per iteration (one per stream); the next iteration's pivot
        // rows and mixtures (which do not depend on the coder states) are
        // fetched one iteration ahead; rows past the group are clamped and
        // their results unused
        float nw[K][3], nA[K][3], nB[K][3];
        uint32_t npv[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const int src = (g << 4) | k;
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            nw[k][j] = __shfl(Q.w[j], src);
            nA[k][j] = __shfl(Q.a[j], src);
            nB[k][j] = __shfl(Q.b[j], src);
          }
          npv[k] = piv[k * 16 + p];
        }
        for (int q0 = 0; q0 < na; q0 += K) {
          float bw[K][3], bA[K][3], bB[K][3];
          uint32_t pv[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              bw[k][j] = nw[k][j];
              bA[k][j] = nA[k][j];
              bB[k][j] = nB[k][j];
            }
            pv[k] = npv[k];
            const int nx = min(q0 + K + k, 15);
            const int src = (g << 4) | nx;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              nw[k][j] = __shfl(Q.w[j], src);
              nA[k][j] = __shfl(Q.a[j], src);
              nB[k][j] = __shfl(Q.b[j], src);
            }
            npv[k] = piv[nx * 16 + p];
          }
          uint32_t slot[K], start[K], freq[K];
          int sym[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            slot[k] = x[k] < CDF_TOTAL ? rev16(x[k]) : (x[k] & 0xffffu);  // spread slot below 2^16
            // bucket: pivots of the pixel at or below the slot (pv of lane p =
            // cdf at 16 (p + 1); lane 15 holds 2^16, so b <= 15)
            const int b = __popcll(__ballot(pv[k] <= slot[k]) & 0xffffull);
            // inside the bucket: cdf at k = 16 b + p for p = 1..15; the
            // bucket's lower bound (p = 0) is cdf at 16 b <= slot
            const int k2 = 16 * b + p;
            const uint32_t c2 = cdf_quant(k2, cdf_eval(max(k2, 1), bw[k], bA[k], bB[k]));
            const int cnt = __popcll(__ballot(c2 <= slot[k]) & 0xfffeull);
            sym[k] = 16 * b + cnt;
            // bounds of the symbol, every read unconditional (no branches)
            const uint32_t lo_r = (uint32_t)__builtin_amdgcn_readlane((int)pv[k], (b + 15) & 15);
            const uint32_t st_r = (uint32_t)__builtin_amdgcn_readlane((int)c2, cnt);
            const uint32_t nc_r = (uint32_t)__builtin_amdgcn_readlane((int)c2, (cnt + 1) & 15);
            const uint32_t np_r = (uint32_t)__builtin_amdgcn_readlane((int)pv[k], b);
            const uint32_t lo = b == 0 ? 0u : lo_r;
            start[k] = cnt == 0 ? lo : st_r;
            freq[k] = (cnt < 15 ? nc_r : np_r) - start[k];
          }
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const bool act = q0 + k < na;
            uint32_t xn = freq[k] * (x[k] >> 16) + slot[k] - start[k];
            if (x[k] < CDF_TOTAL) xn = spread_rank(x[k], start[k], freq[k]);  // wave-uniform
            x[k] = act ? xn : x[k];
            R[k].renorm(x[k], pos[k], lane, act);
            if (p == q0 + k) {
              if (c == 0) xv[0] = sym[k];
              else if (c == 1) xv[1] = sym[k];
              else xv[2] = sym[k];
            }
            if (dump && act) {  // every lane stores the same value
              const int ii = ts + q0 + k;
              const int jj = raster ? (int)(gi - (int64_t)ilo * Wl) : (int)gi - o * ii;
              dump[((int64_t)(y0 + ii) * D.W + (x0 + jj)) * 3 + c] = start[k] | (freq[k] << 16);
            }
          }
        }
        }  // K < 4
        if (c == 0) {
          posterior(M, xv[0], Q.mu, Q.is, has2);
          xr = normalise(xv[0]);
        } else if (c == 1) {
          posterior(M, xv[1], Q.mu, Q.is, has2);
          xg = normalise(xv[1]);
        }
      }
      if (active && g == 0) {
        uint8_t* dst = img + ((int64_t)(y0 + i) * D.W + (x0 + j)) * 3;
        dst[0] = (uint8_t)xv[0];
        dst[1] = (uint8_t)xv[1];
        dst[2] = (uint8_t)xv[2];
        if constexpr (shear) {
          int16_t* cb = ring + (int64_t)(gi & (RING_COLS - 1)) * 3 * rows + H_ + i;
          cb[0] = (int16_t)(2 * xv[0] - 255);
          cb[rows] = (int16_t)(2 * xv[1] - 255);
          cb[2 * rows] = (int16_t)(2 * xv[2] - 255);
        }
      }
      // make this group's pixels visible to the wave's later gathers
      __threadfence_block();
    }
  }
  bool clean = true;
  if constexpr (SAMPLE) {
  } else if constexpr (K >= 8) {
    clean = __ballot(PS.x == RANS_X0 && PS.pos == PS.len) == ~0ull;
  } else if constexpr (K == 4) {
    clean = __ballot(RS.x == RANS_X0 && RS.pos == RS.len) == ~0ull;
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) clean = clean && x[k] == RANS_X0 && pos[k] == R[k].len;
  }
  if (!clean) A.status[n] = ST_CORRUPT;
}

template <int H_, int C_, int K, bool SAMPLE, bool SHEAR>
__global__ void __launch_bounds__(NWAVES_DEC * 64) k_decode(DecArgs A) {
  extern __shared__ float4 smem_f4[];
  float* w = (float*)smem_f4;
  load_weights(w, A.w, A.wfloats);
  const int lane = threadIdx.x & 63;
  uint32_t* piv = (uint32_t*)(w + A.wfloats) + (threadIdx.x >> 6) * A.wave_words;
  for (;;) {
    // one queue pop per wave, by its first active lane, broadcast
    const int leader = uniform(lane);
    int L = 0;
    if (lane == leader) L = atomicAdd(A.counter, 1);
    L = uniform(L);
    if ((int64_t)L >= A.n_lanes) break;
    decode_lane<H_, C_, K, SAMPLE, SHEAR>(A, w, piv, L, lane);
  }
}

__global__ void k_decode_prep(int32_t* status, int n_img, int32_t* counter, int32_t* progress, int64_t n_bands) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (status && i < n_img) status[i] = ST_OK;
  if (progress && i < n_bands) progress[i] = 0;
  if (i == 0) *counter = 0;
}

// per image: sum of per-pixel bits in double, in a fixed order: block (n, r)
// sums part r of image n (thread-strided partial sums, then a fixed tree),
// then one thread per image adds the REDUCE_PARTS partials in order
__global__ void __launch_bounds__(256) k_reduce_bits(const ImgDesc* desc, const float* bits, double* part_out) {
  __shared__ double part[256];
  const ImgDesc D = desc[blockIdx.x];
  const int64_t npx = (int64_t)D.H * D.W;
  const int64_t per = (npx + REDUCE_PARTS - 1) / REDUCE_PARTS;
  const int64_t lo = (int64_t)blockIdx.y * per, hi = lo + per < npx ? lo + per : npx;
  double s = 0.0;
  for (int64_t k = lo + threadIdx.x; k < hi; k += 256) s += (double)bits[D.px_base + k];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part_out[(int64_t)blockIdx.x * REDUCE_PARTS + blockIdx.y] = part[0];
}

__global__ void k_reduce_final(const double* part, int n_img, double* out) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= n_img) return;
  double s = 0.0;
  for (int r = 0; r < REDUCE_PARTS; ++r) s += part[(int64_t)n * REDUCE_PARTS + r];
  out[n] = s;
}

// ------------------------------------------------------------------ monotonicity check
// The quantised CDF is monotone in k (every frequency >= 1) only if the
// hardware exp2 is non-decreasing and the reciprocal non-increasing on the
// arguments cdf_eval gives them. This scans every finite FP32 value in
// increasing order, a chunk of consecutive values per thread, and counts
// adjacent pairs that break the order: out[0] exp2 on all finite inputs,
// out[1] rcp on [1, FLT_MAX], out[2] rcp(1 + exp2(z)) (non-increasing in z) on
// all finite z, out[3] pairs checked.
constexpr uint32_t MONO_NEG = 0x7F800000u;  // finite negative bit patterns (-FLT_MAX .. -0)
constexpr uint64_t MONO_ALL = 2ull * MONO_NEG;
constexpr uint32_t MONO_CHUNK = 4096;

NXD float mono_value(uint64_t i) {  // i-th finite float in increasing order
  const uint32_t b = i < MONO_NEG ? 0xFF7FFFFFu - (uint32_t)i : (uint32_t)(i - MONO_NEG);
  return __uint_as_float(b);
}

__global__ void __launch_bounds__(256) k_check_monotone(unsigned long long* out) {
  const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const uint64_t lo = t * MONO_CHUNK;
  unsigned long long bad_exp = 0, bad_rcp = 0, bad_sig = 0, pairs = 0;
  if (lo < MONO_ALL) {
    const uint64_t hi = lo + MONO_CHUNK < MONO_ALL ? lo + MONO_CHUNK : MONO_ALL;
    const uint64_t first = lo > 0 ? lo - 1 : 0;
    float z = mono_value(first);
    float pe = __builtin_amdgcn_exp2f(z);
    float ps = __builtin_amdgcn_rcpf(1.0f + pe);
    float pr = __builtin_amdgcn_rcpf(z);
    for (uint64_t i = first + 1; i < hi; ++i) {
      z = mono_value(i);
      const float e = __builtin_amdgcn_exp2f(z);
      const float sg = __builtin_amdgcn_rcpf(1.0f + e);
      const float r = __builtin_amdgcn_rcpf(z);
      bad_exp += e < pe ? 1 : 0;
      bad_sig += sg > ps ? 1 : 0;
      // rcp on [1, FLT_MAX]: both values of the pair at or above 1
      bad_rcp += (mono_value(i - 1) >= 1.0f && r > pr) ? 1 : 0;
      ++pairs;
      pe = e;
      ps = sg;
      pr = r;
    }
  }
  if (bad_exp) atomicAdd(out + 0, bad_exp);
  if (bad_rcp) atomicAdd(out + 1, bad_rcp);
  if (bad_sig) atomicAdd(out + 2, bad_sig);
  if (pairs) atomicAdd(out + 3, pairs);
}

__global__ void k_zero4(unsigned long long* out) {
  if (threadIdx.x < 4) out[threadIdx.x] = 0;
}

// ------------------------------------------------------------------ host launchers
bool supported(int h, int C) {
  return (h == 3 && (C == 16 || C == 32 || C == 64)) || (h == 2 && (C == 16 || C == 32 || C == 64)) ||
         (h == 1 && (C == 16 || C == 32));
}

template <int H_, int C_>
static hipError_t pass_t(const PassArgs& a, int grid, hipStream_t s) {
  const size_t lds = (size_t)a.wfloats * 4;
  hipError_t e = allow_lds(k_pass<H_, C_>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_pass<H_, C_>), dim3(grid), dim3(NWAVES * 64), lds, s, a);
  return hipGetLastError();
}

// A wave's LDS: pivot and mixture tables, or a head table of as many pixels
// (a multiple of 4, at most quad_limit) as the LDS left by the weights gives
// each wave. Groups of at most that many pixels take net_quad.
template <int H_, int C_, int K, bool SAMPLE = false>
static hipError_t decode_tt(const DecArgs& args, int grid, int waves, size_t lim, hipStream_t s) {
  DecArgs a = args;
  const int64_t left = ((int64_t)lim / 4 - a.wfloats) / waves;
  a.quad_px = (int)std::min<int64_t>(quad_limit(C_, a.nb), left / HB_STRIDE / 4 * 4);
  a.wave_words = std::max(WAVE_LDS_WORDS, a.quad_px * HB_STRIDE);
  const size_t lds = ((size_t)a.wfloats + (size_t)waves * a.wave_words) * 4;
  if (a.order == 2)
    hipLaunchKernelGGL((k_decode<H_, C_, K, SAMPLE, true>), dim3(grid), dim3(waves * 64), lds, s, a);
  else
    hipLaunchKernelGGL((k_decode<H_, C_, K, SAMPLE, false>), dim3(grid), dim3(waves * 64), lds, s, a);
  return hipGetLastError();
}

// the decoder's dynamic LDS limit, raised to the device maximum by every
// prepare call (not a stream operation: kept out of the launch path, which a
// caller may capture)
template <int H_, int C_, int K>
static hipError_t decode_setup_k() {
  int dev = 0, lim = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&lim, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  for (int sh = 0; sh < 2 && e == hipSuccess; ++sh) {
    if (e == hipSuccess) e = allow_lds(sh ? k_decode<H_, C_, K, false, true> : k_decode<H_, C_, K, false, false>, (size_t)lim);
    if (K == 4 && e == hipSuccess)
      e = allow_lds(sh ? k_decode<H_, C_, 4, true, true> : k_decode<H_, C_, 4, true, false>, (size_t)lim);
  }
  return e;
}

template <int H_, int C_>
static hipError_t decode_setup(int K) {
  if (K == 2) return decode_setup_k<H_, C_, 2>();
  if (K == 4) return decode_setup_k<H_, C_, 4>();
  if (K == 8) return decode_setup_k<H_, C_, 8>();
  if (K == 16) return decode_setup_k<H_, C_, 16>();
  return decode_setup_k<H_, C_, 1>();
}

template <int H_, int C_>
static hipError_t sample_t(const DecArgs& a, int grid, int waves, size_t lim, hipStream_t s) {
  return decode_tt<H_, C_, 4, true>(a, grid, waves, lim, s);
}

template <int H_, int C_>
static hipError_t decode_t(const DecArgs& a, int grid, int waves, size_t lim, hipStream_t s) {
  if (a.K == 2) return decode_tt<H_, C_, 2>(a, grid, waves, lim, s);
  if (a.K == 4) return decode_tt<H_, C_, 4>(a, grid, waves, lim, s);
  if (a.K == 8) return decode_tt<H_, C_, 8>(a, grid, waves, lim, s);
  if (a.K == 16) return decode_tt<H_, C_, 16>(a, grid, waves, lim, s);
  return decode_tt<H_, C_, 1>(a, grid, waves, lim, s);
}

hipError_t launch_pass(int h, int C, const PassArgs& a, int grid, hipStream_t s) {
  if (a.n_tiles == 0) return hipSuccess;
  NX_DISPATCH(pass_t, h, C, a, grid, s);
}

hipError_t prepare_decode(int h, int C, int K) { NX_DISPATCH(decode_setup, h, C, K); }

hipError_t launch_decode(int h, int C, const DecArgs& a, int grid, int waves, size_t lim, hipStream_t s) {
  if (a.n_lanes == 0) return hipSuccess;
  if (waves < 1 || waves > NWAVES_DEC) return hipErrorInvalidValue;
  NX_DISPATCH(decode_t, h, C, a, grid, waves, lim, s);
}

hipError_t launch_sample(int h, int C, const DecArgs& a, int grid, int waves, size_t lim, hipStream_t s) {
  if (a.n_lanes == 0) return hipSuccess;
  if (waves < 1 || waves > NWAVES_DEC) return hipErrorInvalidValue;
  NX_DISPATCH(sample_t, h, C, a, grid, waves, lim, s);
}

template <int O, int K>
static void launch_layout(const RansEncArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_rans_counts<O, K>), dim3((unsigned)(a.n_lanes * K)), dim3(64), 0, s, a);
  const unsigned chunks =
      (unsigned)std::max<int64_t>(1, std::min<int64_t>((a.max_lane_px + SCATTER_PX - 1) / SCATTER_PX, 65535));
  hipLaunchKernelGGL((k_rans_scatter<O, K>), dim3((unsigned)a.n_lanes, chunks), dim3(256), 0, s, a);
}

hipError_t launch_rans_encode(const RansEncArgs& a, hipStream_t s) {
  if (a.n_lanes == 0) return hipSuccess;
  if (a.K == ROW_STREAMS) {
    if (a.wave_per_stream)
      hipLaunchKernelGGL(k_rans_enc_wave<true>, dim3((unsigned)a.n_streams), dim3(64), 0, s, a);
    else
      hipLaunchKernelGGL(k_rans_enc_rows, dim3((unsigned)((a.n_streams + 63) / 64)), dim3(64), 0, s, a);
    return hipGetLastError();
  }
  if (a.h < 1 || a.h > 3 || !valid_interleave(a.K)) return hipErrorInvalidValue;
  const int kx = a.K == 1 ? 0 : a.K == 2 ? 1 : a.K == 4 ? 2 : a.K == 8 ? 3 : 4;
  switch (5 * (a.h - 1) + kx) {
    case 0: launch_layout<2, 1>(a, s); break;
    case 1: launch_layout<2, 2>(a, s); break;
    case 2: launch_layout<2, 4>(a, s); break;
    case 3: launch_layout<2, 8>(a, s); break;
    case 4: launch_layout<2, 16>(a, s); break;
    case 5: launch_layout<3, 1>(a, s); break;
    case 6: launch_layout<3, 2>(a, s); break;
    case 7: launch_layout<3, 4>(a, s); break;
    case 8: launch_layout<3, 8>(a, s); break;
    case 9: launch_layout<3, 16>(a, s); break;
    case 10: launch_layout<4, 1>(a, s); break;
    case 11: launch_layout<4, 2>(a, s); break;
    case 12: launch_layout<4, 4>(a, s); break;
    case 13: launch_layout<4, 8>(a, s); break;
    default: launch_layout<4, 16>(a, s); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.wave_per_stream)
    hipLaunchKernelGGL(k_rans_enc_wave<false>, dim3((unsigned)a.n_streams), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL(k_rans_enc, dim3((unsigned)((a.n_streams + 63) / 64)), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_pack(const PackArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_lane_scan, dim3(a.n_img), dim3(SCAN_THREADS), 0, s, a);
  hipLaunchKernelGGL(k_img_scan, dim3(1), dim3(64), 0, s, a);
  if (a.n_streams > 0) {
    // parts of a stream of the estimated length; a longer one (up to two bytes
    // a symbol) has its blocks take more than one part each
    const int64_t parts = (a.max_stream_bytes + PACK_PART - 1) / PACK_PART;
    hipLaunchKernelGGL(k_pack, dim3((unsigned)a.n_streams, (unsigned)std::max<int64_t>(1, std::min<int64_t>(parts, 64))),
                       dim3(64), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_decode_prep(int32_t* status, int n_img, int32_t* counter, hipStream_t s, int32_t* progress,
                              int64_t n_bands) {
  const int64_t items = std::max<int64_t>(std::max<int64_t>(n_img, n_bands), 1);
  hipLaunchKernelGGL(k_decode_prep, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, status, n_img, counter,
                     progress, n_bands);
  return hipGetLastError();
}

hipError_t launch_reduce_bits(const ImgDesc* desc, int n_img, const float* bits, double* partials, double* out,
                              hipStream_t s) {
  if (n_img == 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_bits, dim3(n_img, REDUCE_PARTS), dim3(256), 0, s, desc, bits, partials);
  hipLaunchKernelGGL(k_reduce_final, dim3((n_img + 63) / 64), dim3(64), 0, s, partials, n_img, out);
  return hipGetLastError();
}

}  // namespace nx

namespace nx {
// Scratch of the no-allocation decoder: a file-scope device array that every
// GPU the library runs on holds until the process ends. In host code its name
// is only a stand-in; the device address of each GPU's copy is looked up once
// per device (with that device current) and kept.
static __device__ __align__(256) uint8_t scratch[STATIC_SCRATCH_BYTES];

hipError_t static_scratch(void** ptr) {
  static std::mutex mu;
  static void* addr[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_check_monotone(unsigned long long* out, hipStream_t s) {
  hipLaunchKernelGGL(k_zero4, dim3(1), dim3(64), 0, s, out);
  const uint64_t threads = (MONO_ALL + MONO_CHUNK - 1) / MONO_CHUNK;
  hipLaunchKernelGGL(k_check_monotone, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, out);
  return hipGetLastError();
}
}  // namespace nx
