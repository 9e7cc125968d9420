// nx_team.hip -- decoding with few lanes: a team of four waves, one per SIMD
// of a CU, decodes one lane (k_decode_team), or one band of a lane with a
// stream per row (k_decode_rows).
//
// A wave that decodes a lane alone spends 26 to 32 thousand cycles on a group
// of 16 pixels, most of them issuing instructions, while the other SIMDs of its CU
// idle if there is at most one lane per CU (or two). A team shares the group:
// a wave takes four of its pixels, from their contexts to their symbols, and the
// team meets once per group, when the context window has the new pixels.
//   network     on v_mfma_f32_4x4x1f32 (16 blocks), four pixels by 64
//               outputs an instruction (net_quad)
//   mixture     16 lanes per pixel, lane m holding component m
// Every value is computed by the operations, in the order, of the other
// decoders and of the encoder: bitwise theirs.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "nx_coder.hpp"
#include "nx_window.hpp"

namespace nx {

// ------------------------------------------------------------------ context window in LDS
// (its places: nx_window.hpp)
// What an input's place has besides the step and the pixel's row is the
// lane's for good.
template <int H_>
NXD void quad_offsets(int (&off)[quad_inputs(H_)], int rows, int lane) {
#pragma unroll
  for (int j = 0; j < quad_inputs(H_); ++j) off[j] = win_tap<H_>(rows, j, lane);
}
// contexts of the wave's pixels at step t, i the window row of the lane's
template <int H_>
NXD void quad_gather(float (&cx)[quad_inputs(H_)], const int (&off)[quad_inputs(H_)], const int16_t* win, int rows,
                     int t, int i) {
  const int16_t* b = win + win_origin<H_>(rows, t, i);
  int raw[quad_inputs(H_)];
#pragma unroll
  for (int j = 0; j < quad_inputs(H_); ++j) raw[j] = b[off[j]];
#pragma unroll
  for (int j = 0; j < quad_inputs(H_); ++j) cx[j] = (float)raw[j] * (1.0f / 255.0f);
}

// both copies of plane `plane` (of column t), row r
NXD void win_put(int16_t* win, int rows, int t, int ch, int r, int v) {
  int16_t* b = win + win_place(rows, t, ch, r);
  b[0] = (int16_t)v;
  b[win_copy(rows)] = (int16_t)v;
}

constexpr int TEAM_WAVES = ROW_WAVES;

// A barrier at the head of a loop whose end writes the window. The wait for a
// wave's LDS operations that __syncthreads() holds is not enough there: ROCm
// 7.2's compiler drops it where nothing is in flight on the way into the loop,
// and then the writes that come round the loop may still be in flight behind
// the barrier. This wait (lgkmcnt(0) alone) is an instruction of its own, which
// it keeps.
NXD void team_barrier() {
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __syncthreads();
}

// ------------------------------------------------------------------ mixture, 16 lanes per pixel
template <int M>
NXD float row_get(float v) {  // component M's value, in every lane of the row
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), DPP_BCAST0 + M, 0xf, 0xf, true));
}
template <int M = 0>
NXD void row_mix10(const Chan16& Q, Mix10& P) {
  P.w[M] = row_get<M>(Q.w);
  P.a[M] = row_get<M>(Q.a);
  P.b[M] = row_get<M>(Q.b);
  if constexpr (M + 1 < 10) row_mix10<M + 1>(Q, P);
}
template <int N>
NXD uint32_t row_ror(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + N, 0xf, 0xf, true);
}
NXD uint32_t row_umax(uint32_t v) {
  v = max(v, row_ror<8>(v));
  v = max(v, row_ror<4>(v));
  v = max(v, row_ror<2>(v));
  return max(v, row_ror<1>(v));
}
NXD uint32_t row_umin(uint32_t v) {
  v = min(v, row_ror<8>(v));
  v = min(v, row_ror<4>(v));
  v = min(v, row_ror<2>(v));
  return min(v, row_ror<1>(v));
}

// The quantised CDF's pivots of a row's pixel: lane m has cdf at 16 (m + 1),
// lane 15 the total (no coder state in it)
NXD uint32_t row_pivots(const Mix10& P, int m) {
  const int k = min(16 * (m + 1), 255);
  const uint32_t v = cdf_quant(k, cdf_eval10(k, P));
  return m < 15 ? v : CDF_TOTAL;
}
// The symbol of `slot` in each row (16 lanes, one pixel): the pivots give its
// bucket of 16, then lane m evaluates the CDF at the bucket's m-th edge, with
// all ten components; the bracketing values are a maximum and a minimum over
// the row, the CDF being increasing. Two dependent evaluations for a symbol,
// of 59 instructions, where a search by component (16 lanes adding their
// terms) takes four of three, 264 in all.
NXD int row_search(const Mix10& P, uint32_t pv, uint32_t slot, int m, int s, uint32_t& start, uint32_t& freq) {
  const int b = row_count(__ballot(pv <= slot), s);
  const int k2 = 16 * b + m;
  const uint32_t c2 = cdf_quant(k2, cdf_eval10(max(k2, 1), P));
  const bool le = c2 <= slot;
  const int cnt = row_count(__ballot(le) & 0xfffefffefffefffeull, s);
  // lane 0: the bucket's lower edge, at or below the slot (cdf(0) = 0)
  const uint32_t below = m == 0 ? (b == 0 ? 0u : c2) : (le ? c2 : 0u);
  const uint32_t above = min(m > 0 && !le ? c2 : CDF_TOTAL, pv > slot ? pv : CDF_TOTAL);
  start = row_umax(below);
  freq = row_umin(above) - start;
  return 16 * b + cnt;
}

// pops one symbol of each row whose act is set from its stream, held in the
// row's lanes
NXD int row_pop(const Mix10& P, uint32_t pv, PixStream& S, bool act, int m, int s, uint32_t& start, uint32_t& freq) {
  const uint32_t lm = S.len - 1u;
  const uint32_t nb0 = S.S[min(S.pos, lm)];
  const uint32_t nb1 = S.S[min(S.pos + 1u, lm)];
  const bool small = S.x < CDF_TOTAL;  // the end of the stream: a spread slot
  const uint32_t slot = small ? rev16(S.x) : (S.x & 0xffffu);
  const int sy = row_search(P, pv, slot, m, s, start, freq);
  uint32_t xn = freq * (S.x >> 16) + slot - start;
  if (__ballot(small && act) != 0ull) {
    const uint32_t xr = spread_rank(S.x, start, freq);
    xn = small ? xr : xn;
  }
  uint32_t pn = S.pos;
  const bool r0 = xn < RANS_L && pn < S.len;
  xn = r0 ? ((xn << 8) | nb0) : xn;
  pn += r0 ? 1u : 0u;
  const bool r1 = xn < RANS_L && pn < S.len;
  xn = r1 ? ((xn << 8) | nb1) : xn;
  pn += r1 ? 1u : 0u;
  S.x = act ? xn : S.x;
  S.pos = act ? pn : S.pos;
  return sy;
}

// ------------------------------------------------------------------ serial pops
// One, two or four streams per lane: the rows of a stream pop one after the
// other, on one wave (wave w: stream w), each search on all 64 lanes: lane
// (p, g) evaluates components g, g + 4, g + 8 at the bucket's edge p, the
// groups' sums added as in cdf_eval. The wave's state is wave-uniform.
// prm: [pixel][g][12] floats, (w, a, b) of the three components; piv: [pixel][16].
struct SerialStream {
  ByteStage R;
  uint32_t x, pos;
};
constexpr int SERIAL_PRM = 48, SERIAL_WORDS = 16 * SERIAL_PRM + 256;

NXD int serial_pop(SerialStream& S, const f4 (&q)[3], uint32_t pv, int lane, uint32_t& start, uint32_t& freq) {
  const int p = lane & 15;
  const uint32_t slot = S.x < CDF_TOTAL ? rev16(S.x) : (S.x & 0xffffu);
  const int b = __popcll(__ballot(pv <= slot) & 0xffffull);
  const int k2 = 16 * b + p;
  const float w[3] = {q[0][0], q[0][3], q[1][2]}, a[3] = {q[0][1], q[1][0], q[1][3]}, c[3] = {q[0][2], q[1][1], q[2][0]};
  const uint32_t c2 = cdf_quant(k2, cdf_eval(max(k2, 1), w, a, c));
  const int cnt = __popcll(__ballot(c2 <= slot) & 0xfffeull);
  const uint32_t st_r = (uint32_t)__builtin_amdgcn_readlane((int)c2, cnt);
  const uint32_t nc_r = (uint32_t)__builtin_amdgcn_readlane((int)c2, (cnt + 1) & 15);
  const uint32_t np_r = (uint32_t)__builtin_amdgcn_readlane((int)pv, b);
  start = b == 0 && cnt == 0 ? 0u : st_r;
  freq = (cnt < 15 ? nc_r : np_r) - start;
  uint32_t xn = freq * (S.x >> 16) + slot - start;
  if (S.x < CDF_TOTAL) xn = spread_rank(S.x, start, freq);
  S.x = xn;
  S.R.renorm(S.x, S.pos, lane);
  return 16 * b + cnt;
}

// ------------------------------------------------------------------ lanes
// LDS of a team after the weights: every wave's head table, the serial pops'
// tables, context window, shared words
constexpr int TEAM_HB_WORDS = TEAM_WAVES * 4 * HB_STRIDE;
constexpr int TEAM_SH_WORDS = 32;
NXHD int64_t team_words(int64_t rows, bool serial) {
  return TEAM_HB_WORDS + (serial ? SERIAL_WORDS : 0) + (WIN_PLANES * rows / 2 + 3) / 4 * 4 + TEAM_SH_WORDS;
}

// KIND of pops: a stream per row of the group or two rows (K = 16, 8), serial
// (K = 1, 2, 4), or none (sampling: the inverse CDF at the pixel's Philox
// slots). Teams of a workgroup (one or two) work in step: the barriers are the
// workgroup's. Each decodes lanes from the queue; between two visits to the
// queue the workgroup runs as many groups as the team nearest its lane's end
// has left, and a team without a lane runs the barriers alone.
constexpr int POPS_ROWS = 0, POPS_SERIAL = 1, POPS_SAMPLE = 2;
static int pops_kind(int K) { return K == 0 ? POPS_SAMPLE : K >= 8 ? POPS_ROWS : POPS_SERIAL; }

template <int H_, int C_, int KIND>
__global__ void __launch_bounds__(2 * TEAM_WAVES * 64) k_decode_team(DecArgs A) {
  extern __shared__ float4 smem_f4[];
  float* wts = (float*)smem_f4;
  load_weights(wts, A.w, A.wfloats);
  const int lane = threadIdx.x & 63, p = lane & 15;
  const int m = lane & 15, s = lane >> 4;
  const int wave = uniform((int)(threadIdx.x >> 6));
  const int teams = (int)(blockDim.x / (64 * TEAM_WAVES)), team = wave / TEAM_WAVES, w4 = wave % TEAM_WAVES;
  const int rows = A.team_rows, K = A.K;
  const int64_t tw = team_words(rows, KIND == POPS_SERIAL);
  float* base = wts + A.wfloats + team * tw;
  float* hb = base + w4 * 4 * HB_STRIDE;
  float* prm = base + TEAM_HB_WORDS;
  uint32_t* piv = (uint32_t*)(prm + 16 * SERIAL_PRM);
  int16_t* win = (int16_t*)(prm + (KIND == POPS_SERIAL ? SERIAL_WORDS : 0));
  int32_t* sh = (int32_t*)(base + tw - TEAM_SH_WORDS);
  constexpr int o = H_ + 1;
  const bool live = m < 10;
  // the rows of the group of a wave's pixels (team_row), with two teams on
  // other SIMDs (wave w is on SIMD w mod 4)
  const int v4 = (w4 + 2 * team) & (TEAM_WAVES - 1);
  const bool pairs = KIND == POPS_ROWS && K == 8;
  const int slot = team_row(v4, s, pairs), nslot = team_row(v4, lane & 3, pairs);  // the mixture's pixel, the network's
  int off[quad_inputs(H_)];
  quad_offsets<H_>(off, rows, lane);
  // barriers of one group
  constexpr int n_bar = 1 + (KIND == POPS_SERIAL ? 6 : 0);

  // the team's lane
  int left = 0;        // groups left
  bool done = false;   // no lanes left for this team
  int n = 0, y0 = 0, x0 = 0, Hl = 0, Wl = 0, W = 0;
  TeamGroup G = TEAM_START;
  uint8_t* img = nullptr;
  uint64_t seed = 0;
  uint32_t* dump = nullptr;
  PixStream P;
  SerialStream Z;

  for (;;) {
    const bool need = left == 0 && !done;
    if (need && w4 == 0 && lane == 0) {
      sh[0] = atomicAdd(A.counter, 1);
      sh[1] = 1;
    }
    __syncthreads();
    int total = 0;
    bool mismatch = false;
    if (need) {
      const int64_t L = uniform(sh[0]);
      done = L >= A.n_lanes;
      if (!done) {
        n = find_img_uniform(A.desc, A.n_img, L);
        const ImgDesc D = uniform_desc(A.desc + n);
        const int q = (int)(L - D.lane_base), nl = D.nlx * D.nly;
        const int ly = q / D.nlx, lx = q - ly * D.nlx;
        y0 = ly * D.ph;
        x0 = lx * D.pw;
        Hl = min(D.ph, D.H - y0);
        Wl = min(D.pw, D.W - x0);
        W = D.W;
        img = D.px + ((int64_t)y0 * D.W + x0) * 3;
        seed = D.seed;
        dump = A.sym_dump ? A.sym_dump + D.px_base * 3 : nullptr;
        bool ok = true;
        if constexpr (KIND != POPS_SAMPLE) {
          // header and stream table, as decode_lane checks them
          const uint8_t* C = A.in + uniform64((int64_t)A.in_off[n]);
          const int64_t clen = uniform64((int64_t)(A.in_off[n + 1] - A.in_off[n]));
          const int64_t pay = HDR_BYTES + 4 * (int64_t)nl * K;
          ok = clen >= pay;
          if (ok) {
            const uint32_t ph = D.ph == D.H ? 0u : (uint32_t)D.ph, pw = D.pw == D.W ? 0u : (uint32_t)D.pw;
            ok = C[0] == 'N' && C[1] == 'L' && C[2] == 'X' && C[3] == 'C' && C[4] == CONTAINER_VERSION && C[5] == 1 &&
                 C[6] == (uint8_t)H_ && C[7] == (uint8_t)K && rd_u32(C + 8) == (uint32_t)D.H &&
                 rd_u32(C + 12) == (uint32_t)D.W && (uint32_t)(C[16] | (C[17] << 8)) == ph &&
                 (uint32_t)(C[18] | (C[19] << 8)) == pw && rd_u32(C + 28) == (uint32_t)nl;
            ok = ok && pay + (int64_t)rd_u32(C + HDR_BYTES + 4 * ((int64_t)nl * K - 1)) == clen;
            ok = uniform(ok ? 1 : 0) != 0;
            if (ok) {
              const uint64_t hsh = (uint64_t)rd_u32(C + 20) | ((uint64_t)rd_u32(C + 24) << 32);
              mismatch = uniform(hsh != A.model_hash ? 1 : 0) != 0;
            }
          }
          ok = ok && !mismatch;
          // this row's stream, or this wave's (serial: waves from K on have none)
          const int64_t e = (int64_t)q * K + (KIND == POPS_ROWS ? slot & (K - 1) : min(w4, K - 1));
          uint32_t lend = 1, lstart = 0;
          if (ok) {
            lend = rd_u32(C + HDR_BYTES + 4 * e);
            lstart = e > 0 ? rd_u32(C + HDR_BYTES + 4 * (e - 1)) : 0u;
            const bool okr = lstart <= lend && pay + (int64_t)lend <= clen && lend - lstart >= 1;
            ok = __ballot(!okr) == 0ull;
          }
          if (ok) {
            if constexpr (KIND == POPS_ROWS) {
              P.S = as_global(C + pay + lstart);
              P.len = lend - lstart;
              stream_begin(P);
            } else {
              Z.R.S = C + pay + uniform_u(lstart);
              Z.R.len = uniform_u(lend - lstart);
              Z.R.fill(0, lane);
              uint32_t xs = 0u, ps = 0u;
#pragma unroll
              for (int b = 0; b < 4; ++b) {
                const bool rd = xs < RANS_L && ps < Z.R.len;
                xs = rd ? ((xs << 8) | Z.R.byte_at((uint32_t)b)) : xs;
                ps += rd ? 1u : 0u;
              }
              Z.x = xs;
              Z.pos = ps;
            }
          }
        }
        if (!ok && lane == 0) sh[1] = 0;
        // the lane's groups of 16 rows
        const int T = Wl + o * (Hl - 1);
        for (int t = lane; t < T; t += 64) total += team_groups_at(t, Hl, Wl, o);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) total += __shfl_xor(total, d, 64);
        total = uniform(total);
        for (int k = w4 * 64 + lane; k < WIN_PLANES * rows / 2; k += TEAM_WAVES * 64) ((uint32_t*)win)[k] = 0u;
        G = TEAM_START;
      }
    }
    __syncthreads();
    if (need && !done) {
      left = uniform(sh[1]) ? total : 0;
      if (left == 0) A.status[n] = mismatch ? ST_MISMATCH : ST_CORRUPT;
    }
    if (w4 == 0 && lane == 0) sh[2] = done ? -1 : left;
    __syncthreads();
    // groups until a team needs the queue again (0: one does already)
    int run = 0x7fffffff;
    bool any = false;
    for (int q = 0; q < teams; ++q) {
      const int v = uniform(((const int32_t*)(wts + A.wfloats + (q + 1) * tw - TEAM_SH_WORDS))[2]);
      if (v >= 0) {
        any = true;
        run = min(run, v);
      }
    }
    if (!any) break;

    for (int it = 0; it < run; ++it) {
      if (left == 0) {
        for (int b = 0; b < n_bar; ++b) __syncthreads();
        continue;
      }
      team_next<H_>(
          G, Hl, Wl, [] { team_barrier(); },
          [&] {
            const int r = w4 == TEAM_WAVES - 1 ? team_clear_row<H_>(G, Hl, lane) : -1;
            if (r >= 0) {
#pragma unroll
              for (int c = 0; c < 3; ++c) win_put(win, rows, G.step, c, H_ + r, 0);
            }
          });
      --left;
      const int gi = uniform(G.step), ts = uniform(G.ts), na = uniform(min(16, G.last - G.ts + 1));
      const int i = ts + slot, j = gi - o * i;
      const bool act = slot < na;
      // a wave without a pixel has nothing to do, or (serial pops) the barriers and its pops
      const bool some = __ballot(act) != 0ull;
      if (KIND != POPS_SERIAL && !some) continue;
      const bool busy = KIND != POPS_SERIAL || some;
      Mix16 M;
      uint32_t sl[3] = {0u, 0u, 0u};
      if (busy) {
        float cx[1][quad_inputs(H_)];
        quad_gather<H_>(cx[0], off, win, rows, gi, min(ts + nslot, Hl - 1));
        net_quad<H_, C_, 1>(lds_weights(wts), A.nb, cx, hb, lane);
        mix_prep16(hb + s * HB_STRIDE, m, M);
        if constexpr (KIND == POPS_SAMPLE) sample_slots(seed, W, y0 + i, x0 + j, sl);
      }
      int xv[3] = {0, 0, 0};
      float xr = 0.0f, xg = 0.0f;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        Chan16 Q;
        Mix10 T;
        uint32_t pv = 0;
        if (busy) {
          chan_params16(M, c, xr, xg, Q);
          row_mix10(Q, T);
          pv = row_pivots(T, m);
        }
        int sy = 0;
        uint32_t start = 0, freq = 0;
        if constexpr (KIND == POPS_SAMPLE) {
          if (busy) sy = row_search(T, pv, sl[c], m, s, start, freq);
        } else if constexpr (KIND == POPS_ROWS) {
          if (busy) {
            sy = row_pop(T, pv, P, act && (K == 16 || s < 2), m, s, start, freq);
            if (K == 8) {
              // rows r and r + 8 share a stream: the second has its turn with
              // the first's state, and hands it back
              auto other = [](uint32_t v) { return (uint32_t)__shfl_xor((int)v, 32); };
              const uint32_t x1 = other(P.x), p1 = other(P.pos);
              P.x = s < 2 ? P.x : x1;
              P.pos = s < 2 ? P.pos : p1;
              if (__ballot(act && s >= 2) != 0ull) {
                uint32_t st2, fr2;
                const int sy2 = row_pop(T, pv, P, act && s >= 2, m, s, st2, fr2);
                sy = s < 2 ? sy : sy2;
                start = s < 2 ? start : st2;
                freq = s < 2 ? freq : fr2;
                const uint32_t x2 = other(P.x), p2 = other(P.pos);
                P.x = s < 2 ? x2 : P.x;
                P.pos = s < 2 ? p2 : P.pos;
              }
            }
          }
        } else {
          // tables of the group's pixels, then each stream's wave pops its rows
          if (busy) {
            if (m < 12) {
              float* e = prm + (slot * 4 + (m & 3)) * 12 + 3 * (m >> 2);
              e[0] = live ? Q.w : 0.0f;
              e[1] = live ? Q.a : 0.0f;
              e[2] = live ? Q.b : 0.0f;
            }
            piv[slot * 16 + m] = pv;
          }
          __syncthreads();
          if (w4 < K) {
            f4 q[3];
            uint32_t pw = 0;
            auto fetch = [&](int r) {
              const f4* e = (const f4*)(prm + (r * 4 + s) * 12);
#pragma unroll
              for (int u = 0; u < 3; ++u) q[u] = e[u];
              pw = piv[r * 16 + p];
            };
            fetch(w4);
            Z.x = uniform_u(Z.x);
            Z.pos = uniform_u(Z.pos);
            Z.R.base = uniform_u(Z.R.base);
            Z.R.len = uniform_u(Z.R.len);
            for (int r = w4; r < na; r += K) {
              const f4 q0[3] = {q[0], q[1], q[2]};
              const uint32_t p0 = pw;
              fetch(min(r + K, 15));
              uint32_t st1, fr1;
              const int s1 = serial_pop(Z, q0, p0, lane, st1, fr1);
              if (lane == 0) sh[8 + r] = s1;
              if (dump && lane == 0) dump[((int64_t)(y0 + ts + r) * W + (x0 + gi - o * (ts + r))) * 3 + c] = st1 | (fr1 << 16);
            }
          }
          __syncthreads();
          sy = sh[8 + slot];
        }
        if (c == 0) xv[0] = sy;
        else if (c == 1) xv[1] = sy;
        else xv[2] = sy;
        if (KIND == POPS_ROWS && dump && act && m == 0)
          dump[((int64_t)(y0 + i) * W + (x0 + j)) * 3 + c] = start | (freq << 16);
        if (c < 2 && busy) {
          posterior16(M, sy, Q, live);
          if (c == 0) xr = normalise(sy);
          else xg = normalise(sy);
        }
      }
      if (act && m < 3) {
        const int v = m == 0 ? xv[0] : (m == 1 ? xv[1] : xv[2]);
        img[((uint32_t)i * (uint32_t)W + (uint32_t)j) * 3u + (uint32_t)m] = (uint8_t)v;  // a window's rows: 32 bits hold it
        win_put(win, rows, gi, m, H_ + i, 2 * v - 255);
      }
    }
    // a team whose lane has ended: every stream back at its start state
    if (run > 0 && left == 0 && !done) {
      bool clean = true;
      if constexpr (KIND == POPS_ROWS) clean = P.x == RANS_X0 && P.pos == P.len;
      if constexpr (KIND == POPS_SERIAL) clean = w4 >= K || (Z.x == RANS_X0 && Z.pos == Z.R.len);
      if (!clean) A.status[n] = ST_CORRUPT;
    }
  }
}

// ------------------------------------------------------------------ row streams
// Row streams (one rANS stream per lane row): a lane is decoded in bands of
// ROW_BAND = 16 rows, a team (workgroup of ROW_WAVES = 4 waves) per band. Each
// row pops its own stream, so every row of a step decodes at once (the whole
// step of Algorithm 1 in parallel); a row's coder state stays in the registers
// of the lanes that decode it. A band's top rows read the h rows above,
// decoded by the band above it, possibly on another CU: each band publishes
// how many steps it has finished (release), and before step t a wave of its
// own (link) waits until the band above has finished step t - 1 (acquire), then
// copies those rows' pixels of that step, at most h, into the window. Bands
// are taken from the queue in order (by the step they start at, across the
// images of the batch), so the band above is always held by a running or
// finished workgroup; its skew of (h + 1) ROW_BAND steps makes waits rare once
// a band has started, and the pixels above are then loaded a step ahead. A
// wait also ends, with the image marked corrupt, if it exceeds
// band_wait_ticks of the 100 MHz clock (20 s unless a test lowers it), so
// every workgroup reaches the end of the kernel whatever happens.
constexpr int32_t BAND_DONE = 0x7fffffff;

NXD int find_img_band(const ImgDesc* __restrict__ d, int n, int64_t key) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int64_t b = uniform64(d[mid].band_base);
    if (b <= key) lo = mid; else hi = mid - 1;
  }
  return uniform(lo);
}

// the whole wave releases its stores, then its first lane publishes
NXD void band_publish(int32_t* slot, int32_t v, int lane) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) __hip_atomic_store(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int H_>
constexpr int band_rows() { return (ROW_BAND + H_ + 3) / 4 * 4; }

// The workgroup has a fifth wave, the band's link to its neighbours: after
// each step's barrier it stores the step's pixels, publishes the step and
// fetches the rows above for the next, so that neither the release nor those
// loads and stores are on the team's path (1,100 of 16,500 cycles a step when
// the team's first wave did it). The pixels are its stores because a release
// waits for the stores of its own wave alone, and a barrier of the workgroup
// for no store to memory: another wave's could still be on their way when the
// step is published. (One 1024 x 1024 image, h = 3, 64 channels, 2 blocks:
// 29.7 -> 28.6 ms, 13.5 thousand cycles a step.)
constexpr int ROW_BLOCK = 64 * (ROW_WAVES + 1);

template <int H_, int C_>
__device__ void decode_band(const DecArgs& A, const float* w, float* hbs, int16_t* win, int32_t* sh, int64_t B) {
  static_assert(ROW_BAND == 16 && ROW_WAVES == 4, "a band is one 16-pixel tile, four rows per wave");
  constexpr int rows = band_rows<H_>();
  const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
  const bool link = wave == ROW_WAVES;
  float* hb = hbs + min(wave, ROW_WAVES - 1) * 4 * HB_STRIDE;
  const int m = lane & 15, s = lane >> 4, pp = 4 * wave + s;  // mixture: component m of band row pp
  const int n = find_img_band(A.desc, A.n_img, B);
  const ImgDesc D = uniform_desc(A.desc + n);
  // which lane of the image and which band of it: lanes in order, full patch
  // rows first, each lane cut into bands_of(Hl) bands
  const int64_t bi = B - D.band_base;
  const int64_t per_prow = (int64_t)D.nlx * bands_of(D.ph);
  const int ly = (int)(bi / per_prow);
  const int y0 = ly * D.ph, Hl = min(D.ph, D.H - y0);
  const int64_t rem = bi - (int64_t)ly * per_prow;
  const int lx = (int)(rem / bands_of(Hl)), bb = (int)(rem - (int64_t)lx * bands_of(Hl));
  const int x0 = lx * D.pw, Wl = min(D.pw, D.W - x0);
  const int nl = D.nlx * D.nly;
  const int r0 = bb * ROW_BAND, r1 = min(Hl, r0 + ROW_BAND) - 1, nrows = r1 - r0 + 1;
  int32_t* mine = A.progress + B;
  // header and stream table (every lane reads the same bytes)
  const uint8_t* C = A.in + uniform64((int64_t)A.in_off[n]);
  const int64_t clen = uniform64((int64_t)(A.in_off[n + 1] - A.in_off[n]));
  const int64_t ns = image_streams(ROW_STREAMS, D.H, D.nlx, D.nly);
  const int64_t pay = HDR_BYTES + 4 * ns;
  bool ok = clen >= pay;
  bool mismatch = false;
  if (ok) {
    const uint32_t ph = D.ph == D.H ? 0u : (uint32_t)D.ph, pw = D.pw == D.W ? 0u : (uint32_t)D.pw;
    ok = C[0] == 'N' && C[1] == 'L' && C[2] == 'X' && C[3] == 'C' && C[4] == CONTAINER_VERSION && C[5] == 1 &&
         C[6] == (uint8_t)H_ && C[7] == (uint8_t)ROW_STREAMS && rd_u32(C + 8) == (uint32_t)D.H &&
         rd_u32(C + 12) == (uint32_t)D.W && (uint32_t)(C[16] | (C[17] << 8)) == ph &&
         (uint32_t)(C[18] | (C[19] << 8)) == pw && rd_u32(C + 28) == (uint32_t)nl;
    ok = ok && pay + (int64_t)rd_u32(C + HDR_BYTES + 4 * (ns - 1)) == clen;
    ok = uniform(ok ? 1 : 0) != 0;
    if (ok) {
      const uint64_t hsh = (uint64_t)rd_u32(C + 20) | ((uint64_t)rd_u32(C + 24) << 32);
      mismatch = uniform(hsh != A.model_hash ? 1 : 0) != 0;
    }
  }
  // this lane's row stream (band row pp; rows past the band's last take the
  // last row's and never pop), in every lane of the row's pixel
  const int64_t ebase = row_entry_base(ly, lx, D.nlx, D.ph, Hl) + r0;
  if (threadIdx.x == 0) sh[0] = 1;
  for (int k = threadIdx.x; k < WIN_PLANES * rows / 2; k += ROW_BLOCK) ((uint32_t*)win)[k] = 0u;
  __syncthreads();
  PixStream P;
  P.x = 0u;
  P.pos = 0u;
  P.len = 1u;
  P.S = as_global(C);
  if (ok && !mismatch) {
    const int64_t e = ebase + min(pp, nrows - 1);
    const uint32_t lend = rd_u32(C + HDR_BYTES + 4 * e);
    const uint32_t lstart = e > 0 ? rd_u32(C + HDR_BYTES + 4 * (e - 1)) : 0u;
    const bool okr = lstart <= lend && pay + (int64_t)lend <= clen && lend - lstart >= 1;
    if (okr) {
      P.S = as_global(C + pay + lstart);
      P.len = lend - lstart;
      stream_begin(P);
    } else {
      sh[0] = 0;
    }
  }
  __syncthreads();
  ok = ok && sh[0] != 0;
  if (mismatch || !ok) {
    if (threadIdx.x == 0) {
      A.status[n] = mismatch ? ST_MISMATCH : ST_CORRUPT;
      band_publish(mine, BAND_DONE, 0);  // the band below must not wait for this one
    }
    __syncthreads();
    return;
  }
  constexpr int o = H_ + 1;
  const int t_lo = o * r0, t_hi = (Wl - 1) + o * r1;
  if (link) {
    // lane 3 q + c takes channel c of row r0 - 1 - q: its value of step t, 0
    // where that is off the lane
    const uint8_t* img = D.px;
    const int uq = min(lane / 3, H_ - 1), uc = lane - 3 * (lane / 3);
    const int i = r0 - 1 - uq;
    const gbytes row = as_global(img + ((int64_t)(y0 + max(i, 0)) * D.W + x0) * 3 + uc);
    // the band's pixels of step t, from the window: lane 3 q + c channel c of row r0 + q
    const int sq = min(lane / 3, ROW_BAND - 1), sc = lane - 3 * (lane / 3);
    auto store = [&](int t) {
      const int is = r0 + sq, j = t - o * is;
      const int v = win[win_place(rows, t, sc, H_ + sq)];
      if (lane < 3 * ROW_BAND && is <= r1 && j >= 0 && j < Wl)
        D.px[((int64_t)(y0 + is) * D.W + (x0 + j)) * 3 + sc] = (uint8_t)((v + 255) >> 1);
    };
    auto fetch = [&](int t) {
      const int j = t - o * i;
      const bool in = bb > 0 && i >= 0 && j >= 0 && j < Wl;
      const int v = row[3 * min(max(j, 0), Wl - 1)];
      if (lane < 3 * H_) win_put(win, rows, t, uc, H_ - 1 - uq, in ? 2 * v - 255 : 0);
    };
    int32_t seen = bb == 0 ? BAND_DONE : 0;  // steps of the band above known to be finished
    const int32_t* up = A.progress + (B - 1);
    for (int t = t_lo; t <= t_hi; ++t) {
      if (seen < t) {
        // wait until the band above has finished step t - 1
        int32_t v = uniform(__hip_atomic_load(up, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT));
        if (v < t) {
          const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
          while (v < t) {
            __builtin_amdgcn_s_sleep(4);
            v = uniform(__hip_atomic_load(up, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT));
            if (v < t && __builtin_amdgcn_s_memrealtime() - t0 > A.band_wait_ticks) {
              A.status[n] = ST_CORRUPT;  // never expected: the image cannot be trusted
              v = BAND_DONE;
            }
          }
        }
        seen = v;
      }
      if (t == t_lo)  // the window's columns before the band's first step
        for (int d = H_ * (H_ + 2); d > 1; --d) fetch(t - d);
      fetch(t - 1);
      // the band's step t - 1 is finished in every wave (its pixels in the window)
      __syncthreads();
      if (t > t_lo) store(t - 1);
      band_publish(mine, t, lane);
    }
    __syncthreads();
    store(t_hi);
    band_publish(mine, BAND_DONE, lane);
  } else {
    uint32_t* dump = A.sym_dump ? A.sym_dump + D.px_base * 3 : nullptr;
    const bool live = m < 10;
    const int i = r0 + pp;
    int off[quad_inputs(H_)];
    quad_offsets<H_>(off, rows, lane);
    for (int t = t_lo; t <= t_hi; ++t) {
      team_barrier();
      const int j = t - o * i;
      const bool act = i <= r1 && j >= 0 && j < Wl;
      int xv[3] = {0, 0, 0};
      if (__ballot(act) != 0ull) {
        {
          float cx[1][quad_inputs(H_)];
          quad_gather<H_>(cx[0], off, win, rows, t, 4 * wave + (lane & 3));
          net_quad<H_, C_, 1>(lds_weights(w), A.nb, cx, hb, lane);
        }
        Mix16 M;
        mix_prep16(hb + s * HB_STRIDE, m, M);
        float xr = 0.0f, xg = 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          Chan16 Q;
          chan_params16(M, c, xr, xg, Q);
          Mix10 T;
          row_mix10(Q, T);
          uint32_t start, freq;
          const int sy = row_pop(T, row_pivots(T, m), P, act, m, s, start, freq);
          if (c == 0) xv[0] = sy;
          else if (c == 1) xv[1] = sy;
          else xv[2] = sy;
          if (dump && act && m == 0) dump[((int64_t)(y0 + i) * D.W + (x0 + j)) * 3 + c] = start | (freq << 16);
          if (c == 0) {
            posterior16(M, sy, Q, live);
            xr = normalise(sy);
          } else if (c == 1) {
            posterior16(M, sy, Q, live);
            xg = normalise(sy);
          }
        }
      }
      // the window's column t: the decoded pixels, 0 in the other rows
      if (m < 3) {
        const int v = m == 0 ? xv[0] : (m == 1 ? xv[1] : xv[2]);
        win_put(win, rows, t, m, H_ + pp, act ? 2 * v - 255 : 0);
      }
    }
    team_barrier();
  }
  // every row's stream must end in the start state with every byte read
  if (!link && pp < nrows && m == 0 && !(P.x == RANS_X0 && P.pos == P.len)) A.status[n] = ST_CORRUPT;
  __syncthreads();
}

// LDS of the row decoder after the weights: the waves' head tables, the
// context window, then a few shared words
template <int H_>
constexpr size_t rows_lds_extra() {
  return (size_t)(TEAM_HB_WORDS + WIN_PLANES * band_rows<H_>() / 2 + 4) * sizeof(float);
}

template <int H_, int C_>
__global__ void __launch_bounds__(ROW_BLOCK) k_decode_rows(DecArgs A) {
  extern __shared__ float4 smem_f4[];
  float* w = (float*)smem_f4;
  load_weights(w, A.w, A.wfloats);
  float* hb = w + A.wfloats;
  int16_t* win = (int16_t*)(hb + TEAM_HB_WORDS);
  int32_t* sh = (int32_t*)(hb + TEAM_HB_WORDS + WIN_PLANES * band_rows<H_>() / 2);  // band and flag words
  for (;;) {
    if (threadIdx.x == 0) sh[2] = atomicAdd(A.counter, 1);
    __syncthreads();
    const int64_t Q = sh[2];
    __syncthreads();
    if (Q >= A.n_bands) break;
    // the queue's order of the bands (start step, then image and lane), or image order
    const int64_t B = A.band_order ? (int64_t)uniform(A.band_order[Q]) : Q;
    if (B < 0 || B >= A.n_bands) continue;  // only a damaged workspace: never decode out of range
    decode_band<H_, C_>(A, w, hb, win, sh, B);
  }
}

// ------------------------------------------------------------------ launchers
static hipError_t lds_limit(int& lim) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&lim, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  return e;
}

template <int H_, int C_>
static hipError_t team_setup_t(int K) {
  int lim = 0;
  const hipError_t e = lds_limit(lim);
  if (e != hipSuccess) return e;
  const int kind = pops_kind(K);
  if (kind == POPS_ROWS) return allow_lds(k_decode_team<H_, C_, POPS_ROWS>, (size_t)lim);
  if (kind == POPS_SERIAL) return allow_lds(k_decode_team<H_, C_, POPS_SERIAL>, (size_t)lim);
  return allow_lds(k_decode_team<H_, C_, POPS_SAMPLE>, (size_t)lim);
}

template <int H_, int C_>
static hipError_t rows_setup_t() {
  int lim = 0;
  const hipError_t e = lds_limit(lim);
  return e == hipSuccess ? allow_lds(k_decode_rows<H_, C_>, (size_t)lim) : e;
}

hipError_t prepare_team(int h, int C, int K) { NX_DISPATCH(team_setup_t, h, C, K); }

hipError_t prepare_rows(int h, int C) { NX_DISPATCH(rows_setup_t, h, C); }

static size_t team_lds(int64_t wfloats, int teams, int rows, bool serial) {
  return (size_t)(wfloats + teams * team_words(rows, serial)) * sizeof(float);
}

int decode_teams(const TeamQuery& q) {
  if (q.order == 0 || q.rows < 4 || q.rows > 4096) return 0;
  const int teams = team_count(q.C, q.nb, q.K, q.n_lanes, q.step_rows, q.cus);
  return teams && team_lds(q.wfloats, teams, (int)q.rows, q.K > 0 && q.K < 8) <= q.lds ? teams : 0;
}

template <int H_, int C_>
static hipError_t team_t(const DecArgs& a, int kind, int teams, hipStream_t s) {
  const size_t lds = team_lds(a.wfloats, teams, a.team_rows, kind == POPS_SERIAL);
  const dim3 grid((unsigned)((a.n_lanes + teams - 1) / teams)), block((unsigned)(64 * TEAM_WAVES * teams));
  if (kind == POPS_ROWS)
    hipLaunchKernelGGL((k_decode_team<H_, C_, POPS_ROWS>), grid, block, lds, s, a);
  else if (kind == POPS_SERIAL)
    hipLaunchKernelGGL((k_decode_team<H_, C_, POPS_SERIAL>), grid, block, lds, s, a);
  else
    hipLaunchKernelGGL((k_decode_team<H_, C_, POPS_SAMPLE>), grid, block, lds, s, a);
  return hipGetLastError();
}

hipError_t launch_decode_team(int h, int C, const DecArgs& a, int teams, hipStream_t s) {
  if (a.n_lanes == 0) return hipSuccess;
  if (teams < 1 || teams > 2 || (a.K != 0 && !valid_interleave(a.K))) return hipErrorInvalidValue;
  NX_DISPATCH(team_t, h, C, a, pops_kind(a.K), teams, s);
}

template <int H_, int C_>
static hipError_t rows_t(const DecArgs& a, int grid, hipStream_t s) {
  const size_t lds = (size_t)a.wfloats * 4 + rows_lds_extra<H_>();
  hipLaunchKernelGGL((k_decode_rows<H_, C_>), dim3(grid), dim3(ROW_BLOCK), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_decode_rows(int h, int C, const DecArgs& a, int grid, hipStream_t s) {
  if (a.n_bands == 0) return hipSuccess;
  NX_DISPATCH(rows_t, h, C, a, grid, s);
}

}  // namespace nx
