// nx_coder.hpp -- device pieces shared by the coder's kernels (nx_kernels.hip,
// nx_team.hip): wave-uniform plan lookups, the coder's spread slots and
// streams, CDF evaluation over all ten components in a lane; and the host
// helpers their launchers share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nx_device.hpp"
#include "nx_kernels.hpp"
#include "nx_order.hpp"

namespace nx {

NXD int find_img(const ImgDesc* __restrict__ d, int n, int64_t key, bool by_lane) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int64_t b = by_lane ? d[mid].lane_base : d[mid].tile_base;
    if (b <= key) lo = mid; else hi = mid - 1;
  }
  return lo;
}

NXD uint32_t rd_u32(const uint8_t* p) {
  return (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16) | ((uint32_t)p[3] << 24);
}

NXD int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
NXD int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// the same search with every step wave-uniform (key must be wave-uniform)
NXD int find_img_uniform(const ImgDesc* __restrict__ d, int n, int64_t key, bool by_lane = true) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int64_t b = uniform64(by_lane ? d[mid].lane_base : d[mid].tile_base);
    if (b <= key) lo = mid; else hi = mid - 1;
  }
  return uniform(lo);
}

// Descriptor fields as wave-uniform values. Every lane loads the same
// descriptor; saying so (readfirstlane) keeps all control flow that depends
// on it uniform: the compiler then never splits a wave across the exits of the
// persistent loops.
NXD ImgDesc uniform_desc(const ImgDesc* __restrict__ p) {
  ImgDesc D = *p;
  D.px = (uint8_t*)uniform64((int64_t)D.px);
  D.H = uniform(D.H);
  D.W = uniform(D.W);
  D.ph = uniform(D.ph);
  D.pw = uniform(D.pw);
  D.nlx = uniform(D.nlx);
  D.nly = uniform(D.nly);
  D.lane_base = uniform64(D.lane_base);
  D.px_base = uniform64(D.px_base);
  D.tile_base = uniform64(D.tile_base);
  D.ntx = uniform(D.ntx);
  D.slot_base = uniform64(D.slot_base);
  D.seed = (uint64_t)uniform64((int64_t)D.seed);
  return D;
}

NXD uint32_t uniform_u(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// the whole workgroup (any block size) copies the weight image into LDS
NXD void load_weights(float* lds, const float* __restrict__ w, int64_t nfloats) {
  const int64_t n4 = nfloats >> 2;
  for (int64_t i = threadIdx.x; i < n4; i += blockDim.x) ((float4*)lds)[i] = ((const float4*)w)[i];
  __syncthreads();
}

// ------------------------------------------------------------------ coder states
// Spread slots. A push of symbol (s, f) from a state x < f (only near the
// start of a stream) takes the x-th (from 0) slot y of [0, 2^16) whose 16-bit
// reversal lies in [s, s + f): reversal deals the range out about 2^16 / f
// apart, so the state grows by about the symbol's probability, where the
// usual rule would jump to s + x. The decoder recognises such a state (it is
// below 2^16), searches the symbol with the reversed slot and pops by the
// rank of y among the symbol's slots. Both walk the reversal's 16 bits from
// the lowest: the range values with low bits r (j of them) and bit j clear
// number floor((s + f - 1 - r) / 2^(j+1)) - floor((s - 1 - r) / 2^(j+1))
// (the floors are arithmetic shifts).
NXD uint32_t rev16(uint32_t v) { return __builtin_bitreverse32(v) >> 16; }

NXD int32_t spread_count(int32_t lo, int32_t hi, int32_t r, int sh) { return ((hi - r) >> sh) - ((lo - r) >> sh); }

NXD uint32_t spread_select(uint32_t x, uint32_t s, uint32_t f) {
  const int32_t lo = (int32_t)s - 1, hi = (int32_t)(s + f) - 1;
  int32_t r = 0, left = (int32_t)x;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int32_t n0 = spread_count(lo, hi, r, j + 1);
    const bool one = left >= n0;
    left -= one ? n0 : 0;
    r |= one ? (1 << j) : 0;
  }
  return rev16((uint32_t)r);
}

NXD uint32_t spread_rank(uint32_t y, uint32_t s, uint32_t f) {
  const uint32_t v = rev16(y);
  const int32_t lo = (int32_t)s - 1, hi = (int32_t)(s + f) - 1;
  int32_t n = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int32_t r = (int32_t)(v & ((1u << j) - 1u));
    n += ((v >> j) & 1u) ? spread_count(lo, hi, r, j + 1) : 0;
  }
  return (uint32_t)n;
}

// Bytes of the lane payload, staged 256 at a time: lane l of the wave holds
// bytes base + 4l .. base + 4l + 3; a byte is fetched with a lane read.
struct ByteStage {
  const uint8_t* S;
  uint32_t len, base;
  uint32_t word;
  NXD void fill(uint32_t at, int lane) {
    // clamped, unconditional loads; bytes past the end read as 0
    base = at;
    const gbytes g = as_global(S);
    uint32_t v = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t o = at + 4 * (uint32_t)lane + b;
      const uint32_t byte = g[o < len ? o : len - 1];
      v |= (o < len ? byte : 0u) << (8 * b);
    }
    word = v;
  }
  // byte at pos, pos >= base; the caller keeps pos < base + 256 (bytes past
  // the window read as garbage, never as an out-of-range lane)
  NXD uint32_t byte_at(uint32_t pos) const {
    const uint32_t off = pos - base;
    const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)word, (int)((off >> 2) & 63u));
    return (v >> (8 * (off & 3u))) & 255u;
  }
  NXD uint32_t get(uint32_t pos, int lane) {
    if (pos - base >= 256u) fill(pos, lane);
    return byte_at(pos);
  }
  // rANS renormalisation after a pop: at most two bytes are read (the popped
  // state is at least 2^7 while bytes remain), each only while x < L and
  // bytes remain; no branch except the rare window refill
  NXD void renorm(uint32_t& x, uint32_t& pos, int lane, bool act = true) {
    if (pos + 2u > base + 256u && pos < len) fill(pos & ~3u, lane);
    const uint32_t b0 = byte_at(pos), b1 = byte_at(pos + 1u);
    const bool r0 = act && x < RANS_L && pos < len;
    x = r0 ? ((x << 8) | b0) : x;
    pos += r0 ? 1u : 0u;
    const bool r1 = x < RANS_L && pos < len;
    x = r1 ? ((x << 8) | b1) : x;
    pos += r1 ? 1u : 0u;
  }
};

// K >= 8: one stream per pixel row of a 16-row group (K = 16), or one per
// pair of rows p and p + 8 (K = 8); lane (p, g) holds stream p mod K's state,
// the same in every lane of the pixel (and, for K = 8, of both rows)
struct PixStream {
  gbytes S;
  uint32_t len, pos, x;
};

// a stream's initial state: its first bytes, most significant first, read
// while x < L (at most four; loads clamped into the stream, len >= 1)
NXD void stream_begin(PixStream& P) {
  uint32_t xs = 0u, ps = 0u;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint32_t byte = P.S[min((uint32_t)b, P.len - 1u)];
    const bool rd = xs < RANS_L && ps < P.len;
    xs = rd ? ((xs << 8) | byte) : xs;
    ps += rd ? 1u : 0u;
  }
  P.x = xs;
  P.pos = ps;
}

// ------------------------------------------------------------------ ten components in a lane
// A pixel's mixture for the channel: (w, a, b) of component m.
struct Mix10 {
  float w[10], a[10], b[10];
};

// F at bin edge k over all ten components in this lane. The terms and the
// additions are those of cdf_eval: per lane group g the sum
// s_g = (t_g + t_{g+4}) + t_{g+8} (groups 2 and 3 add an exact zero), then
// (s_0 + s_1) + (s_2 + s_3); so the value is bit-identical to the encoder's.
NXD float cdf_eval10(int k, const Mix10& P) {
  const float e = bin_edge(k);
  float t[10];
#pragma unroll
  for (int m = 0; m < 10; ++m) {
    const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(-e, P.a[m], P.b[m]));
    t[m] = P.w[m] * __builtin_amdgcn_rcpf(1.0f + x);
  }
  const float s0 = (t[0] + t[4]) + t[8];
  const float s1 = (t[1] + t[5]) + t[9];
  const float s2 = t[2] + t[6];
  const float s3 = t[3] + t[7];
  return (s0 + s1) + (s2 + s3);
}

// bits of row g in a wave-wide ballot, counted
NXD int row_count(uint64_t bal, int g) {
  const uint32_t half = (g & 2) ? (uint32_t)(bal >> 32) : (uint32_t)bal;
  return __builtin_popcount((half >> ((g & 1) << 4)) & 0xffffu);
}

// ------------------------------------------------------------------ host helpers
// kernels keep the whole weight image in LDS: allow up to the device limit
template <typename K>
static hipError_t allow_lds(K kernel, size_t lds) {
  const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) (void)hipGetLastError();  // reported here, not by the next launch's check
  return e;
}

#define NX_DISPATCH(FN, h, C, ...)                          \
  do {                                                      \
    if (h == 3 && C == 64) return FN<3, 64>(__VA_ARGS__);   \
    if (h == 3 && C == 32) return FN<3, 32>(__VA_ARGS__);   \
    if (h == 3 && C == 16) return FN<3, 16>(__VA_ARGS__);   \
    if (h == 2 && C == 64) return FN<2, 64>(__VA_ARGS__);   \
    if (h == 2 && C == 32) return FN<2, 32>(__VA_ARGS__);   \
    if (h == 2 && C == 16) return FN<2, 16>(__VA_ARGS__);   \
    if (h == 1 && C == 32) return FN<1, 32>(__VA_ARGS__);   \
    if (h == 1 && C == 16) return FN<1, 16>(__VA_ARGS__);   \
    return hipErrorInvalidValue;                            \
  } while (0)

}  // namespace nx
