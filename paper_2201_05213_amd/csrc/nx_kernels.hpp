// nx_kernels.hpp -- launch interface between the host runtime (nx_capi.cpp)
// and the kernels (nx_kernels.hip). Plain structs of device pointers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nx_layout.hpp"

namespace nx {

// status codes written to the per-image device status array (match nellox.h)
constexpr int ST_OK = 0;
constexpr int ST_CORRUPT = 4;
constexpr int ST_MISMATCH = 5;

struct PassArgs {
  const float* w;          // device weight image
  int64_t wfloats;
  int nb;
  const ImgDesc* desc;     // device copy of the plan
  int n_img;
  int64_t n_tiles;
  int mode;                // 0 symbols, 1 continuous bits, 2 full CDF rows
  uint32_t* sym;           // mode 0: (start | freq << 16) per pixel and channel
  float* bits;             // mode 0: quantised ideal bits per pixel (nullable);
                           // mode 1: continuous bits per pixel
  int32_t* cdf;            // mode 2: [pixel][3][257]
};

struct RansEncArgs {
  const ImgDesc* desc;
  int n_img;
  int64_t n_lanes;
  int64_t n_streams;       // rANS streams of the batch (n_lanes K, or the lane rows)
  int order;               // 0 raster, 1 wavefront
  int h;
  int K;                   // rANS streams per lane (ROW_STREAMS: one per lane row)
  const uint32_t* sym;
  uint8_t* slots;
  uint32_t* lane_len;      // symbols per stream (gather), then bytes per stream (encoder)
  uint32_t* rev;           // per stream, its symbols in coding order (reverse decode order);
                           // image n's streams from desc[n].rev_base, stream_rev_words each
  int32_t* after;          // per stream and step t: the stream's symbols in steps after t;
                           // from desc[n].after_base, stream_after_entries each
  int64_t max_lane_px;     // pixels of the largest lane
  int wave_per_stream;     // a wave per stream, else a thread (rans_wave)
};

// Whether each rANS stream is coded by a wave of its own. A wave per stream
// takes 89 cycles a symbol while it has its SIMD to itself, and about 65 times
// the waves of the SIMD beyond (4 cycles an instruction); a thread per stream
// 320 to 410, whatever their number (measured, streams of 768 to 1,024
// symbols of unequal length). So the wave is ahead up to about five streams on
// each of the 4 SIMDs of a CU; the line is at four. Row streams have no pass
// that lays their symbols out: a thread reads a row of its own, and the wave
// stays ahead for longer.
inline bool rans_wave(int64_t n_streams, bool rows, int cus) {
  return n_streams <= (rows ? 8 : 4) * 4 * (int64_t)cus;
}

struct PackArgs {
  const ImgDesc* desc;
  int n_img;
  int64_t n_lanes;
  int64_t n_streams;       // rANS streams of the batch
  int order, h;
  int K;                   // rANS streams per lane (ROW_STREAMS: one per lane row)
  uint64_t model_hash;
  const uint8_t* slots;
  const uint32_t* lane_len;  // per stream (global stream index, image n's from desc[n].stream_base)
  uint32_t* lane_end;      // scratch: cumulative payload bytes per stream
  uint64_t* img_bytes;     // scratch: container bytes per image
  uint8_t* out;
  uint64_t* out_offsets;   // n_img + 1
  uint64_t out_cap;
  int32_t* overflow;       // set when the containers would exceed out_cap
  int64_t max_stream_bytes;  // an estimate of the longest stream, for the grid
};

// The largest group of pixels that the wave-per-lane decoder takes by fours
// (net_quad); larger ones take a tile of 16 (net_forward). A tile's matrix
// instructions do the work of 16 outputs and 16 pixels in 32 cycles, a quad's of
// 64 outputs, used or not, and four pixels in 8: what a quad costs against a tile
// goes as 1 / C. Time of groups of 4, 8 and 12 pixels by quads against tiles
// (768 to 2,048 lanes, either layout, 1 to 3 blocks): 64 channels 1.48-1.80, 1.31-1.50 and
// 1.10-1.21 times as fast; 32 channels 1.14-1.29, 1.02-1.10 and 0.89-0.97; 16
// channels 1.00-1.08, 0.88-0.99 and 0.74-0.89. With 16 channels a block's two
// layers are longer by fours, chains of 16 dependent instructions with a
// transpose each, so that what the gather saves is used up after about four
// blocks (raster order, h = 3, 0 to 24 blocks: 1.03, 1.02, 1.01, 1.00 with 3,
// 0.995 with 4, 0.98 with 6, 0.97 with 8, 0.92 with 24; 32 channels 1.2 with 8).
constexpr int quad_limit(int C, int nb = 0) { return C >= 64 ? 12 : C >= 32 ? 8 : nb <= 4 ? 4 : 0; }

struct DecArgs {
  const float* w;
  int64_t wfloats;
  int nb;
  const ImgDesc* desc;     // px = output image
  int n_img;
  int64_t n_lanes;
  int order;
  int K;                   // rANS streams per lane
  uint64_t model_hash;
  const uint8_t* in;
  const uint64_t* in_off;  // n_img + 1
  int32_t* status;         // n_img
  int32_t* counter;        // work queue head
  uint32_t* sym_dump;      // nullable: (start | freq << 16) used per pixel/channel
  uint8_t* ring;           // order 2: grid x waves context rings of ring_wave_bytes(ring_rows)
  int ring_rows;
  int team_rows;           // teams: rows of a team's context window in LDS
  int wave_words, quad_px; // a wave's LDS in words; groups of at most quad_px pixels take net_quad (set at launch)
  int32_t* progress;       // row streams: per band, the steps it has finished (zeroed by the prep)
  int64_t n_bands;         // row streams: bands of the batch (the queue's work items)
  uint64_t band_wait_ticks;  // row streams: the longest wait on the band above (100 MHz clock ticks)
  const int32_t* band_order; // row streams, nullable: queue position -> band (in image order)
};
// row streams: the default limit of a band's wait on the band above (20 s);
// a wait that exceeds it marks the image corrupt and lets the band finish
constexpr uint64_t BAND_WAIT_TICKS = 2000000000ull;

// Training objective and gradient (nx_train.hip). n images of H x W, all
// pixel tensors pixel-major.
struct TrainArgs {
  const uint8_t* imgs;     // n x H x W x 3
  int n, H, W, ntx;        // ntx = ceil(W / 16)
  int64_t npx, n_tiles;    // n H W, n H ntx
  int nb, Cp, KP;          // KP = conv inputs padded to a multiple of 16
  const float* wimg;       // forward weight image
  const float* wimgT;      // transposed weight image
  int64_t wfloats, wTfloats;
  float* bits;             // [npx] continuous bits per pixel
  float* ctx;              // [npx][KP] conv inputs (normalised taps)
  float* u;                // [2 nb + 1][npx][Cp] inputs of the 1x1 layers and the head
  float* theta;            // [npx][112] head rows
  float* delta;            // [2 nb + 1][npx][Cp] output deltas: first layer, then per block W1, W2
  float* dtheta;           // [npx][112] head-row deltas
  const float* grad_bits;  // [n] d loss / d bits of image n
};

// layer kinds of the weight-gradient launch (they set the layer's shape)
constexpr int WGRAD_FIRST = 0, WGRAD_BLOCK = 1, WGRAD_HEAD = 2, WGRAD_HEAD_REST = 3;
// the head's rows go to two layer entries, of WGRAD_HEAD_TILES row tiles and of
// the rest, which keeps every layer's accumulators at most 4 row tiles wide
constexpr int WGRAD_HEAD_PARTS = 2, WGRAD_HEAD_TILES = 4;
constexpr int WGRAD_MAX_LAYERS = 11;  // the head's parts, first layer, up to 8 1x1 layers

struct WgradLayer {
  const float* delta;      // [npx][ld_delta], rows 16-byte aligned
  const float* in;         // [npx][ld_in], rows 16-byte aligned
  int ld_delta, ld_in;
  int64_t w_off, b_off;    // offsets of this layer's dW [rows][cols] and db in a partial
  int kind;                // one of the above
};

struct WgradArgs {
  WgradLayer layer[WGRAD_MAX_LAYERS];  // indexed by blockIdx.y
  int64_t npx, chunk, nchunks, ngrad;
  float* partial;          // [nchunks][ngrad]
};

struct GradReduceArgs {
  int h, C, Cp, nb, KP;
  int64_t off_conv, off_blocks, off_head, bias_conv, bias_blocks, bias_head;
  int64_t nchunks, ngrad;
  const float* partial;
  float* grad;             // parameter vector layout
};

// decoder workgroup shape: waves per workgroup and the LDS it needs beyond
// the weight image (per wave a pivot table and a mixture table)
constexpr int DECODE_WAVES = 12;
constexpr int DECODE_LDS_EXTRA = DECODE_WAVES * (256 + 16 * 36) * 4;

// host launchers (return hipError_t of the launch); h in {1,2,3}, C in {16,32,64}
bool supported(int h, int C);
hipError_t launch_pass(int h, int C, const PassArgs& a, int grid, hipStream_t s);
hipError_t launch_rans_encode(const RansEncArgs& a, hipStream_t s);
hipError_t launch_pack(const PackArgs& a, hipStream_t s);
hipError_t launch_decode_prep(int32_t* status, int n_img, int32_t* counter, hipStream_t s,
                              int32_t* progress = nullptr, int64_t n_bands = 0);
// row streams: the band decoder (a team of four waves, and one more, per workgroup, one band at a time)
constexpr int ROW_WAVES = 4;
hipError_t launch_decode_rows(int h, int C, const DecArgs& a, int grid, hipStream_t s);
// Few lanes: teams of four waves per lane (nx_team.hip), `teams` lanes a
// workgroup and CU. decode_teams: how many, or 0 for the wave-per-lane
// decoder (launch_decode, launch_sample). A lone wave issues a group of 16
// pixels in 26 to 32 thousand cycles (h = 3, 64 channels, 2 blocks), a team in
// 14 to 17; two teams share their SIMDs' issue, 20 thousand for a group of
// each. Measured, a wave per lane against teams, 37 model sizes, lanes from
// 8 x 8 to 64 x 64, 12 x 100 and 90 x 8, every kind of pops:
//   one lane per CU   one team 1.13 to 1.93 times as fast (256 lanes of 64 x 64,
//                     8 streams, that model: 4.30 -> 2.23 ms); with 16 channels
//                     and 24 blocks 1.0 to 1.1, but 0.95 to 0.98 with 4 streams
//   two               two teams 1.0 to 2.0 times (512 such lanes: 4.34 -> 3.34 ms)
//                     where at most two of a team's waves have pixels, so that
//                     the two teams are on different SIMDs, and with 2 streams.
//                     Where more have, the network counts, which four pixels
//                     take in a chain of single inputs: 64 channels 1.0 to 1.5
//                     (0.95 with 8 streams), 32 channels 0.93 to 1.2 up to 3
//                     blocks and 0.89 to 1.1 with 8, 16 channels 0.97 to 1.2
//                     without blocks, 0.91 to 1.1 with 2, 0.79 to 1.0 with 8
//   three, four       0.50 to 0.86 (1,024 lanes of 32 x 32, 4 streams:
//                     1.63 -> 2.65 ms)
// So the line is at two lanes per CU, for two teams by the waves that have pixels
// and the depth, in either wavefront layout, where the window fits the LDS
// left by the weights.
struct TeamQuery {
  int C, nb;           // the model's channels (padded) and blocks
  int K;               // rANS streams per lane, 0 to sample (also DecArgs.K of the launch)
  int order;
  int64_t wfloats, n_lanes;
  int64_t rows;        // window rows of the tallest lane
  int step_rows;       // the most rows of a wavefront step (0: not known)
  int cus;
  size_t lds;
};
int decode_teams(const TeamQuery& q);
// the waves of a team with pixels in a group of that many rows (team_row)
constexpr int team_busy(int K, int rows) {
  const int r = rows < 1 || rows > 16 ? 16 : rows;
  return K == 8 ? ((r < 8 ? r : 8) + 1) / 2 : (r + 3) / 4;
}
// the rule without the window
constexpr int team_count(int C, int nb, int K, int64_t n_lanes, int step_rows, int cus) {
  if (n_lanes < 1 || n_lanes > 2 * (int64_t)cus) return 0;
  if (C <= 16 && nb > 8 && K == 4) return 0;
  if (n_lanes <= cus) return 1;
  const bool deep = C >= 64 ? false : C >= 32 ? nb > 4 : nb > 0;
  return deep && K != 2 && team_busy(K, step_rows) > 2 ? 0 : 2;
}
hipError_t launch_decode_team(int h, int C, const DecArgs& a, int teams, hipStream_t s);
// raise the LDS limit of the team kernel for K, or of the row-stream decoder
hipError_t prepare_team(int h, int C, int K);
hipError_t prepare_rows(int h, int C);
// raise the decoder kernels' LDS limit (at every prepare, outside any stream capture)
hipError_t prepare_decode(int h, int C, int K);
// waves per workgroup in 1..DECODE_WAVES (the LDS, of at most `lds` bytes, takes each wave's tables);
// prepare_decode must have run for (h, C, a.K)
hipError_t launch_decode(int h, int C, const DecArgs& a, int grid, int waves, size_t lds, hipStream_t s);
// ancestral sampling with the decoder's schedule (DecArgs: in, in_off, status
// and sym_dump unused; every image descriptor carries its seed)
hipError_t launch_sample(int h, int C, const DecArgs& a, int grid, int waves, size_t lds, hipStream_t s);
// per-image FP64 sums of per-pixel bits, in a fixed order (partials: n_img
// x REDUCE_PARTS doubles of scratch)
constexpr int REDUCE_PARTS = 64;
hipError_t launch_reduce_bits(const ImgDesc* desc, int n_img, const float* bits, double* partials, double* out,
                              hipStream_t s);

// the no-allocation decoder's scratch: STATIC_SCRATCH_BYTES of device memory
// per GPU (a file-scope array); static_scratch gives the current device's
// address, looked up on the first call per device
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)32 << 20;
hipError_t static_scratch(void** ptr);

// exhaustive order check of the hardware exp2 and reciprocal (out: 4 counters)
hipError_t launch_check_monotone(unsigned long long* out, hipStream_t s);

constexpr int TRAIN_BLOCK = 16 * 64;  // threads per workgroup of the per-tile training kernels
hipError_t launch_swizzle(const float* params, int h, int C, int Cp, int nb, float* wimg, int64_t nw, float* wimgT,
                          int64_t nwT, hipStream_t s);
hipError_t launch_train_fwd(int h, int Cp, const TrainArgs& a, int grid, hipStream_t s);
hipError_t launch_train_bwd(int h, int Cp, const TrainArgs& a, int grid, hipStream_t s);
hipError_t launch_wgrad(int CT, int KT, const WgradArgs& a, int nlayers, hipStream_t s);
// resident workgroups of that launch per CU (0 if the runtime cannot tell)
int wgrad_blocks_per_cu(int CT, int KT);
hipError_t launch_grad_reduce(const GradReduceArgs& a, hipStream_t s);
hipError_t launch_bits_img(const float* bits, int n, int64_t per_img, double* out, hipStream_t s);

}  // namespace nx
