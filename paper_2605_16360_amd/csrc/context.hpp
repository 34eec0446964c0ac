// Host-side state behind the opaque proxykv_ctx: configuration, device workspace and the device
// copy of the mapper weights.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <vector>

#include "../../include/proxykv.h"

namespace pkv {

struct DeviceBuffer {
  void* ptr = nullptr;
  size_t bytes = 0;
};

// Counters of the in-place compaction: an equal piece of `block` for each of the first streams that make such calls.  Nothing orders calls of
// different streams, on caches of their own, so they must not meet in the counters.  A piece is 4 bytes per 160 KB that a call moves, so
// that 32 of them are 0.08 % of that (512 rows of 12 345 tokens of D = 128, half kept: 45 KB each).
constexpr int kInplaceStreams = 32;
struct InplaceCounters {
  std::mutex mutex;  // held from where a call finds its counters until its launches are made
  DeviceBuffer block;
  hipStream_t stream[kInplaceStreams];
  int streams = 0;
  // Blocks that became too small: calls that were made may still count there.  Each has at most half the bytes of the next.
  void* older[48];
  int n_older = 0;
};

// Device pointers into one allocation that holds the prepared mapper weights.
struct EncoderLayerWeights {
  const uint16_t* in_w;   // fp16 [3*d_time, d_time]
  const float* in_b;      // [3*d_time]
  const uint16_t* out_w;  // fp16 [d_time, d_time]
  const float* out_b;
  const float *ln1_g, *ln1_b;
  const uint16_t* ffn1_w;  // fp16 [d_ffn, d_time]
  const float* ffn1_b;
  const uint16_t* ffn2_w;  // fp16 [d_time, d_ffn]
  const float* ffn2_b;
  const float *ln2_g, *ln2_b;
};

struct MapperWeights {
  const float* conv1_w;                  // fp32 [H_kv*3, c_mid]
  const float *bn1_scale, *bn1_shift;    // batch norm and conv bias folded: y = conv * scale + shift
  float stem_cw = 0.0f, stem_cs = 0.0f;  // |first conv block's output| <= stem_cw * max|x| + stem_cs (host values)
  const uint16_t* conv2_w;               // fp16 [d_time, 3*c_mid], k index = tap * c_mid + channel
  const float *bn2_scale, *bn2_shift;
  std::vector<EncoderLayerWeights> enc;
  const uint16_t* kv_w;                  // fp16 [2*H_kv*d_head_x, d_time]: key rows, then value rows
  const float* kv_b;                     // [2*H_kv*d_head_x]
  const float* queries;                  // [H_l, d_head_x]
  const float* out_w;                    // [d_head_x]
  float out_b;
  const float* pe;                       // fp32 [win, d_time] sinusoidal table
  const void *blk_w = nullptr, *blk_b = nullptr;  // the encoder's weights and biases once more, in the order in which mapper_block.hip reads them
};

// What launch li (0 .. n_enc_layers) of mapper_block.hip reads per wave, in fragments of 1 KB: weights and biases.
inline size_t block_frags(const proxykv_config& c, int li) {
  return (li > 0 ? 128 + (size_t)c.d_ffn / 2 : 0) + (li < c.n_enc_layers ? 384 : 0);
}
inline size_t block_bias_frags(const proxykv_config& c, int li) {
  return (li > 0 ? 16 + (size_t)c.d_ffn / 64 : 0) + (li < c.n_enc_layers ? 24 : 0);
}
constexpr size_t kBlkFragBytes = 1024, kBlkRing = 16;  // a wave asks for weights up to sixteen fragments ahead
// Puts w.enc's matrices and biases in that order (w.blk_w, w.blk_b); implemented in mapper_block.hip.
hipError_t pack_encoder_blocks(const proxykv_config& c, const MapperWeights& w, void* blk_w, void* blk_b, hipStream_t stream);

constexpr int kMapLanes = 2;

// Row length of the stage-3 K/V projection's output: 2*H_kv*d_head_x rounded up to the GEMM's column tile.
inline int kv3_stride(const proxykv_config& c) { return (2 * c.H_kv * c.d_head_x + 255) / 256 * 256; }

// Mapper activations for one batch of proxy layers (the network runs once per distinct proxy layer, and its weights are
// shared by all of them, so a batch's layers lie one behind the other on the M axis of every launch).
struct MapperWorkspace {
  DeviceBuffer x;      // fp32 [Tp, d_time] per layer: residual stream over all window rows
  DeviceBuffer xb;     // fp16 [Tp, d_time]: attention output (large tiles); the stem's output, feeding the first projection (small tiles)
  DeviceBuffer work;   // what one kernel leaves for the next (LanePointers in mapper.hpp)
  DeviceBuffer s3;     // fp32 [Np, (H_l + 1) * H_s]  stage 3: per token the H_l x H_s logits, then <w_o, V[s]> of every slot
  DeviceBuffer range;  // 16 words: partial maxima of |score| (bits)
  DeviceBuffer pre;    // fp32 [Tp, d_time]: small inputs only: sums that the next kernel normalises as it reads them
};

}  // namespace pkv

struct proxykv_ctx {
  proxykv_config cfg;
  int last_hip_error = 0;
  bool weights_set = false;
  // stage timing: events at the boundaries of the PROXYKV_N_STAGES stages of proxykv_prune
  bool profile = false, ev_created = false;
  hipEvent_t ev[PROXYKV_N_STAGES + 1] = {};
  bool ev_recorded[PROXYKV_N_STAGES + 1] = {};
  pkv::DeviceBuffer weight_blob, block_blob;       // block_blob: the encoder's weights in the large tiles' order
  pkv::MapperWeights w;
  std::vector<int32_t> pairing;  // [L_l] 0-based proxy layer per target layer
  // workspace
  pkv::DeviceBuffer q_bf16, kctx_bf16, krec_bf16;  // bf16 copies of fp32 inputs
  pkv::DeviceBuffer neg_lse;                       // fp32 [L_s, H_q, N_q], or (reference, sum) pairs of several workgroups
  pkv::DeviceBuffer x_parts;                       // sum form: the column sums of several workgroups per key block
  size_t parts_short = 0;                          // bytes of x_parts that the device did not have
  pkv::DeviceBuffer x_ws;                          // fp32 [L_s, H_kv, N]
  pkv::DeviceBuffer yhat_ws;                       // fp32 [L_l, H_l, N]
  pkv::DeviceBuffer topk_ws;                       // state of Top-K where workgroups share a row
  pkv::InplaceCounters inplace;
  bool topk_short = false;                         // memory was short: topk_ws has no masks, or only the narrower histograms
  bool fused_select = false;                       // proxykv_prune: selection and gather in one launch (measured slower)
  pkv::MapperWorkspace m[pkv::kMapLanes];          // one per lane; only the lanes a length needs are allocated
  int64_t map_len = 0;                             // longest context that m has been sized for
  // lanes 1 .. kMapLanes-1: streams (default priority, non-blocking) and the events that fork them from and join
  // them into the caller's stream, which is lane 0
  bool lanes_created = false;
  hipStream_t lane_stream[pkv::kMapLanes] = {};
  hipEvent_t lane_fork = nullptr, lane_join[pkv::kMapLanes] = {};
  int distinct_layers = 1;                         // distinct proxy layers in `pairing`
};

namespace pkv {

// Number of windows and total window rows for context length N.
inline void window_plan(int64_t N, int win, int stride, int64_t* n_win, int64_t* total_rows) {
  if (N <= win) {
    *n_win = 1;
    *total_rows = N;
    return;
  }
  const int64_t k = (N - win + stride - 1) / stride + 1;
  *n_win = k;
  *total_rows = (k - 1) * (int64_t)win + (N - (k - 1) * (int64_t)stride);
}

// How the mapper runs a context of N tokens: the distinct proxy layers in `n_batches` batches, dealt to `lanes` streams.
// Small layers leave the chip idle one by one (1500 rows are 12 blocks on 256 CUs), so a batch takes
// several, up to kMapBatchRows rows.  Two batches side by side, on streams and in workspaces of their own, let one's loads, stores
// and attention run beside the other's products, so layers of more than kMapSplitRows rows together make an even number
// of batches (3 layers of 3000 tokens in one 990 us, in two 953); a batch takes two layers if they are no more than kMapPairRows rows.
// Every row holds about 6 KB of workspace for as long as the context lives, so the limits are where more costs more than it gives.
// 16 distinct layers, us, one layer per batch / as here:
//   N = 1500   1753 / 1491     N = 4096   7575 / 5973     N = 8192   13 756 / 13 939     N = 32 768   60 440 / 60 527
constexpr int64_t kMapBatchRows = 65536, kMapPairRows = 131072, kMapSplitRows = 8192;
constexpr int kMaxBatch = 32;
static_assert(kMapBatchRows >= 256 * kMaxBatch && kMapSplitRows >= 256 * kMaxBatch, "a small-tile batch is neither cut nor split");
// Up to this many rows, each layer's counted in whole tiles of 64, the small tiles are faster (large tiles on the left, us: one layer of
// 2048 rows 790 / 570, two of 1250 708 / 672, eight of 256 594 / 491, 20 of 110 586 / 591), beyond it the large ones, whose half blocks
// take the same time until the chip is full (two layers of 1300 rows 717 / 730, eight of 380 614 / 709, 16 of 140 588 / 646, 28 of
// 80 587 / 720; with whole blocks alone the line lay at 4096 rows: one layer of 5548 rows 1139, with half blocks 821).
constexpr int64_t kMapSmallRows = 2560;
struct MapPlan {
  int64_t N, n_win, T;  // tokens, windows and window rows of a layer
  int64_t Tp, Np;       // window rows and tokens of a layer, padded to the GEMM's 256-row tile
  int n_batches, batch, lanes;  // batch: layers of the largest batch
  bool small;           // few rows: the small-tile kernels
};
// `most` layers per batch and `most_lanes` lanes: what a workspace has room for.  Neither changes a result: the kernels' arithmetic
// does not depend on the other layers of a batch, and `small` is decided by the layers alone.
inline MapPlan map_plan(const proxykv_config& c, int64_t N, int distinct_layers, int most = kMaxBatch, int most_lanes = kMapLanes) {
  MapPlan p;
  p.N = N;
  window_plan(N, c.win, c.stride, &p.n_win, &p.T);
  p.Tp = (p.T + 255) / 256 * 256;
  p.Np = (N + 255) / 256 * 256;
  const int64_t few = (distinct_layers + kMaxBatch - 1) / kMaxBatch;  // batches, if only their number of layers were limited
  p.small = (distinct_layers + few - 1) / few * ((p.T + 63) / 64 * 64) <= kMapSmallRows && c.n_enc_layers > 0;
  int64_t cap = kMapBatchRows / p.Tp;
  if (cap < 2) cap = 2 * p.Tp <= kMapPairRows ? 2 : 1;
  if (cap > most) cap = most;
  int64_t n = (distinct_layers + cap - 1) / cap;
  if (distinct_layers * p.Tp > kMapSplitRows && n % kMapLanes != 0) n += kMapLanes - n % kMapLanes;
  if (n > distinct_layers) n = distinct_layers;
  p.n_batches = (int)n;
  p.batch = (int)((distinct_layers + n - 1) / n);
  p.lanes = (int)(n < most_lanes ? n : most_lanes);
  return p;
}
// Bytes of `work` per layer, the largest of what is there at a time: the stem's first output, read before the encoder starts;
// q, k and v and, with the small tiles, the attention's output, all read before the FFN's hidden rows are written; those, which the
// small tiles alone write, read before the next layer's q, k and v are; the overlap-averaged encoder output.  (With a buffer for each of
// these a row took 12 KB.)
inline size_t map_work_bytes(const proxykv_config& c, const MapPlan& p, bool small) {
  const size_t row = (size_t)c.d_time * 2, Tp = (size_t)p.Tp;
  const size_t attn = (small ? 4 : 3) * Tp * row, hid = small ? Tp * (size_t)c.d_ffn * 2 : 0;
  const size_t h1 = ((size_t)(p.N + 2) * c.c_mid * 2 + 255) / 256 * 256, zg = (size_t)p.Np * row;
  const size_t a = attn > hid ? attn : hid, b = h1 > zg ? h1 : zg;
  return a > b ? a : b;
}
// The largest small-tile batch of all lengths of up to p.N tokens: that of the longest.
struct SmallBatch {
  int64_t layers;
  MapPlan plan;
};
inline SmallBatch small_batch(const proxykv_config& c, const MapPlan& p, int distinct_layers) {
  const int64_t few = (distinct_layers + kMaxBatch - 1) / kMaxBatch, b = (distinct_layers + few - 1) / few;
  int64_t n = kMapSmallRows / b / 64 * 64;
  if (n > c.win) n = c.win;
  return {b, map_plan(c, n < p.N ? n : p.N, distinct_layers)};
}

// Runs the mapper for every distinct proxy layer; implemented in mapper.hip.
// Returns a hipError_t; the workspace must already be large enough for the plan.
hipError_t mapper_forward(proxykv_ctx* ctx, const MapPlan& p, const float* x, float* yhat, hipStream_t stream);

}  // namespace pkv
