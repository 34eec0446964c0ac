// Host-side state behind the opaque proxykv_ctx: configuration, device workspace and the device
// copy of the mapper weights.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "../../include/proxykv.h"

namespace pkv {

struct DeviceBuffer {
  void* ptr = nullptr;
  size_t bytes = 0;
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
  const float* conv1_w;                  // fp32 [c_mid, H_kv*3]
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
};

constexpr int kMapLanes = 2;

// Row length of the stage-3 K/V projection's output: 2*H_kv*d_head_x rounded up to the GEMM's column tile.
inline int kv3_stride(const proxykv_config& c) { return (2 * c.H_kv * c.d_head_x + 255) / 256 * 256; }

// Mapper activations for one batch of proxy layers (the network runs once per distinct proxy layer, and its weights are
// shared by all of them, so a batch's layers lie one behind the other on the M axis of every launch).
struct MapperWorkspace {
  // per layer of the batch:
  DeviceBuffer h1;       // fp16 [(N+2), c_mid]  stem conv1 output with one zero row at each end
  DeviceBuffer x;        // fp32 [Tp, d_time]    residual stream over all window rows
  DeviceBuffer xb;       // fp16 [Tp, d_time]    fp16 copy feeding the GEMMs
  DeviceBuffer qk;       // fp16 [Tp, 2*d_time]  q and k of the current layer
  DeviceBuffer vt;       // fp16 [n_win, heads, 64, vt_ld]  v transposed per window and head
  DeviceBuffer ao;       // fp16 [Tp, d_time]    attention output
  DeviceBuffer hid;      // fp16 [Tp, d_ffn]
  DeviceBuffer zg;       // fp16 [Np, d_time]    overlap-averaged encoder output
  DeviceBuffer s3;       // fp32 [Np, (H_l + 1) * H_s]  stage 3: per token the H_l x H_s logits, then <w_o, V[s]> of every slot
  DeviceBuffer pre;      // fp32 [Tp, d_time]    small inputs only: sums that the next kernel normalises as it reads them
  DeviceBuffer range;    // 16 words: partial maxima of |score| (bits)
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
  pkv::DeviceBuffer weight_blob;
  pkv::MapperWeights w;
  std::vector<int32_t> pairing;  // [L_l] 0-based proxy layer per target layer
  // workspace
  pkv::DeviceBuffer q_bf16, kctx_bf16, krec_bf16;  // bf16 copies of fp32 inputs
  pkv::DeviceBuffer neg_lse;                       // fp32 [L_s, H_q, N_q], or (reference, sum) pairs of several workgroups
  pkv::DeviceBuffer x_parts;                       // sum form: the column sums of several workgroups per key block
  pkv::DeviceBuffer x_ws;                          // fp32 [L_s, H_kv, N]
  pkv::DeviceBuffer yhat_ws;                       // fp32 [L_l, H_l, N]
  pkv::DeviceBuffer topk_ws;                       // per-row histograms and counters of the Top-K of rows split over workgroups
  bool fused_select = false;                       // proxykv_prune: selection and gather in one launch (measured slower)
  pkv::MapperWorkspace m[pkv::kMapLanes];          // one per lane; only the lanes a length needs are allocated
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

// How the mapper runs a context of N tokens: `batch` distinct proxy layers at a time, batches dealt to `lanes` streams.
// Small layers leave the chip idle one by one (512 window rows are 12 output tiles of the QKV product), so a batch takes
// as many of them as make kMapBatchRows rows (about 14 KB of workspace each).  Long contexts need several batches; two of
// them side by side, on streams and in workspaces of their own, let one's stores and residual reads run under the other's
// matrix work.  Measured, 16 distinct layers, one layer per batch on four streams / all on one stream in batches of
// 262 144 rows / as here: N = 1500 6.15 / 2.21 / 2.21 ms, N = 8192 19.3 / 19.0 / 18.5 ms, N = 32 768 82.0 / 84.1 / 81.4 ms.
constexpr int64_t kMapBatchRows = 131072;
constexpr int kMaxBatch = 32;
// Up to this many rows in a batch the small tiles are faster (large tiles on the left: one layer of 512 rows 867 / 231 us, of 2000
// rows 1060 / 566 us; 16 layers of 256 rows 970 / 882 us).
constexpr int64_t kMapSmallRows = 4096;
struct MapPlan {
  int64_t n_win, T;   // windows and window rows of a layer
  int64_t Tp, Np;     // window rows and tokens of a layer, padded to the GEMM's 256-row tile
  int64_t vt_ld;      // row length of the transposed v
  int batch, lanes;
  bool small;         // few rows: the small-tile kernels
};
inline MapPlan map_plan(const proxykv_config& c, int64_t N, int distinct_layers) {
  MapPlan p;
  window_plan(N, c.win, c.stride, &p.n_win, &p.T);
  p.Tp = (p.T + 255) / 256 * 256;
  p.Np = (N + 255) / 256 * 256;
  p.vt_ld = p.n_win > 1 ? c.win : p.Tp;
  int64_t cap = kMapBatchRows / p.Tp;
  cap = cap < 1 ? 1 : (cap > kMaxBatch ? kMaxBatch : cap);
  const int64_t n_batches = (distinct_layers + cap - 1) / cap;
  p.batch = (int)((distinct_layers + n_batches - 1) / n_batches);
  const int64_t used = (distinct_layers + p.batch - 1) / p.batch;
  p.lanes = used < kMapLanes ? (int)used : kMapLanes;
  p.small = p.batch * p.T <= kMapSmallRows && c.n_enc_layers > 0;
  return p;
}

// Runs the mapper for every distinct proxy layer; implemented in mapper.hip.
// Returns a hipError_t; the workspace must already be large enough.
hipError_t mapper_forward(proxykv_ctx* ctx, const float* x, int64_t N, float* yhat, hipStream_t stream);

}  // namespace pkv
