// C ABI of the ProxyKV hot path: argument validation, context and workspace management, and the
// sequencing of the kernels.  Every check runs before the first HIP call of an entry point.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "context.hpp"
#include "kernels.hpp"

using pkv::DeviceBuffer;

namespace {

inline bool hip_ok(proxykv_ctx* ctx, hipError_t e) {
  if (e == hipSuccess) return true;
  if (ctx) ctx->last_hip_error = (int)e;
  (void)hipGetLastError();
  return false;
}

#define PKV_HIP(ctx, call)                                \
  do {                                                    \
    if (!hip_ok((ctx), (call))) return PROXYKV_EHIP;      \
  } while (0)

int validate_config(const proxykv_config* c) {
  if (!c) return PROXYKV_EINVAL;
  if (c->L_s <= 0 || c->H_q <= 0 || c->H_kv <= 0 || c->d <= 0 || c->L_l <= 0 || c->H_l <= 0 || c->D <= 0)
    return PROXYKV_EINVAL;
  if (c->H_q % c->H_kv != 0) return PROXYKV_EINVAL;
  if (c->d_time <= 0 || c->c_mid <= 0 || c->n_enc_layers < 0 || c->n_enc_heads <= 0 || c->d_ffn <= 0 ||
      c->d_head_x <= 0 || c->win <= 0 || c->stride <= 0 || c->stride > c->win || c->device < 0)
    return PROXYKV_EINVAL;
  if (c->reduce != PROXYKV_REDUCE_MAX && c->reduce != PROXYKV_REDUCE_SUM) return PROXYKV_EINVAL;
  if (c->d != 64 && c->d != 128) return PROXYKV_EUNSUPPORTED;
  if ((c->D * 2) % 16 != 0) return PROXYKV_EUNSUPPORTED;
  if (c->d_time != 512 || c->n_enc_heads != 8 || c->d_head_x != 64 || c->win != 2048 || c->stride != 1024 ||
      c->c_mid % 256 != 0 || c->d_ffn % 256 != 0 || c->H_kv > 16 || c->H_l > 64)
    return PROXYKV_EUNSUPPORTED;
  return PROXYKV_OK;
}

int validate_lengths(int64_t N, int64_t N_q, int64_t chunk) {
  if (N <= 0 || N_q <= 0 || chunk <= 0) return PROXYKV_EINVAL;
  if (N >= (1ll << 31) - 4096 || N_q >= (1ll << 31) - 4096 || chunk >= (1ll << 31)) return PROXYKV_EINVAL;
  return PROXYKV_OK;
}

void free_buffer(DeviceBuffer& b) {
  if (b.ptr) (void)hipFree(b.ptr);
  b.ptr = nullptr;
  b.bytes = 0;
}

// The mapper's workspace, lane by lane.  The last buffer is used by the small tiles only.
constexpr int kLaneBuffers = 6;
void lane_buffers(pkv::MapperWorkspace& m, DeviceBuffer* (&b)[kLaneBuffers]) {
  DeviceBuffer* all[kLaneBuffers] = {&m.x, &m.xb, &m.work, &m.s3, &m.range, &m.pre};
  std::copy(all, all + kLaneBuffers, b);
}
void free_lanes(proxykv_ctx* ctx) {
  for (pkv::MapperWorkspace& m : ctx->m) {
    DeviceBuffer* b[kLaneBuffers];
    lane_buffers(m, b);
    for (DeviceBuffer* x : b) free_buffer(*x);
  }
  ctx->map_len = 0;
}

// whether `stream` records a graph (or it cannot be told)
bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// `need`: the mapper's workspace is given up where that makes room
int ensure(proxykv_ctx* ctx, DeviceBuffer& b, size_t bytes, hipStream_t stream, bool need = true) {
  if (bytes <= b.bytes) return PROXYKV_OK;
  if (b.ptr) {
    // earlier work on the stream may still read the old buffer
    PKV_HIP(ctx, hipStreamSynchronize(stream));
    PKV_HIP(ctx, hipFree(b.ptr));
    b.ptr = nullptr;
    b.bytes = 0;
  }
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, bytes);
  if (need && e == hipErrorOutOfMemory && ctx->map_len > 0) {
    // the mapper makes do with less: it takes what is left when it runs next
    (void)hipGetLastError();
    PKV_HIP(ctx, hipStreamSynchronize(stream));
    free_lanes(ctx);
    e = hipMalloc(&p, bytes);
  }
  if (e != hipSuccess) {
    hip_ok(ctx, e);
    return e == hipErrorOutOfMemory ? PROXYKV_ENOMEM : PROXYKV_EHIP;
  }
  // start from zeros: padding that no kernel writes is read, and dropped, as finite values
  e = hipMemset(p, 0, bytes);
  if (e != hipSuccess) {
    hip_ok(ctx, e);
    (void)hipFree(p);
    return PROXYKV_EHIP;
  }
  b.ptr = p;
  b.bytes = bytes;
  return PROXYKV_OK;
}

// ---- workspace

// number of distinct proxy layers that the target layers are paired with
int count_distinct(const proxykv_config& c) {
  int distinct = 0, prev = -1;
  for (int ll = 0; ll < c.L_l; ++ll) {
    const int ls = (int)(((int64_t)(ll + 1) * c.L_s + c.L_l - 1) / c.L_l - 1);
    distinct += ls != prev;
    prev = ls;
  }
  return distinct;
}

// A lane's buffers, in bytes for one layer of the plan's length (row counts of GEMM outputs, and of the residuals they read, are
// padded to the GEMM's 256-row tile).
struct LaneBytes {
  size_t per_layer[kLaneBuffers];
};
LaneBytes lane_bytes(const proxykv_config& c, const pkv::MapPlan& p) {
  const size_t row = (size_t)p.Tp * c.d_time;
  return {{row * 4, row * 2, pkv::map_work_bytes(c, p, p.small), (size_t)p.Np * (size_t)(c.H_l + 1) * (size_t)c.H_kv * 4, 64, row * 4}};
}
// bytes of buffer i of a lane: the plan's largest batch.  Shorter calls are served from the same workspace, so `pre` and, as long as
// that takes no more than these layers would with the small tiles, `work` cover the small-tile batches of all shorter lengths (they
// have one lane, unless there are more layers than a batch takes).
size_t lane_need(const proxykv_config& c, const pkv::MapPlan& p, const LaneBytes& lb, int lane, int distinct, int i) {
  constexpr int kWork = 2, kRange = 4, kPre = kLaneBuffers - 1;
  if (i == kRange) return pkv::kMaxBatch * lb.per_layer[i];  // a line per layer: a long plan's few would limit a short call's batch
  const size_t own = i == kPre ? 0 : (size_t)p.batch * lb.per_layer[i];
  if ((i != kWork && i != kPre) || c.n_enc_layers == 0 || (lane > 0 && distinct <= pkv::kMaxBatch)) return own;
  const pkv::SmallBatch s = pkv::small_batch(c, p, distinct);
  if (i == kPre) return (size_t)(s.layers * s.plan.Tp) * (size_t)c.d_time * 4;
  return std::max(own, std::min((size_t)s.layers * pkv::map_work_bytes(c, s.plan, true), (size_t)p.batch * pkv::map_work_bytes(c, p, true)));
}
// layers of the plan's length that lane m has room for
int lane_room(pkv::MapperWorkspace& m, const pkv::MapPlan& p, const LaneBytes& lb) {
  DeviceBuffer* b[kLaneBuffers];
  lane_buffers(m, b);
  size_t room = (size_t)pkv::kMaxBatch;
  for (int i = 0; i < kLaneBuffers - (p.small ? 0 : 1); ++i) room = std::min(room, b[i]->bytes / lb.per_layer[i]);
  return (int)room;
}

// The mapper's plan for N tokens, with the workspace for it.  A context that has served a longer one has room for every shorter
// one, if not always for as many layers at a time as would be asked for: then the batches are smaller, and nothing is allocated
// (the call may be under capture).  Where the device has too little memory, the batches are halved until they fit.
int reserve_map(proxykv_ctx* ctx, int64_t N, hipStream_t stream, pkv::MapPlan* out) {
  const proxykv_config& c = ctx->cfg;
  const int distinct = ctx->distinct_layers;
  pkv::MapPlan p = pkv::map_plan(c, N, distinct);
  const LaneBytes lb = lane_bytes(c, p);
  if (N <= ctx->map_len) {
    int room = lane_room(ctx->m[0], p, lb), lanes = 1;
    for (; lanes < p.lanes; ++lanes) {
      const int r = lane_room(ctx->m[lanes], p, lb);
      if (r < 1) break;
      room = std::min(room, r);
    }
    if (room >= 1) {
      *out = pkv::map_plan(c, N, distinct, room, lanes);
      return PROXYKV_OK;
    }
  }
  ctx->map_len = 0;
  for (;;) {
    int rc = PROXYKV_OK;
    for (int lane = 0; lane < p.lanes && rc == PROXYKV_OK; ++lane) {
      DeviceBuffer* b[kLaneBuffers];
      lane_buffers(ctx->m[lane], b);
      for (int i = 0; i < kLaneBuffers && rc == PROXYKV_OK; ++i) rc = ensure(ctx, *b[i], lane_need(c, p, lb, lane, distinct, i), stream);
    }
    if (rc == PROXYKV_ENOMEM && (p.batch > 1 || p.lanes > 1)) {
      PKV_HIP(ctx, hipStreamSynchronize(stream));
      free_lanes(ctx);
      p = p.batch > 1 ? pkv::map_plan(c, N, distinct, (p.batch + 1) / 2) : pkv::map_plan(c, N, distinct, 1, 1);
      continue;
    }
    if (rc != PROXYKV_OK) return rc;
    break;
  }
  if (p.lanes > 1 && !ctx->lanes_created) {
    for (int i = 1; i < pkv::kMapLanes; ++i) {
      if (!ctx->lane_stream[i]) PKV_HIP(ctx, hipStreamCreateWithFlags(&ctx->lane_stream[i], hipStreamNonBlocking));
      if (!ctx->lane_join[i]) PKV_HIP(ctx, hipEventCreateWithFlags(&ctx->lane_join[i], hipEventDisableTiming));
    }
    if (!ctx->lane_fork) PKV_HIP(ctx, hipEventCreateWithFlags(&ctx->lane_fork, hipEventDisableTiming));
    ctx->lanes_created = true;
  }
  ctx->map_len = N;
  *out = p;
  return PROXYKV_OK;
}

// What scoring and pruning need beside the mapper.  Every size grows with N and N_q, so that a workspace that has served the longest
// call serves all shorter ones.  `parts`: the column sums of several workgroups per key block too (the sum and the causal
// form; the max form has none).
struct Sizes {
  size_t neg_lse, x_parts, x_ws, yhat_ws;
};
Sizes workspace_sizes(const proxykv_config& c, int64_t N, int64_t N_q) {
  return {pkv::score_lse_bytes(c.L_s, c.H_q, N_q), pkv::score_parts_bytes(c.L_s, c.H_kv, c.d, N), (size_t)c.L_s * c.H_kv * (size_t)N * 4,
          (size_t)c.L_l * c.H_l * (size_t)N * 4};
}
int reserve_score(proxykv_ctx* ctx, int64_t N, int64_t N_q, bool parts, hipStream_t stream) {
  const Sizes s = workspace_sizes(ctx->cfg, N, N_q);
  int rc = ensure(ctx, ctx->neg_lse, s.neg_lse, stream);
  if (rc == PROXYKV_OK && parts && (ctx->parts_short == 0 || s.x_parts < ctx->parts_short)) {
    rc = ensure(ctx, ctx->x_parts, s.x_parts, stream);
    if (rc == PROXYKV_ENOMEM) {  // then one workgroup per key block
      ctx->parts_short = s.x_parts;
      rc = PROXYKV_OK;
    }
  }
  return rc;
}
// workgroups per key block that pass 2 may use
int query_splits(const proxykv_ctx* ctx, bool sum, bool causal, int64_t N, int64_t N_q) {
  const proxykv_config& c = ctx->cfg;
  const int s = pkv::score_query_splits(sum, causal, c.L_s, c.H_q, c.H_kv, c.d, N, N_q);
  return sum && ctx->x_parts.bytes < (size_t)s * c.L_s * c.H_kv * (size_t)N * 4 ? 1 : s;
}
// The masks are done without where they do not fit beside what is there (112 rows of 170 000 scores 67 -> 78 us), and where the wide
// histograms do not fit, the narrow ones take their place.
int reserve_topk(proxykv_ctx* ctx, int64_t rows, int64_t N, hipStream_t stream) {
  const size_t least = pkv::topk_scratch_bytes_least(rows, N);
  if (ctx->topk_short && ctx->topk_ws.bytes >= least) return PROXYKV_OK;
  int rc = ensure(ctx, ctx->topk_ws, pkv::topk_scratch_bytes(rows, N), stream, false);
  ctx->topk_short = rc == PROXYKV_ENOMEM;
  if (rc == PROXYKV_ENOMEM) rc = ensure(ctx, ctx->topk_ws, pkv::topk_scratch_bytes_no_masks(rows, N), stream);
  if (rc == PROXYKV_ENOMEM) rc = ensure(ctx, ctx->topk_ws, least, stream);
  return rc;
}
// Room for the in-place compaction's counters, `piece` bytes for every stream.  Where there is none, what was there stays.  (The mutex is held.)
size_t inplace_block_bytes(size_t piece) { return (piece + 255) / 256 * 256 * pkv::kInplaceStreams; }
bool reserve_inplace(proxykv_ctx* ctx, size_t piece) {
  pkv::InplaceCounters& c = ctx->inplace;
  size_t bytes = inplace_block_bytes(piece);
  if (bytes <= c.block.bytes) return true;
  bytes = std::max(bytes, 2 * c.block.bytes);
  if (c.block.ptr && c.n_older == (int)(sizeof(c.older) / sizeof(c.older[0]))) return false;
  // (another stream's capture does not forbid it: nothing that is captured has to do with this memory)
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (!hip_ok(ctx, hipThreadExchangeStreamCaptureMode(&mode))) return false;
  void* p = nullptr;
  const hipError_t e = hipMalloc(&p, bytes);
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (!hip_ok(ctx, e)) return false;
  if (c.block.ptr) c.older[c.n_older++] = c.block.ptr;
  c.block = {p, bytes};
  return true;
}
// The counters of a call on `stream`, whose calls follow each other; nullptr where there is no room for them or for another stream.  (The mutex is held.)
void* inplace_counters(proxykv_ctx* ctx, size_t bytes, hipStream_t stream) {
  pkv::InplaceCounters& c = ctx->inplace;
  if (stream == hipStreamPerThread) return nullptr;  // the same handle in every thread, and not the same stream
  int i = 0;
  while (i < c.streams && c.stream[i] != stream) ++i;
  if (i == pkv::kInplaceStreams || !reserve_inplace(ctx, bytes)) return nullptr;
  if (i == c.streams) c.stream[c.streams++] = stream;
  return (uint8_t*)c.block.ptr + c.block.bytes / pkv::kInplaceStreams * i;
}
// Whole rows are moved without counters: where rows are short, where there are no counters to be had, and while the stream captures.  A graph may
// be replayed on any stream, after a later call has taken other memory and after the context is gone, so a captured call holds the
// caller's pointers only.  (Half of 512 rows of 12 345 tokens, 652 us replayed instead of 548.)
int inplace_impl(proxykv_ctx* ctx, void* k, void* v, const int32_t* idx, int64_t rows, int64_t N, int64_t K, int64_t row_bytes, const int32_t* counts,
                 int heads, hipStream_t stream) {
  const size_t need = pkv::compact_inplace_scratch_bytes(rows, K, row_bytes, heads);
  std::unique_lock<std::mutex> lock(ctx->inplace.mutex, std::defer_lock);
  void* counters = nullptr;
  if (need > 0 && !capturing(stream)) {
    lock.lock();
    counters = inplace_counters(ctx, need, stream);
  }
  PKV_HIP(ctx, pkv::launch_compact_inplace(k, v, idx, rows, N, K, row_bytes, counts, heads, counters, counters ? need : 0, stream));
  return PROXYKV_OK;
}
// What the counters take for any number of kept tokens of this context's rows, with a budget per head or per layer
size_t inplace_bytes(const proxykv_config& c, int64_t N) {
  if (c.D * 2 > 512) return 0;  // not for proxykv_compact_inplace
  const int64_t rows = (int64_t)c.L_l * c.H_l;
  const size_t own = pkv::compact_inplace_scratch_most(rows, N, c.D * 2, 1), shared = pkv::compact_inplace_scratch_most(rows, N, c.D * 2, c.H_l);
  return own > shared ? own : shared;
}
int reserve_prune(proxykv_ctx* ctx, int64_t N, hipStream_t stream) {
  const Sizes s = workspace_sizes(ctx->cfg, N, 1);
  int rc = ensure(ctx, ctx->x_ws, s.x_ws, stream);
  if (rc == PROXYKV_OK) rc = ensure(ctx, ctx->yhat_ws, s.yhat_ws, stream);
  if (rc == PROXYKV_OK) rc = reserve_topk(ctx, (int64_t)ctx->cfg.L_l * ctx->cfg.H_l, N, stream);
  return rc;
}

// fp32 -> IEEE half bits, round to nearest even (subnormals and overflow to infinity included)
uint16_t host_f16(float f) {
  uint32_t x;
  memcpy(&x, &f, 4);
  const uint16_t sign = (uint16_t)((x >> 16) & 0x8000u);
  const uint32_t ax = x & 0x7fffffffu;
  if (ax > 0x7f800000u) return (uint16_t)(sign | 0x7e00u);
  if (ax >= 0x477ff000u) return (uint16_t)(sign | 0x7c00u);  // >= 65520 rounds to infinity
  if (ax < 0x38800000u) {                                      // below 2^-14: half subnormal, unit 2^-24
    float a;
    memcpy(&a, &ax, 4);
    return (uint16_t)(sign | (uint32_t)nearbyint((double)a * 16777216.0));
  }
  const uint32_t mant = ax & 0x7fffffu, exp = (ax >> 23) - 127 + 15;
  uint32_t h = (exp << 10) | (mant >> 13);
  const uint32_t rem = mant & 0x1fffu;
  if (rem > 0x1000u || (rem == 0x1000u && (h & 1u))) ++h;
  return (uint16_t)(sign | h);
}

// Builds the prepared weight image on the host: a byte vector plus offsets of every section.
struct Stager {
  std::vector<uint8_t> bytes;
  size_t put_f32(const float* src, size_t n) {
    const size_t off = (bytes.size() + 255) & ~(size_t)255;
    bytes.resize(off + n * 4);
    memcpy(bytes.data() + off, src, n * 4);
    return off;
  }
  size_t put_f16(const float* src, size_t n) {
    const size_t off = (bytes.size() + 255) & ~(size_t)255;
    bytes.resize(off + n * 2);
    uint16_t* d = reinterpret_cast<uint16_t*>(bytes.data() + off);
    for (size_t i = 0; i < n; ++i) d[i] = host_f16(src[i]);
    return off;
  }
};

// Records stage boundary `i` on the stream when stage timing is switched on.
int mark(proxykv_ctx* ctx, int i, hipStream_t stream) {
  if (!ctx->profile) return PROXYKV_OK;
  PKV_HIP(ctx, hipEventRecord(ctx->ev[i], stream));
  ctx->ev_recorded[i] = true;
  return PROXYKV_OK;
}

int score_impl(proxykv_ctx* ctx, const void* q_rec, const void* k_ctx, const void* k_rec, int32_t dtype, int64_t N,
               int64_t N_q, int32_t chunk, float* x_out, hipStream_t stream) {
  const proxykv_config& c = ctx->cfg;
  const uint16_t *q = (const uint16_t*)q_rec, *kc = (const uint16_t*)k_ctx, *kr = (const uint16_t*)k_rec;
  const bool rounds = dtype == PROXYKV_FP32 && pkv::score_rounds_itself(c.L_s, c.H_q, c.H_kv, c.d, N, N_q);
  int rc;
  if (dtype == PROXYKV_FP32) {
    const size_t nq = (size_t)c.L_s * c.H_q * (size_t)N_q * c.d, nkc = (size_t)c.L_s * c.H_kv * (size_t)N * c.d,
                 nkr = (size_t)c.L_s * c.H_kv * (size_t)N_q * c.d;
    if ((rc = ensure(ctx, ctx->q_bf16, nq * 2, stream))) return rc;
    if ((rc = ensure(ctx, ctx->kctx_bf16, nkc * 2, stream))) return rc;
    if ((rc = ensure(ctx, ctx->krec_bf16, nkr * 2, stream))) return rc;
    const float* const in[3] = {(const float*)q_rec, (const float*)k_ctx, (const float*)k_rec};
    uint16_t* const out[3] = {(uint16_t*)ctx->q_bf16.ptr, (uint16_t*)ctx->kctx_bf16.ptr, (uint16_t*)ctx->krec_bf16.ptr};
    const int64_t n[3] = {(int64_t)nq, (int64_t)nkc, (int64_t)nkr};
    if (!rounds) PKV_HIP(ctx, pkv::launch_f32_to_bf16(in, out, n, stream));
    q = (const uint16_t*)ctx->q_bf16.ptr;
    kc = (const uint16_t*)ctx->kctx_bf16.ptr;
    kr = (const uint16_t*)ctx->krec_bf16.ptr;
  }
  const bool sum = c.reduce == PROXYKV_REDUCE_SUM;
  if ((rc = reserve_score(ctx, N, N_q, sum, stream))) return rc;
  float* nl = (float*)ctx->neg_lse.ptr;
  int rcm;
  if ((rcm = mark(ctx, 0, stream))) return rcm;
  const int splits = pkv::score_splits(c.L_s, c.H_q, c.d, N, N_q);
  const int q_splits = query_splits(ctx, sum, false, N, N_q);
  const int64_t n_clear = !sum && (splits > 1 || q_splits > 1) ? (int64_t)c.L_s * c.H_kv * N : 0;
  if (rounds)
    PKV_HIP(ctx, pkv::launch_score_lse_fp32((const float*)q_rec, (const float*)k_ctx, (const float*)k_rec, nl, splits, x_out, n_clear,
                                            (uint16_t*)ctx->q_bf16.ptr, (uint16_t*)ctx->kctx_bf16.ptr, c.L_s, c.H_q, c.H_kv, c.d, N, N_q, chunk, stream));
  else
    PKV_HIP(ctx, pkv::launch_score_lse(q, kc, kr, nl, splits, x_out, n_clear, c.L_s, c.H_q, c.H_kv, c.d, N, N_q, chunk, stream));
  if ((rcm = mark(ctx, 1, stream))) return rcm;
  if (sum)
    PKV_HIP(ctx, pkv::launch_score_colsum(q, kc, nl, splits, x_out, (float*)ctx->x_parts.ptr, q_splits, c.L_s, c.H_q, c.H_kv, c.d, N, N_q, false, stream));
  else
    PKV_HIP(ctx, pkv::launch_score_colmax(q, kc, nl, splits, x_out, q_splits, c.L_s, c.H_q, c.H_kv, c.d, N, N_q, stream));
  if ((rcm = mark(ctx, 2, stream))) return rcm;
  return PROXYKV_OK;
}

// causal self-attention, summed over the query axis: pass 1 with no context keys and one chunk that spans the
// sequence (query i sees its own keys j <= i), then the causal column sum
int score_self_impl(proxykv_ctx* ctx, const void* q_in, const void* k_in, int32_t dtype, int64_t N, float* x_out,
                    hipStream_t stream) {
  const proxykv_config& c = ctx->cfg;
  const uint16_t *q = (const uint16_t*)q_in, *k = (const uint16_t*)k_in;
  const bool rounds = dtype == PROXYKV_FP32 && pkv::score_rounds_itself(c.L_s, c.H_q, c.H_kv, c.d, N, N);
  int rc;
  if (dtype == PROXYKV_FP32) {
    const size_t nq = (size_t)c.L_s * c.H_q * (size_t)N * c.d, nk = (size_t)c.L_s * c.H_kv * (size_t)N * c.d;
    if ((rc = ensure(ctx, ctx->q_bf16, nq * 2, stream))) return rc;
    if ((rc = ensure(ctx, ctx->krec_bf16, nk * 2, stream))) return rc;
    const float* const in[3] = {(const float*)q_in, (const float*)k_in, nullptr};
    uint16_t* const out[3] = {(uint16_t*)ctx->q_bf16.ptr, (uint16_t*)ctx->krec_bf16.ptr, nullptr};
    const int64_t n[3] = {(int64_t)nq, (int64_t)nk, 0};
    if (!rounds) PKV_HIP(ctx, pkv::launch_f32_to_bf16(in, out, n, stream));
    q = (const uint16_t*)ctx->q_bf16.ptr;
    k = (const uint16_t*)ctx->krec_bf16.ptr;
  }
  if ((rc = reserve_score(ctx, N, N, true, stream))) return rc;
  float* nl = (float*)ctx->neg_lse.ptr;
  int rcm;
  if ((rcm = mark(ctx, 0, stream))) return rcm;
  const int splits = pkv::score_splits(c.L_s, c.H_q, c.d, N, N);
  const int q_splits = query_splits(ctx, true, true, N, N);
  if (rounds)
    PKV_HIP(ctx, pkv::launch_score_lse_fp32((const float*)q_in, (const float*)k_in, (const float*)k_in, nl, splits, x_out, 0,
                                            (uint16_t*)ctx->q_bf16.ptr, (uint16_t*)ctx->krec_bf16.ptr, c.L_s, c.H_q, c.H_kv, c.d, 0, N, (int)N, stream));
  else
    PKV_HIP(ctx, pkv::launch_score_lse(q, k, k, nl, splits, x_out, 0, c.L_s, c.H_q, c.H_kv, c.d, 0, N, (int)N, stream));
  if ((rcm = mark(ctx, 1, stream))) return rcm;
  PKV_HIP(ctx, pkv::launch_score_colsum(q, k, nl, splits, x_out, (float*)ctx->x_parts.ptr, q_splits, c.L_s, c.H_q, c.H_kv, c.d, N, N, true, stream));
  if ((rcm = mark(ctx, 2, stream))) return rcm;
  return PROXYKV_OK;
}

int map_impl(proxykv_ctx* ctx, const float* x, int64_t N, float* yhat, hipStream_t stream) {
  int rc;
  pkv::MapPlan p;
  if ((rc = reserve_map(ctx, N, stream, &p))) return rc;
  PKV_HIP(ctx, pkv::mapper_forward(ctx, p, x, yhat, stream));
  return PROXYKV_OK;
}

}  // namespace

extern "C" {

void proxykv_default_mapper(proxykv_config* cfg) {
  if (!cfg) return;
  cfg->d_time = 512;
  cfg->c_mid = 256;
  cfg->n_enc_layers = 6;
  cfg->n_enc_heads = 8;
  cfg->d_ffn = 2048;
  cfg->d_head_x = 64;
  cfg->win = 2048;
  cfg->stride = 1024;
  cfg->reduce = PROXYKV_REDUCE_MAX;
  cfg->device = 0;
}

int proxykv_create(proxykv_ctx** out, const proxykv_config* cfg) {
  if (!out) return PROXYKV_EINVAL;
  *out = nullptr;
  const int rc = validate_config(cfg);
  if (rc) return rc;
  proxykv_ctx* ctx = new (std::nothrow) proxykv_ctx();
  if (!ctx) return PROXYKV_ENOMEM;
  ctx->cfg = *cfg;
  ctx->pairing.resize(cfg->L_l);
  for (int ll = 0; ll < cfg->L_l; ++ll)
    ctx->pairing[ll] = (int32_t)(((int64_t)(ll + 1) * cfg->L_s + cfg->L_l - 1) / cfg->L_l - 1);
  ctx->distinct_layers = count_distinct(*cfg);
  *out = ctx;
  return PROXYKV_OK;
}

int proxykv_destroy(proxykv_ctx* ctx) {
  if (!ctx) return PROXYKV_OK;
  std::vector<DeviceBuffer*> all = {&ctx->weight_blob, &ctx->block_blob, &ctx->q_bf16, &ctx->kctx_bf16, &ctx->krec_bf16,
                                    &ctx->neg_lse, &ctx->x_parts, &ctx->x_ws,   &ctx->yhat_ws, &ctx->topk_ws, &ctx->inplace.block};
  for (pkv::MapperWorkspace& m : ctx->m) {
    DeviceBuffer* b[kLaneBuffers];
    lane_buffers(m, b);
    all.insert(all.end(), b, b + kLaneBuffers);
  }
  bool any = ctx->ev_created || ctx->lanes_created;
  for (DeviceBuffer* b : all) any = any || b->ptr;
  if (any) {
    (void)hipSetDevice(ctx->cfg.device);
    (void)hipDeviceSynchronize();
    for (DeviceBuffer* b : all) free_buffer(*b);
    for (int i = 0; i < ctx->inplace.n_older; ++i) (void)hipFree(ctx->inplace.older[i]);
    if (ctx->ev_created)
      for (int i = 0; i < PROXYKV_N_STAGES + 1; ++i) (void)hipEventDestroy(ctx->ev[i]);
    for (int i = 1; i < pkv::kMapLanes; ++i) {
      if (ctx->lane_stream[i]) (void)hipStreamDestroy(ctx->lane_stream[i]);
      if (ctx->lane_join[i]) (void)hipEventDestroy(ctx->lane_join[i]);
    }
    if (ctx->lane_fork) (void)hipEventDestroy(ctx->lane_fork);
  }
  delete ctx;
  return PROXYKV_OK;
}

size_t proxykv_mapper_weight_count(const proxykv_config* c) {
  if (validate_config(c)) return 0;
  const size_t D = c->d_time, C1 = c->c_mid, F = c->d_ffn, dh = c->d_head_x, Hs = c->H_kv, Hl = c->H_l;
  size_t n = C1 * Hs * 3 + C1 + 4 * C1 + D * C1 * 3 + D + 4 * D;
  n += (size_t)c->n_enc_layers * (3 * D * D + 3 * D + D * D + D + 2 * D + F * D + F + D * F + D + 2 * D);
  n += 2 * (Hs * dh * D + Hs * dh) + Hl * dh + dh + 1;
  return n;
}

int proxykv_set_mapper_weights(proxykv_ctx* ctx, const float* blob, size_t n_floats) {
  if (!ctx || !blob) return PROXYKV_EINVAL;
  const proxykv_config& c = ctx->cfg;
  if (n_floats != proxykv_mapper_weight_count(&c)) return PROXYKV_EINVAL;
  const size_t D = c.d_time, C1 = c.c_mid, F = c.d_ffn, dh = c.d_head_x, Hs = c.H_kv, Hl = c.H_l;
  const double eps = 1e-5;
  const float* p = blob;
  auto take = [&](size_t n) {
    const float* r = p;
    p += n;
    return r;
  };
  Stager st;
  // stem: fold conv bias and inference batch norm into scale/shift (host double arithmetic)
  auto fold = [&](const float* bias, const float* g, const float* b, const float* mu, const float* var, size_t n,
                  size_t* off_scale, size_t* off_shift) {
    std::vector<float> sc(n), sh(n);
    for (size_t i = 0; i < n; ++i) {
      const double s = (double)g[i] / sqrt((double)var[i] + eps);
      sc[i] = (float)s;
      sh[i] = (float)(((double)bias[i] - (double)mu[i]) * s + (double)b[i]);
    }
    *off_scale = st.put_f32(sc.data(), n);
    *off_shift = st.put_f32(sh.data(), n);
  };
  const float* c1w = take(C1 * Hs * 3);
  const float* c1b = take(C1);
  const float *g1 = take(C1), *b1 = take(C1), *m1 = take(C1), *v1 = take(C1);
  std::vector<float> c1t(C1 * Hs * 3);  // a channel's weights lie C1 apart: the kernel's lanes are channels
  for (size_t ch = 0; ch < C1; ++ch)
    for (size_t i = 0; i < Hs * 3; ++i) c1t[i * C1 + ch] = c1w[ch * Hs * 3 + i];
  const size_t o_c1w = st.put_f32(c1t.data(), c1t.size());
  size_t o_s1, o_h1;
  fold(c1b, g1, b1, m1, v1, C1, &o_s1, &o_h1);
  // bound of the first block's output, |GELU(y)| <= |y| <= |scale_c| * sum |w_c| * max|x| + |shift_c|
  double cw = 0.0, cs = 0.0;
  for (size_t ch = 0; ch < C1; ++ch) {
    const double sgn = (double)g1[ch] / sqrt((double)v1[ch] + eps), sc = fabs(sgn);
    double wsum = 0.0;
    for (size_t i = 0; i < Hs * 3; ++i) wsum += fabs((double)c1w[ch * Hs * 3 + i]);
    const double sh = fabs(((double)c1b[ch] - (double)m1[ch]) * sgn + (double)b1[ch]);
    if (sc * wsum > cw) cw = sc * wsum;
    if (sh > cs) cs = sh;
  }
  ctx->w.stem_cw = (float)(cw * 1.0001);
  ctx->w.stem_cs = (float)(cs * 1.0001 + 1e-6);
  const float* c2w = take(D * C1 * 3);
  const float* c2b = take(D);
  const float *g2 = take(D), *b2 = take(D), *m2 = take(D), *v2 = take(D);
  std::vector<float> c2r(D * C1 * 3);  // [c][c1][tap] -> [c][tap][c1]
  for (size_t co = 0; co < D; ++co)
    for (size_t ci = 0; ci < C1; ++ci)
      for (size_t tap = 0; tap < 3; ++tap) c2r[(co * 3 + tap) * C1 + ci] = c2w[(co * C1 + ci) * 3 + tap];
  const size_t o_c2w = st.put_f16(c2r.data(), c2r.size());
  size_t o_s2, o_h2;
  fold(c2b, g2, b2, m2, v2, D, &o_s2, &o_h2);
  struct EncOff {
    size_t in_w, in_b, out_w, out_b, ln1_g, ln1_b, f1_w, f1_b, f2_w, f2_b, ln2_g, ln2_b;
  };
  std::vector<EncOff> eo(c.n_enc_layers);
  for (int i = 0; i < c.n_enc_layers; ++i) {
    EncOff& e = eo[i];
    e.in_w = st.put_f16(take(3 * D * D), 3 * D * D);
    e.in_b = st.put_f32(take(3 * D), 3 * D);
    e.out_w = st.put_f16(take(D * D), D * D);
    e.out_b = st.put_f32(take(D), D);
    e.ln1_g = st.put_f32(take(D), D);
    e.ln1_b = st.put_f32(take(D), D);
    e.f1_w = st.put_f16(take(F * D), F * D);
    e.f1_b = st.put_f32(take(F), F);
    e.f2_w = st.put_f16(take(D * F), D * F);
    e.f2_b = st.put_f32(take(D), D);
    e.ln2_g = st.put_f32(take(D), D);
    e.ln2_b = st.put_f32(take(D), D);
  }
  // head: key and value projections stacked into one [2*Hs*dh, D] matrix
  const float* kw = take(Hs * dh * D);
  const float* kb = take(Hs * dh);
  const float* vw = take(Hs * dh * D);
  const float* vb = take(Hs * dh);
  // rows padded with zeros to the GEMM's 256-column tile (pkv::kv3_stride)
  const size_t kv_rows = (size_t)pkv::kv3_stride(c);
  std::vector<float> kvw(kv_rows * D, 0.0f), kvb(kv_rows, 0.0f);
  memcpy(kvw.data(), kw, Hs * dh * D * 4);
  memcpy(kvw.data() + Hs * dh * D, vw, Hs * dh * D * 4);
  memcpy(kvb.data(), kb, Hs * dh * 4);
  memcpy(kvb.data() + Hs * dh, vb, Hs * dh * 4);
  const size_t o_kvw = st.put_f16(kvw.data(), kvw.size());
  const size_t o_kvb = st.put_f32(kvb.data(), kvb.size());
  const size_t o_q = st.put_f32(take(Hl * dh), Hl * dh);
  const size_t o_ow = st.put_f32(take(dh), dh);
  const float out_b = *take(1);
  // sinusoidal positions 0 .. win-1 (Sec. 4.1, stage 2), evaluated in double
  std::vector<float> pe((size_t)c.win * D);
  for (int pos = 0; pos < c.win; ++pos)
    for (size_t i = 0; i < D; i += 2) {
      const double ang = (double)pos / pow(10000.0, (double)i / (double)D);
      pe[(size_t)pos * D + i] = (float)sin(ang);
      pe[(size_t)pos * D + i + 1] = (float)cos(ang);
    }
  const size_t o_pe = st.put_f32(pe.data(), pe.size());

  PKV_HIP(ctx, hipSetDevice(c.device));
  int rc = ensure(ctx, ctx->weight_blob, st.bytes.size(), nullptr);
  if (rc) return rc;
  PKV_HIP(ctx, hipMemcpy(ctx->weight_blob.ptr, st.bytes.data(), st.bytes.size(), hipMemcpyHostToDevice));
  const uint8_t* base = (const uint8_t*)ctx->weight_blob.ptr;
  auto F32 = [&](size_t off) { return (const float*)(base + off); };
  auto B16 = [&](size_t off) { return (const uint16_t*)(base + off); };
  pkv::MapperWeights& w = ctx->w;
  w.conv1_w = F32(o_c1w);
  w.bn1_scale = F32(o_s1);
  w.bn1_shift = F32(o_h1);
  w.conv2_w = B16(o_c2w);
  w.bn2_scale = F32(o_s2);
  w.bn2_shift = F32(o_h2);
  w.enc.resize(c.n_enc_layers);
  for (int i = 0; i < c.n_enc_layers; ++i) {
    const EncOff& e = eo[i];
    w.enc[i] = {B16(e.in_w), F32(e.in_b), B16(e.out_w), F32(e.out_b), F32(e.ln1_g), F32(e.ln1_b),
                B16(e.f1_w), F32(e.f1_b), B16(e.f2_w),  F32(e.f2_b),  F32(e.ln2_g), F32(e.ln2_b)};
  }
  w.kv_w = B16(o_kvw);
  w.kv_b = F32(o_kvb);
  w.queries = F32(o_q);
  w.out_w = F32(o_ow);
  w.out_b = out_b;
  w.pe = F32(o_pe);
  if (c.n_enc_layers > 0) {
    size_t frags = 0, bias_frags = 0;
    for (int li = 0; li <= c.n_enc_layers; ++li) {
      frags += 4 * pkv::block_frags(c, li);
      bias_frags += 4 * pkv::block_bias_frags(c, li);
    }
    const size_t w_bytes = (frags + pkv::kBlkRing) * pkv::kBlkFragBytes;  // the last wave asks for as much beyond its last
    rc = ensure(ctx, ctx->block_blob, w_bytes + (bias_frags + 4) * pkv::kBlkFragBytes, nullptr);
    if (rc) return rc;
    void* bias = (uint8_t*)ctx->block_blob.ptr + w_bytes;
    PKV_HIP(ctx, pkv::pack_encoder_blocks(c, w, ctx->block_blob.ptr, bias, nullptr));
    PKV_HIP(ctx, hipStreamSynchronize(nullptr));
    w.blk_w = ctx->block_blob.ptr;
    w.blk_b = bias;
  }
  ctx->weights_set = true;
  return PROXYKV_OK;
}

int proxykv_workspace_bytes(const proxykv_config* cfg, int64_t N, int64_t N_q, size_t* out_bytes) {
  if (!out_bytes) return PROXYKV_EINVAL;
  int rc = validate_config(cfg);
  if (rc) return rc;
  if ((rc = validate_lengths(N, N_q, 1))) return rc;
  const int distinct = count_distinct(*cfg);
  const Sizes s = workspace_sizes(*cfg, N, N_q);
  const pkv::MapPlan p = pkv::map_plan(*cfg, N, distinct);
  const LaneBytes lb = lane_bytes(*cfg, p);
  size_t total = s.neg_lse + s.x_parts + s.x_ws + s.yhat_ws + pkv::topk_scratch_bytes((int64_t)cfg->L_l * cfg->H_l, N) + inplace_block_bytes(inplace_bytes(*cfg, N));
  for (int lane = 0; lane < p.lanes; ++lane)
    for (int i = 0; i < kLaneBuffers; ++i) total += lane_need(*cfg, p, lb, lane, distinct, i);
  *out_bytes = total;
  return PROXYKV_OK;
}

int proxykv_reserve(proxykv_ctx* ctx, int64_t N, int64_t N_q) {
  if (!ctx) return PROXYKV_EINVAL;
  int rc = validate_lengths(N, N_q, 1);
  if (rc) return rc;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  if ((rc = reserve_score(ctx, N, N_q, true, nullptr))) return rc;  // (proxykv_score_self has parts in any context)
  if ((rc = reserve_prune(ctx, N, nullptr))) return rc;
  {
    std::lock_guard<std::mutex> lock(ctx->inplace.mutex);
    (void)reserve_inplace(ctx, inplace_bytes(ctx->cfg, N));  // (in-place calls do without)
  }
  pkv::MapPlan p;
  return reserve_map(ctx, N, nullptr, &p);  // last: it makes do with what is left
}

int proxykv_keep_count(int64_t N, double keep_ratio, int64_t* K_out) {
  if (!K_out || N <= 0 || !(keep_ratio > 0.0) || !(keep_ratio <= 1.0)) return PROXYKV_EINVAL;
  int64_t K = (int64_t)floor(keep_ratio * (double)N);
  if (K < 1) K = 1;
  if (K > N) K = N;
  *K_out = K;
  return PROXYKV_OK;
}

int proxykv_layer_pairing(const proxykv_config* cfg, int32_t* pairing_host) {
  if (!cfg || !pairing_host || cfg->L_s <= 0 || cfg->L_l <= 0) return PROXYKV_EINVAL;
  for (int ll = 0; ll < cfg->L_l; ++ll)
    pairing_host[ll] = (int32_t)(((int64_t)(ll + 1) * cfg->L_s + cfg->L_l - 1) / cfg->L_l - 1);
  return PROXYKV_OK;
}

int proxykv_score(proxykv_ctx* ctx, const void* q_rec, const void* k_ctx, const void* k_rec, int32_t dtype, int64_t N,
                  int64_t N_q, int32_t chunk, float* x_out, void* stream) {
  if (!ctx || !q_rec || !k_ctx || !k_rec || !x_out) return PROXYKV_EINVAL;
  if (dtype != PROXYKV_BF16 && dtype != PROXYKV_FP32) return PROXYKV_EINVAL;
  const int rc = validate_lengths(N, N_q, chunk);
  if (rc) return rc;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  // stage timing describes a whole proxykv_prune: a score call on its own leaves no complete record behind
  const int rcs = score_impl(ctx, q_rec, k_ctx, k_rec, dtype, N, N_q, chunk, x_out, (hipStream_t)stream);
  for (int i = 0; i < PROXYKV_N_STAGES + 1; ++i) ctx->ev_recorded[i] = false;
  return rcs;
}

int proxykv_score_self(proxykv_ctx* ctx, const void* q, const void* k, int32_t dtype, int64_t N, float* x_out, void* stream) {
  if (!ctx || !q || !k || !x_out) return PROXYKV_EINVAL;
  if (dtype != PROXYKV_BF16 && dtype != PROXYKV_FP32) return PROXYKV_EINVAL;
  const int rc = validate_lengths(N, N, N);
  if (rc) return rc;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  const int rcs = score_self_impl(ctx, q, k, dtype, N, x_out, (hipStream_t)stream);
  for (int i = 0; i < PROXYKV_N_STAGES + 1; ++i) ctx->ev_recorded[i] = false;
  return rcs;
}

int proxykv_map(proxykv_ctx* ctx, const float* x, int64_t N, float* yhat, void* stream) {
  if (!ctx || !x || !yhat) return PROXYKV_EINVAL;
  const int rc = validate_lengths(N, 1, 1);
  if (rc) return rc;
  if (!ctx->weights_set) return PROXYKV_ESTATE;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  return map_impl(ctx, x, N, yhat, (hipStream_t)stream);
}

int proxykv_topk(proxykv_ctx* ctx, const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out,
                 void* stream) {
  if (!ctx || !scores || !idx_out) return PROXYKV_EINVAL;
  if (rows <= 0 || rows >= (1ll << 31) || N <= 0 || N >= (1ll << 31) - 4096 || K < 1 || K > N) return PROXYKV_EINVAL;
  if (N > pkv::kTopkSingleMax && rows > 65535) return PROXYKV_EUNSUPPORTED;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  const int rc = reserve_topk(ctx, rows, N, (hipStream_t)stream);
  if (rc) return rc;
  PKV_HIP(ctx, pkv::launch_topk(scores, rows, N, K, idx_out, ctx->topk_ws.ptr, ctx->topk_ws.bytes, (hipStream_t)stream));
  return PROXYKV_OK;
}

int proxykv_compact(proxykv_ctx* ctx, const void* k_in, const void* v_in, const int32_t* idx, int64_t rows, int64_t N,
                    int64_t K, int64_t D, void* k_out, void* v_out, void* stream) {
  if (!ctx || !k_in || !v_in || !idx || !k_out || !v_out) return PROXYKV_EINVAL;
  if (rows <= 0 || rows > 65535 || N <= 0 || N >= (1ll << 31) || K < 1 || K > N || D <= 0) return PROXYKV_EINVAL;
  if ((D * 2) % 16 != 0 || D * 2 > 4096 || 256 % ((D * 2) / 16) != 0) return PROXYKV_EUNSUPPORTED;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  PKV_HIP(ctx, pkv::launch_compact(k_in, v_in, idx, rows, N, K, D * 2, k_out, v_out, (hipStream_t)stream));
  return PROXYKV_OK;
}

int proxykv_compact_inplace(proxykv_ctx* ctx, void* k, void* v, const int32_t* idx, int64_t rows, int64_t N, int64_t K,
                            int64_t D, void* stream) {
  if (!ctx || !k || !v || !idx) return PROXYKV_EINVAL;
  if (rows <= 0 || N <= 0 || N >= (1ll << 31) || K < 1 || K > N || D <= 0) return PROXYKV_EINVAL;
  if ((D * 2) % 16 != 0 || D * 2 > 512) return PROXYKV_EUNSUPPORTED;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  return inplace_impl(ctx, k, v, idx, rows, N, K, D * 2, nullptr, 1, (hipStream_t)stream);
}

int proxykv_topk_pooled(proxykv_ctx* ctx, const float* scores, int64_t layers, int64_t heads, int64_t N, int64_t K,
                        int32_t* flat_out, int32_t* counts_out, void* stream) {
  if (!ctx || !scores || !flat_out || !counts_out) return PROXYKV_EINVAL;
  if (layers <= 0 || heads <= 0 || N <= 0 || K < 1 || K > N) return PROXYKV_EINVAL;
  if (layers * heads >= (1ll << 31) || heads * N >= (1ll << 31) - 4096) return PROXYKV_EINVAL;
  if (heads * N > pkv::kTopkSingleMax && layers > 65535) return PROXYKV_EUNSUPPORTED;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  const int rc = reserve_topk(ctx, layers, heads * N, (hipStream_t)stream);
  if (rc) return rc;
  PKV_HIP(ctx, pkv::launch_topk(scores, layers, heads * N, heads * K, flat_out, ctx->topk_ws.ptr, ctx->topk_ws.bytes, (hipStream_t)stream));
  PKV_HIP(ctx, pkv::launch_head_counts(flat_out, layers, heads, N, K, counts_out, (hipStream_t)stream));
  return PROXYKV_OK;
}

int proxykv_compact_pooled(proxykv_ctx* ctx, void* k, void* v, const int32_t* flat, const int32_t* counts, int64_t layers,
                           int64_t heads, int64_t N, int64_t K, int64_t D, void* stream) {
  if (!ctx || !k || !v || !flat || !counts) return PROXYKV_EINVAL;
  if (layers <= 0 || heads <= 0 || N <= 0 || K < 1 || K > N || D <= 0) return PROXYKV_EINVAL;
  if (layers * heads >= (1ll << 31) || heads * N >= (1ll << 31) - 4096) return PROXYKV_EINVAL;
  if ((D * 2) % 16 != 0 || D * 2 > 512) return PROXYKV_EUNSUPPORTED;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  return inplace_impl(ctx, k, v, flat, layers * heads, N, K, D * 2, counts, (int)heads, (hipStream_t)stream);
}

int proxykv_mask(proxykv_ctx* ctx, const int32_t* idx, int64_t rows, int64_t N, int64_t K, uint8_t* mask_out, void* stream) {
  if (!ctx || !idx || !mask_out) return PROXYKV_EINVAL;
  if (rows <= 0 || N <= 0 || N >= (1ll << 31) || K < 1 || K > N) return PROXYKV_EINVAL;
  PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
  PKV_HIP(ctx, pkv::launch_mask(idx, rows, N, K, mask_out, (hipStream_t)stream));
  return PROXYKV_OK;
}

int proxykv_prune(proxykv_ctx* ctx, const void* q_rec, const void* k_ctx, const void* k_rec, int32_t dtype, int64_t N,
                  int64_t N_q, int32_t chunk, double keep_ratio, const void* k_in, const void* v_in, void* k_out,
                  void* v_out, int32_t* idx_out, float* x_out, float* yhat_out, int64_t* K_host, void* stream) {
  if (!ctx || !q_rec || !k_ctx || !k_rec || !k_in || !v_in || !k_out || !v_out || !idx_out) return PROXYKV_EINVAL;
  if (dtype != PROXYKV_BF16 && dtype != PROXYKV_FP32) return PROXYKV_EINVAL;
  int rc = validate_lengths(N, N_q, chunk);
  if (rc) return rc;
  int64_t K = 0;
  if ((rc = proxykv_keep_count(N, keep_ratio, &K))) return rc;
  if (!ctx->weights_set) return PROXYKV_ESTATE;
  const proxykv_config& c = ctx->cfg;
  const int64_t rows = (int64_t)c.L_l * c.H_l;
  if (rows > 65535 || 256 % ((c.D * 2) / 16) != 0) return PROXYKV_EUNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  PKV_HIP(ctx, hipSetDevice(c.device));
  pkv::MapPlan plan;  // everything is there before the first launch
  if ((rc = reserve_score(ctx, N, N_q, c.reduce == PROXYKV_REDUCE_SUM, s)) || (rc = reserve_prune(ctx, N, s)) || (rc = reserve_map(ctx, N, s, &plan)))
    return rc;
  float* x = x_out ? x_out : (float*)ctx->x_ws.ptr;
  float* y = yhat_out ? yhat_out : (float*)ctx->yhat_ws.ptr;
  if ((rc = score_impl(ctx, q_rec, k_ctx, k_rec, dtype, N, N_q, chunk, x, s))) return rc;
  if ((rc = map_impl(ctx, x, N, y, s))) return rc;
  if ((rc = mark(ctx, 3, s))) return rc;
  const int cpr = c.D * 2 / 16;
  if (ctx->fused_select && 1024 % cpr == 0) {
    // selection and gather in one launch: the workgroup that has written a stretch of a row's kept indices moves those
    // tokens' K and V rows; the whole launch is booked as the compaction stage
    if ((rc = mark(ctx, 4, s))) return rc;
    PKV_HIP(ctx, pkv::launch_topk_gather(y, rows, N, K, idx_out, ctx->topk_ws.ptr, ctx->topk_ws.bytes, k_in, v_in, (int64_t)c.D * 2, k_out, v_out, s));
  } else {
    PKV_HIP(ctx, pkv::launch_topk(y, rows, N, K, idx_out, ctx->topk_ws.ptr, ctx->topk_ws.bytes, s));
    if ((rc = mark(ctx, 4, s))) return rc;
    PKV_HIP(ctx, pkv::launch_compact(k_in, v_in, idx_out, rows, N, K, (int64_t)c.D * 2, k_out, v_out, s));
  }
  if ((rc = mark(ctx, 5, s))) return rc;
  if (K_host) *K_host = K;
  return PROXYKV_OK;
}

int proxykv_set_fused_select(proxykv_ctx* ctx, int on) {
  if (!ctx) return PROXYKV_EINVAL;
  ctx->fused_select = on != 0;
  return PROXYKV_OK;
}

int proxykv_profile_enable(proxykv_ctx* ctx, int on) {
  if (!ctx) return PROXYKV_EINVAL;
  if (on && !ctx->ev_created) {
    PKV_HIP(ctx, hipSetDevice(ctx->cfg.device));
    for (int i = 0; i < PROXYKV_N_STAGES + 1; ++i) PKV_HIP(ctx, hipEventCreate(&ctx->ev[i]));
    ctx->ev_created = true;
  }
  ctx->profile = on != 0;
  for (int i = 0; i < PROXYKV_N_STAGES + 1; ++i) ctx->ev_recorded[i] = false;
  return PROXYKV_OK;
}

int proxykv_profile_read(proxykv_ctx* ctx, float* ms_host) {
  if (!ctx || !ms_host) return PROXYKV_EINVAL;
  if (!ctx->profile || !ctx->ev_created) return PROXYKV_ESTATE;
  for (int i = 0; i < PROXYKV_N_STAGES + 1; ++i)
    if (!ctx->ev_recorded[i]) return PROXYKV_ESTATE;
  PKV_HIP(ctx, hipEventSynchronize(ctx->ev[PROXYKV_N_STAGES]));
  for (int i = 0; i < PROXYKV_N_STAGES; ++i) PKV_HIP(ctx, hipEventElapsedTime(&ms_host[i], ctx->ev[i], ctx->ev[i + 1]));
  return PROXYKV_OK;
}

const char* proxykv_strerror(int status) {
  switch (status) {
    case PROXYKV_OK: return "ok";
    case PROXYKV_EINVAL: return "invalid argument";
    case PROXYKV_EUNSUPPORTED: return "shape or option not supported by this build";
    case PROXYKV_ENOMEM: return "out of device memory";
    case PROXYKV_ESTATE: return "context not ready (mapper weights not set)";
    case PROXYKV_EHIP: return "HIP runtime error";
    case PROXYKV_ELIMIT: return "size beyond a fixed limit of this entry point";
    default: return "unknown status";
  }
}

int proxykv_last_hip_error(const proxykv_ctx* ctx) { return ctx ? ctx->last_hip_error : 0; }

}  // extern "C"
