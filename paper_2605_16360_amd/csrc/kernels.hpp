// Launchers of the HIP kernels; each enqueues on `stream` and returns the launch's hipError_t.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pkv {

// fp32 -> bf16 (round to nearest even) of three arrays (n[i] elements, a multiple of eight; 0 = none).
hipError_t launch_f32_to_bf16(const float* const in[3], uint16_t* const out[3], const int64_t n[3], hipStream_t stream);

// Scoring, pass 1: neg_lse[l, h, i] = -log2(sum_k 2^(c * <q_i, k>)) / c with c = log2(e) / sqrt(d),
// the sum running over the N context keys and the visible reconstruction keys of query i.
// With splits = score_splits(...) > 1 several workgroups share a query's keys: neg_lse then takes 8 * splits bytes per query
// instead of four.  x [n_x] is cleared for pass 2 (n_x = 0: left alone).
size_t score_lse_bytes(int L_s, int H_q, int64_t N_q);  // of neg_lse, for all inputs of up to N_q queries
int score_splits(int L_s, int H_q, int d, int64_t N, int64_t N_q);
hipError_t launch_score_lse(const uint16_t* q, const uint16_t* k_ctx, const uint16_t* k_rec, float* neg_lse, int splits,
                            float* x, int64_t n_x, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, int chunk,
                            hipStream_t stream);
// The same at d = 64 without shared blocks, in another order of instructions (same bits); launch_score_lse picks.
hipError_t launch_score_lse_piped(const uint16_t* q, const uint16_t* k_ctx, const uint16_t* k_rec, float* neg_lse, float* x, int64_t n_x, int L_s,
                                  int H_q, int H_kv, int64_t N, int64_t N_q, int chunk, hipStream_t stream);
// The same with fp32 inputs, which the kernel rounds by itself; q16 [L_s, H_q, N_q, d] and k16 (k_ctx, or with N = 0 k_rec) take the
// rounded copies for pass 2.  Only where score_rounds_itself.
bool score_rounds_itself(int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q);
hipError_t launch_score_lse_fp32(const float* q, const float* k_ctx, const float* k_rec, float* neg_lse, int splits, float* x, int64_t n_x,
                                 uint16_t* q16, uint16_t* k16, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, int chunk,
                                 hipStream_t stream);
// Scoring, pass 2: x[l, g, n] = 2^(c * max over (head of group g, query i) of (<q_i, k_n> + neg_lse[l, h, i])).
// neg_lse and splits as pass 1 left them.  q_splits = score_query_splits(...) workgroups share a key block's queries; with
// splits > 1 or q_splits > 1 they raise x, which pass 1 has to clear.
size_t score_parts_bytes(int L_s, int H_kv, int d, int64_t N);  // of `parts` below, for all inputs of up to N keys
int score_query_splits(bool sum, bool causal, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q);
hipError_t launch_score_colmax(const uint16_t* q, const uint16_t* k_ctx, const float* neg_lse, int splits, float* x,
                               int q_splits, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q,
                               hipStream_t stream);

// Scoring, pass 2 in the sum form: x[l, g, n] = sum over (head of group g, query i) of 2^(c * (<q_i, k_n> + neg_lse[l, h, i])).
// causal: the keys are the queries' own sequence (N == N_q) and query i adds to keys n <= i only.
// With q_splits > 1 `parts` takes q_splits * L_s * H_kv * N floats on the way.
hipError_t launch_score_colsum(const uint16_t* q, const uint16_t* k_ctx, const float* neg_lse, int splits, float* x,
                               float* parts, int q_splits, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, bool causal,
                               hipStream_t stream);
// Per-row Top-K.  Rows longer than 36 864 scores are split over several workgroups and need `scratch` (device memory, any
// contents, 256-byte aligned; rows <= 65535 then) of topk_scratch_bytes(rows, N) bytes, which serve all calls of no more and no
// longer rows, or, where the scores are read once more each, of topk_scratch_bytes_no_masks(rows, N) or topk_scratch_bytes_least(rows, N).
constexpr int64_t kTopkSingleMax = 36864;  // longest row one workgroup selects from
size_t topk_scratch_bytes(int64_t rows, int64_t N);
size_t topk_scratch_bytes_no_masks(int64_t rows, int64_t N);
size_t topk_scratch_bytes_least(int64_t rows, int64_t N);
// `patience`: how long, in ticks of 10 ns, a workgroup waits for the others of its row before it selects by itself (topk.hip).
constexpr unsigned long long kTopkPatience = 20000;
hipError_t launch_topk(const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out, void* scratch,
                       size_t scratch_bytes, hipStream_t stream, unsigned long long patience = kTopkPatience);
// The same selection with every workgroup gathering the token rows it kept: k_out[r, j, :] = k_in[r, idx[r, j], :] and
// likewise v (row_bytes per token, 1024 / (row_bytes / 16) a whole number).
hipError_t launch_topk_gather(const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out, void* scratch,
                              size_t scratch_bytes, const void* k_in, const void* v_in, int64_t row_bytes, void* k_out,
                              void* v_out, hipStream_t stream);

hipError_t launch_compact(const void* k_in, const void* v_in, const int32_t* idx, int64_t rows, int64_t N,
                          int64_t K, int64_t row_bytes, void* k_out, void* v_out, hipStream_t stream);

// In-place variant: tokens 0 .. K-1 of every row of k and v become the kept tokens in order.  With `scratch` (device memory, any
// contents) of compact_inplace_scratch_bytes several workgroups share a row; that is 0 where one per row is better or has to do.  A launch on
// another stream must not use the same scratch memory before this one is over: parts of a row wait for each other in it without a bound.
size_t compact_inplace_scratch_bytes(int64_t rows, int64_t K, int64_t row_bytes, int heads);
// no less than that for any number of kept tokens up to K
size_t compact_inplace_scratch_most(int64_t rows, int64_t K, int64_t row_bytes, int heads);
hipError_t launch_compact_inplace(void* k, void* v, const int32_t* idx, int64_t rows, int64_t N, int64_t K, int64_t row_bytes,
                                  const int32_t* counts, int heads, void* scratch, size_t scratch_bytes, hipStream_t stream);
// counts [layers, heads] from a layer's ascending flat indices h * N + n (heads * K per layer)
hipError_t launch_head_counts(const int32_t* flat, int64_t layers, int64_t heads, int64_t N, int64_t K, int32_t* counts,
                              hipStream_t stream);
// mask[r, n] = 1 if n is one of idx[r, :], else 0.
hipError_t launch_mask(const int32_t* idx, int64_t rows, int64_t N, int64_t K, uint8_t* mask, hipStream_t stream);
}  // namespace pkv
