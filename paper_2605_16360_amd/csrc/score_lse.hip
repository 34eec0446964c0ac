// Launches of scoring pass 1 (score_lse.hpp) on bf16 inputs, and the rules that they follow.
#include "score_lse.hpp"

namespace pkv {

// Columns of an MFMA tile.  16 x 16 x 32 instructions draw less than 32 x 32 x 16, but there are twice as many to issue: at d = 128, where
// the products take as long as the exponentials, they gain once there is enough work for the chip's power to set its clock (28 x 12 heads,
// 10 007 keys, both passes 18 170 -> 17 000 us), but not in short launches, up to query blocks times keys of 2^20 or with shared
// blocks.  Both passes, 32 / 16 columns, us: 214 keys 37.6 / 39.8, 257 53.4 / 55.7, 300 55.1 / 57.0, 420 74.0 / 75.8, 600 128.3 / 130.3,
// 300 queries of 1500 keys 129.2 / 131.0; beyond the line 900 240.7 / 242.5, 1024 268.8 / 263.7, 300 queries of 4000 296.2 / 296.6, 500
// 368.7 / 361.8.  Causal, with the longest blocks first, they gain from 400 tokens on (56.3 / 55.5, 700 97.2 / 91.6; 300 44.1 / 46.7, in
// the order of the blocks 51.2).  At d = 64, where the vector ALU sets the time, they do not (16 x 32 heads, 8192 keys 9030 and
// 9050; causal, 4097 tokens, pass 1 alone 885 and 920).
constexpr int64_t kLseWideWork = 1 << 20;

// Workgroups per query block: as many as fill the chip (three per CU at d = 64), if the query blocks alone give it less than half
// of that, with at least one tile each; beyond eight the shares of a query cost pass 2 more than they save.  One layer of 4
// heads, 128 queries of 512 keys, both passes 22.7 -> 15.5 us; 2000 queries of 2000 keys 105 -> 31 us; 16 000 of 16 000 644 -> 583.
// At d = 128 two workgroups per CU are resident; 256 to 383 blocks are shared all the same, since one whole block per place leaves
// half of the CUs with one and half with two (336 blocks, both passes, whole / shared: 1000 keys 81 / 88 us, 4096 226 / 221,
// 8192 426 / 409, 16 000 770 / 730).
int score_splits(int L_s, int H_q, int d, int64_t N, int64_t N_q) {
  const int64_t blocks = (N_q + 128 * kLseCols - 1) / (128 * kLseCols) * H_q * L_s;
  const int64_t tiles = (N + 8192 / d - 1) / (8192 / d) + 1;
  if (blocks >= 384) return 1;
  int64_t s = 768 / blocks;
  s = s < tiles ? s : tiles;
  return (int)(s < kMaxLseSplits ? s : kMaxLseSplits);
}

// fp32 inputs that pass 1 rounds by itself instead of a launch in front, which costs 3 us and reads and writes them once.  The keys, up to
// kRoundKeys of them, are then staged in twice the bytes, and what that costs is decided by how many XCDs read them: the workgroups of a
// KV head that read one share of its keys (its heads' query blocks) lie on one XCD where there are eight shares, and past their L2 every
// further XCD reads the share again.  Both passes, with a launch / so, us, or so's part of the time.  One XCD: one layer of 4 heads, 4000
// tokens 38.2 / 36.6 (8000 85.5 / 88.8); 2 x 32/8 heads, 256 queries of 4096 keys 0.93, 16 x 16/16, 64 of 4096 0.89.  Two for eight
// workgroups: 12 x 16/2, 64 of 4096 0.91.  Four for seven: 24 x 14/2, 256 of 1600 0.95, 64 of 4096 0.94; eight for 21: 6 x 14/2, 700 of 4096
// 1.04.  Four for six: 28 x 12/2, 64 of 1600 1.04, of 4096 1.17.  One for each, 64 of 4096: 20 x 8/4 1.14, 14 x 14/2 1.19, 9 x 32/8 1.31.
// Few keys are rounded either way, as long as queries times keys are few too: one layer of 4 heads, 128 of 512 16.1 / 14.7; 4 x 32/8, 256 of
// 512 0.91; 8 x 32/8, 256 of 256 0.99, of 512 1.01, 64 of 1000 0.97, of 2000 1.10; of more blocks than CUs fewer: 9 x 32/8, 64 of 400 0.93, of 800
// 1.11, 24 of 513 1.04; 256 of 100 0.91, of 200 1.04.
constexpr int64_t kRoundKeys = 4096, kRoundKeysLeast = 128, kRoundWork = 1 << 24;
bool score_rounds_itself(int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q) {
  const int splits = score_splits(L_s, H_q, d, N, N_q);
  if (d != 64 || N > kRoundKeys || splits < 2) return false;
  const int blocks = (int)((N_q + 128 * kLseCols - 1) / (128 * kLseCols)), readers = H_q / H_kv * blocks;
  unsigned xcds = 0;
  for (int r = 0; r < readers; ++r) xcds |= 1u << (unsigned)(r * splits % kScoreXcds);
  const int copies = __builtin_popcount(xcds);
  if (copies == 1 || 4 * readers >= 7 * copies) return true;
  const int64_t few = (int64_t)L_s * H_q * blocks <= 256 ? 1024 : 512;
  return N <= kRoundKeysLeast || (N <= few && (int64_t)L_s * H_q * N_q * N <= kRoundWork);
}

// The most that any input of up to N_q queries takes: one float per query, or pairs of up to 768 workgroups (score_splits).
size_t score_lse_bytes(int L_s, int H_q, int64_t N_q) {
  const size_t rows = (size_t)L_s * H_q * (size_t)N_q, most = (size_t)768 * 128 * kLseCols;
  const size_t pairs = rows * kMaxLseSplits < most ? rows * kMaxLseSplits : most;
  return rows * 4 > pairs * sizeof(LsePart) ? rows * 4 : pairs * sizeof(LsePart);
}

// At d = 64 a workgroup of its own per block runs piped, except in the causal form up to 2048 tokens, where blocks have few whole tiles.  Both
// passes, the other way / piped, us: 16 x 32 heads of 300 queries and keys 46.4 / 45.2, 2000 757 / 739, 8192 8728 / 8606, 16 000 32 680 / 31 810;
// 24 x 14 heads of 10 000 8950 / 8590; causal, 1000 tokens 140 / 145, 2000 432 / 431, 4097 1547 / 1525.  (What is left is power: on zeros,
// which draw little, 8192 7072 / 6503.  Three and four column tiles per wave with two workgroups per CU 8886 and 8529 at 8192, but 2454 and 2385
// at 4000, where two take 2330.)
constexpr int64_t kPipeCausal = 2048;

hipError_t launch_score_lse(const uint16_t* q, const uint16_t* k_ctx, const uint16_t* k_rec, float* neg_lse, int splits,
                            float* x, int64_t n_x, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, int chunk,
                            hipStream_t stream) {
  const int G = H_q / H_kv;
  const float c = 1.4426950408889634f / sqrtf((float)d), inv_c = 1.0f / c;
  // two column sub-tiles per wave; three workgroups per CU at d = 64 (at most 168 registers), two at d = 128
  constexpr int NCOL = kLseCols;
  if (d == 64 && splits == 1 && (N > 0 || N_q > kPipeCausal))
    return launch_score_lse_piped(q, k_ctx, k_rec, neg_lse, x, n_x, L_s, H_q, H_kv, N, N_q, chunk, stream);
  const dim3 grid = lse_grid(L_s, H_q, N_q, splits);
#define PKV_LSE(D, W, MINB, SPLIT)                                                                                         \
  score_lse_kernel<D, NCOL, W, MINB, SPLIT><<<grid, 256, 0, stream>>>(q, k_ctx, k_rec, neg_lse, H_q, G, (int)N, (int)N_q, chunk, \
                                                                   c, inv_c, splits, x, n_x, nullptr, nullptr)
  if (d == 64) {
    if (splits > 1) PKV_LSE(64, 32, 3, true);
    else PKV_LSE(64, 32, 3, false);
  } else {
    const bool wide = N > 0 && (int64_t)grid.x * H_q * L_s * N <= kLseWideWork;
    if (splits > 1 || wide) PKV_LSE(128, 32, 2, true);
    else PKV_LSE(128, 16, 2, false);
  }
#undef PKV_LSE
  return hipGetLastError();
}

}  // namespace pkv
