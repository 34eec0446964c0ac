// Scoring pass 1 (score_lse.hpp) at d = 64 with one unit's exponentials between the next one's products.
#include "score_lse.hpp"

namespace pkv {

hipError_t launch_score_lse_piped(const uint16_t* q, const uint16_t* k_ctx, const uint16_t* k_rec, float* neg_lse, float* x, int64_t n_x, int L_s,
                                  int H_q, int H_kv, int64_t N, int64_t N_q, int chunk, hipStream_t stream) {
  const float c = 1.4426950408889634f / sqrtf(64.0f), inv_c = 1.0f / c;
  score_lse_kernel<64, kLseCols, 32, 3, false, uint16_t, true><<<lse_grid(L_s, H_q, N_q, 1), 256, 0, stream>>>(
      q, k_ctx, k_rec, neg_lse, H_q, H_q / H_kv, (int)N, (int)N_q, chunk, c, inv_c, 1, x, n_x, nullptr, nullptr);
  return hipGetLastError();
}

}  // namespace pkv
