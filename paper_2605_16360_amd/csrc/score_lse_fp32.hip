// Scoring pass 1 (score_lse.hpp) on fp32 inputs that it rounds by itself.
#include "score_lse.hpp"

namespace pkv {

hipError_t launch_score_lse_fp32(const float* q, const float* k_ctx, const float* k_rec, float* neg_lse, int splits, float* x, int64_t n_x,
                                 uint16_t* q16, uint16_t* k16, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, int chunk,
                                 hipStream_t stream) {
  if (d != 64 || splits < 2) return hipErrorInvalidValue;
  const float c = 1.4426950408889634f / sqrtf((float)d), inv_c = 1.0f / c;
  score_lse_kernel<64, kLseCols, 32, 2, true, float><<<lse_grid(L_s, H_q, N_q, splits), 256, 0, stream>>>(
      q, k_ctx, k_rec, neg_lse, H_q, H_q / H_kv, (int)N, (int)N_q, chunk, c, inv_c, splits, x, n_x, q16, k16);
  return hipGetLastError();
}

}  // namespace pkv
