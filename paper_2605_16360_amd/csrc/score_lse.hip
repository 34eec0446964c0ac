// Proxy importance scoring, pass 1 (paper Sec. 3: softmax of Q K^T / sqrt(d) per query row): the
// row log-sum-exp of every reconstruction query over the N context keys plus the reconstruction
// keys of its own chunk up to and including itself.
//
// The logit matrix is never stored: K Q^T tiles are computed with v_mfma_f32_32x32x16_bf16.  The
// queries of a workgroup (the "columns", 32*NCOL per wave) stay in registers as the MFMA B operand
// for the whole kernel; the keys (the "rows") stream through 16 KB LDS tiles.  With rows on the
// MFMA M axis a lane owns ONE query column and 16 key rows of every tile, so the sum over keys runs
// inside a lane and needs one cross-lane step (lane ^ 32) at the end.
//
// With c = log2(e) / sqrt(d) the kernel accumulates lsum = sum 2^(c*s - m_ref) per lane and column.
// The vector ALU, not the matrix pipe, bounds this pass (one v_exp_f32 costs two ALU slots), so the
// work per element is cut to the three instructions that cannot be avoided (fma, exp2, add): no
// running maximum is tracked.  The reference m_ref is an attained logit of the column; it is only
// replaced when the sum of one 16-element chain leaves [0, 2^64), which the first chain of every
// column does by construction (m_ref starts at -1e30) and later chains practically never do.  A term
// can exceed the reference by up to 2^64 and every term far below it is negligible against the
// attained one, so neither overflow nor underflow loses anything.  The kernel writes -L2 / c per
// row, L2 = m_ref + log2(lsum), which pass 2 uses as the accumulator's initial value.
//
// Tiles that causality, a chunk boundary or the end of the context cuts are masked and summed the same way; the checked
// path, whose chains wait for each other (three times as long per tile), is left for columns without a reference and for
// sums out of range.  The first reference comes from the first 32 keys.  16 layers of 4097 tokens, causal: 1343 -> 995 us.
//
// Streaming: three LDS buffers and one barrier per tile.  While tile t is computed, tile t+2 goes
// from registers to LDS and tile t+3 is fetched from global memory into registers.
//
// Few queries (one layer, a short sequence) leave most of the chip without a workgroup.  The key tiles of a query block are
// then shared by several workgroups, each of which leaves its reference and sum of every query; pass 2 puts them together
// where it reads a query's log-sum-exp.
#include "kernels.hpp"
#include "score_common.hpp"

namespace pkv {
namespace {

// A chain's sum outside [0, kRebase) makes its lanes take a new reference.
constexpr float kRebase = 1.8446744e19f;  // 2^64
// Interior tiles are summed without any check; a column's running sum outside [0, kTileRedo) afterwards
// undoes the tile and sums it again chain by chain with the check.
constexpr float kTileRedo = 1.2676506e30f;  // 2^100

// SPLIT: `splits` workgroups per query block, neg_lse holds (reference, sum) pairs [splits][L_s * H_q * N_q].
// x [n_x] (n_x may be 0) is cleared for a pass 2 whose workgroups raise it.
template <int D, int NCOL, int MINB, bool SPLIT>
__global__ __launch_bounds__(256, MINB) void score_lse_kernel(const uint16_t* __restrict__ q,
                                                               const uint16_t* __restrict__ k_ctx,
                                                               const uint16_t* __restrict__ k_rec,
                                                               float* __restrict__ neg_lse, int H_q, int G, int N,
                                                               int N_q, int chunk, float c, float inv_c, int splits,
                                                               float* __restrict__ x, int64_t n_x) {
  using C = ScoreCfg<D>;
  __shared__ u32x4 lds[kNBuf * C::TILE_U4];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int h = blockIdx.y, l = blockIdx.z, H_kv = H_q / G, hs = h / G;
  constexpr int QB = 128 * NCOL;
  const int split = SPLIT ? blockIdx.x % splits : 0;
  const int i0 = (SPLIT ? blockIdx.x / splits : blockIdx.x) * QB;
  if (n_x > 0) {
    const int64_t wg = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const int64_t stride = (int64_t)gridDim.x * gridDim.y * gridDim.z * 256;
    for (int64_t i = wg * 256 + tid; i < n_x; i += stride) x[i] = 0.0f;
  }
  const uint16_t* qh = q + (size_t)(l * H_q + h) * N_q * D;
  const uint16_t* kc = k_ctx + (size_t)(l * H_kv + hs) * N * D;
  const uint16_t* kr = k_rec + (size_t)(l * H_kv + hs) * N_q * D;

  // resident B operand: the wave's queries
  bf16x8 b[NCOL][C::KK];
  int qi[NCOL], qlo[NCOL];
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) {
    qi[cs] = i0 + (wave * NCOL + cs) * 32 + l32;
    const int row = qi[cs] < N_q ? qi[cs] : N_q - 1;
    qlo[cs] = (row / chunk) * chunk;  // (a column past the last query sees that query's chunk, so that it has a reference too)
#pragma unroll
    for (int kk = 0; kk < C::KK; ++kk)
      b[cs][kk] = as_bf16x8(*reinterpret_cast<const u32x4*>(qh + (size_t)row * D + kk * 16 + half * 8));
  }
  float nref[NCOL], lsum[NCOL];  // nref = -m_ref
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) {
    nref[cs] = 1.0e30f;
    lsum[cs] = 0.0f;
  }

  // tile list: the context tiles, then the reconstruction tiles from the start of the block's chunk to
  // its last query
  const int n_ctx = (N + C::ROWS - 1) / C::ROWS;
  const int i_end = (i0 + QB < N_q ? i0 + QB : N_q);  // one past the block's last query
  const int rec_lo = (i0 / chunk) * chunk;            // first reconstruction key any query of the block sees
  const int n_rec = (i_end - rec_lo + C::ROWS - 1) / C::ROWS;
  const int total_all = n_ctx + n_rec, n_whole = N / C::ROWS;  // n_whole: context tiles that the end does not cut
  // this workgroup's tiles: t0, ..., t0 + total - 1 of the list
  const int t0 = SPLIT ? (int)((int64_t)total_all * split / splits) : 0;
  const int total = SPLIT ? (int)((int64_t)total_all * (split + 1) / splits) - t0 : total_all;
  const int wave_i_lo = i0 + wave * NCOL * 32;  // first query of this wave
  TileRegs<D> regs;
  auto fetch_to = [&](TileRegs<D>& r, int t) {
    t += t0;
    if (t < n_ctx) tile_fetch<D>(r, kc, t * C::ROWS, N, tid);
    else tile_fetch<D>(r, kr, rec_lo + (t - n_ctx) * C::ROWS, i_end, tid);
  };
  auto fetch = [&](int t) { fetch_to(regs, t); };

  // sum of one chain: 16 x (fma, exp2, add); re-based when it leaves [0, 2^64)
  auto accumulate = [&](const f32x16& acc, int cs) {
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
      s0 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 0], c, nref[cs]));
      s1 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 1], c, nref[cs]));
      s2 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 2], c, nref[cs]));
      s3 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 3], c, nref[cs]));
    }
    float sum = (s0 + s1) + (s2 + s3);
    const bool bad = !(sum < kRebase);  // too large, infinite or NaN
    if (__builtin_amdgcn_ballot_w64(bad)) {
      if (bad) {
        const float tm = max16_tree(acc, kNegInf) * c;
        // all 16 rows masked: keep the reference (their terms are zero under any finite reference)
        const float nm = tm > -1.0e30f ? tm : -nref[cs];
        lsum[cs] *= __builtin_amdgcn_exp2f(-nref[cs] - nm);
        nref[cs] = -nm;
        sum = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r], c, nref[cs]));
      }
    }
    lsum[cs] += sum;
  };

  // sum of one chain, no check: 16 x (fma, exp2, add)
  auto fast_sum = [&](const f32x16& acc, int cs) {
    float s0 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[0], c, nref[cs]));
    float s1 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[1], c, nref[cs]));
    float s2 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[2], c, nref[cs]));
    float s3 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[3], c, nref[cs]));
#pragma unroll
    for (int r = 4; r < 16; r += 4) {
      s0 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 0], c, nref[cs]));
      s1 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 1], c, nref[cs]));
      s2 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 2], c, nref[cs]));
      s3 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 3], c, nref[cs]));
    }
    return (s0 + s1) + (s2 + s3);
  };
  // the keys of an interior tile, visible to every query of the block, summed without checks
  auto interior_tile = [&](const u32x4* buf) {
#pragma unroll
    for (int s = 0; s < C::SUB; ++s) {
      bf16x8 a[C::KK];
#pragma unroll
      for (int kk = 0; kk < C::KK; ++kk) a[kk] = frag_read<D>(buf, s * 32 + l32, kk * 2 + half);
      f32x16 acc[NCOL];
#pragma unroll
      for (int cs = 0; cs < NCOL; ++cs) {
        acc[cs] = splat16(0.0f);
#pragma unroll
        for (int kk = 0; kk < C::KK; ++kk) acc[cs] = mfma_32x32x16(a[kk], b[cs][kk], acc[cs]);
      }
#pragma unroll
      for (int cs = 0; cs < NCOL; ++cs) lsum[cs] += fast_sum(acc[cs], cs);
    }
  };

  // Where a chain of the tile at row0 (32 keys from jbase on, the wave's column sub-tile cs) stands: nothing of it is visible,
  // some of it, or all.  All of it is where every key lies at or before the first query, and inside its last one's chunk.
  auto hidden = [&](bool is_rec, int jbase, int limit, int cs) {
    return jbase >= limit || (is_rec && jbase > wave_i_lo + cs * 32 + 31);
  };
  auto cut = [&](bool is_rec, int jbase, int limit, int cs) {
    const int cs_i_lo = wave_i_lo + cs * 32;
    return is_rec ? !(jbase + 31 <= cs_i_lo && jbase >= ((cs_i_lo + 31) / chunk) * chunk) : jbase + 32 > limit;
  };
  // a column sees the context keys below N, the reconstruction keys from its chunk's first to its own: one range either way, so
  // that the mask is three instructions per element (as a choice per element it compiled to two branches for each, fetched for a
  // few tiles: 28 layers of 12 heads of 128, 200 queries of 2000 keys, both passes: 123 -> 109 us)
  auto mask_chain = [&](f32x16& acc, bool is_rec, int jbase, int cs) {
    const int first = is_rec ? qlo[cs] : 0, last = is_rec ? qi[cs] : N - 1;
    const int from = first - (jbase + half * 4);
    const uint32_t span = (uint32_t)(last - first);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = (uint32_t)((r >> 2) * 8 + (r & 3) - from) <= span ? acc[r] : kNegInf;
  };
  // a tile that causality, a chunk boundary or the end of the context cuts: its visible chains, summed without checks
  auto cut_tile = [&](const u32x4* buf, bool is_rec, int row0, int limit) {
#pragma unroll 1
    for (int s = 0; s < C::SUB; ++s) {
      const int jbase = row0 + s * 32;
      if (hidden(is_rec, jbase, limit, NCOL - 1)) break;
      bf16x8 a[C::KK];
#pragma unroll
      for (int kk = 0; kk < C::KK; ++kk) a[kk] = frag_read<D>(buf, s * 32 + l32, kk * 2 + half);
#pragma unroll
      for (int cs = 0; cs < NCOL; ++cs) {
        if (hidden(is_rec, jbase, limit, cs)) continue;
        f32x16 acc = splat16(0.0f);
#pragma unroll
        for (int kk = 0; kk < C::KK; ++kk) acc = mfma_32x32x16(a[kk], b[cs][kk], acc);
        if (cut(is_rec, jbase, limit, cs)) mask_chain(acc, is_rec, jbase, cs);
        lsum[cs] += fast_sum(acc, cs);
      }
    }
  };
  // the first reference of every column: the largest visible logit of the first 32 keys of a tile (if any is visible)
  auto first_reference = [&](const u32x4* buf, bool interior, bool is_rec, int row0) {
    bf16x8 a[C::KK];
#pragma unroll
    for (int kk = 0; kk < C::KK; ++kk) a[kk] = frag_read<D>(buf, l32, kk * 2 + half);
#pragma unroll
    for (int cs = 0; cs < NCOL; ++cs) {
      f32x16 acc = splat16(0.0f);
#pragma unroll
      for (int kk = 0; kk < C::KK; ++kk) acc = mfma_32x32x16(a[kk], b[cs][kk], acc);
      if (!interior) mask_chain(acc, is_rec, row0, cs);
      const float tm = max16_tree(acc, kNegInf) * c;
      if (tm > -1.0e30f) nref[cs] = -tm;
    }
  };

  // sums a tile without checks; false, and the sums as they were, if one of them went out of range
  auto sum_unchecked = [&](auto&& sum_tile) {
    float before[NCOL];
#pragma unroll
    for (int cs = 0; cs < NCOL; ++cs) before[cs] = lsum[cs];
    sum_tile();
    bool bad = false;
#pragma unroll
    for (int cs = 0; cs < NCOL; ++cs) bad |= !(lsum[cs] < kTileRedo);
    if (__builtin_amdgcn_ballot_w64(bad) == 0) return true;
#pragma unroll
    for (int cs = 0; cs < NCOL; ++cs) lsum[cs] = before[cs];
    return false;
  };

  if (total > 0) {
    TileRegs<D> second;  // the first two tiles are asked for together
    fetch(0);
    if (total > 1) fetch_to(second, 1);
    tile_store<D>(regs, lds, tid);
    if (total > 1) tile_store<D>(second, lds + C::TILE_U4, tid);
  }
  // Every load so far (the wave's queries among them) has landed before the loop: a share without tiles skips the stores that
  // wait for them, so without this the compiler cannot tell that they arrived long ago, and waits in front of the MFMAs of
  // every tile for the prefetch just issued (16 layers of 32 heads, 64 queries of 9000 keys, both passes: 262 -> 253 us).
  __builtin_amdgcn_s_waitcnt(kVmcnt0);
  if (total > 2) fetch(2);

  for (int t = 0; t < total; ++t) {
    // every wave has finished tile t-1: its buffer takes tile t+2, the registers take tile t+3
    __syncthreads();
    if (t + 2 < total) tile_store<D>(regs, lds + ((t + 2) % kNBuf) * C::TILE_U4, tid);
    if (t + 3 < total) fetch(t + 3);
    const u32x4* buf = lds + (t % kNBuf) * C::TILE_U4;
    const int tg = t0 + t;
    // Whole context tiles, nearly all there are, go round a loop of their own: with the choices below in it a tile of heads of
    // 128 took 1 to 3 % longer (28 layers of 12 heads, 300 queries of 16 000 keys, both passes: 1123 -> 1108 us).
    const bool whole = t > 0 && tg < n_whole;
    if (whole && sum_unchecked([&]() { interior_tile(buf); })) continue;
    const bool is_rec = tg >= n_ctx;
    const int row0 = is_rec ? rec_lo + (tg - n_ctx) * C::ROWS : tg * C::ROWS;
    // Summed without checks, and again chain by chain with them if a sum went out of range (as it does where a column has
    // no reference yet).  A reconstruction tile is interior too when all its keys lie at or before the block's first query
    // and inside the chunk of its last one (then inside every query's chunk).
    const int limit = is_rec ? i_end : N;
    const bool interior = is_rec ? row0 + C::ROWS - 1 <= i0 && row0 >= ((i_end - 1) / chunk) * chunk : row0 + C::ROWS <= N;
    // Where there are few tiles, cut ones take the checks at once, and so does the first of a share: the way to a first
    // reference and the code of a second loop, fetched for a tile or two, cost more than they save (16 layers, causal:
    // 200 tokens 30 -> 22 us, 450 tokens 62 -> 51 us, 1000 tokens, eight tiles and more, the same either way).
    bool redo = whole || (total < 8 && !interior) || (SPLIT && t == 0 && total < 4);
    if (!redo) {
      if (t == 0) first_reference(buf, interior, is_rec, row0);
      redo = !sum_unchecked([&]() {
        if (interior) interior_tile(buf);
        else cut_tile(buf, is_rec, row0, limit);
      });
    }
    if (redo) {
#pragma unroll 1
      for (int s = 0; s < C::SUB; ++s) {
        const int jbase = row0 + s * 32;
        if (hidden(is_rec, jbase, limit, NCOL - 1)) break;
        bf16x8 a[C::KK];
#pragma unroll
        for (int kk = 0; kk < C::KK; ++kk) a[kk] = frag_read<D>(buf, s * 32 + l32, kk * 2 + half);
#pragma unroll
        for (int cs = 0; cs < NCOL; ++cs) {
          if (hidden(is_rec, jbase, limit, cs)) continue;
          f32x16 acc = splat16(0.0f);
#pragma unroll
          for (int kk = 0; kk < C::KK; ++kk) acc = mfma_32x32x16(a[kk], b[cs][kk], acc);
          if (cut(is_rec, jbase, limit, cs)) mask_chain(acc, is_rec, jbase, cs);
          accumulate(acc, cs);
        }
      }
    }
  }
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) {
    const float m1 = -nref[cs];
    const float m2 = swap_halves(m1), l2 = swap_halves(lsum[cs]);
    const float m = __builtin_fmaxf(m1, m2);
    const float tot = lsum[cs] * __builtin_amdgcn_exp2f(m1 - m) + l2 * __builtin_amdgcn_exp2f(m2 - m);
    if constexpr (SPLIT) {
      if (half == 0 && qi[cs] < N_q)
        reinterpret_cast<LsePart*>(neg_lse)[((size_t)split * gridDim.z * H_q + l * H_q + h) * N_q + qi[cs]] = LsePart{m, tot};
    } else {
      const float L2 = m + __builtin_amdgcn_logf(tot);
      if (half == 0 && qi[cs] < N_q) neg_lse[(size_t)(l * H_q + h) * N_q + qi[cs]] = -L2 * inv_c;
    }
  }
}

}  // namespace

constexpr int kLseCols = 2;  // column sub-tiles per wave; 128 * kLseCols queries per workgroup

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

// The most that any input of up to N_q queries takes: one float per query, or pairs of up to 768 workgroups (score_splits).
size_t score_lse_bytes(int L_s, int H_q, int64_t N_q) {
  const size_t rows = (size_t)L_s * H_q * (size_t)N_q, most = (size_t)768 * 128 * kLseCols;
  const size_t pairs = rows * kMaxLseSplits < most ? rows * kMaxLseSplits : most;
  return rows * 4 > pairs * sizeof(LsePart) ? rows * 4 : pairs * sizeof(LsePart);
}

hipError_t launch_score_lse(const uint16_t* q, const uint16_t* k_ctx, const uint16_t* k_rec, float* neg_lse, int splits,
                            float* x, int64_t n_x, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, int chunk,
                            hipStream_t stream) {
  const int G = H_q / H_kv;
  const float c = 1.4426950408889634f / sqrtf((float)d), inv_c = 1.0f / c;
  // two column sub-tiles per wave; three workgroups per CU at d = 64 (at most 168 registers), two at d = 128
  constexpr int NCOL = kLseCols;
  // the query blocks of a head are dealt over all XCDs (measured: fewer L2 misses than one KV group per XCD, whose
  // blocks drift apart along a key stream slightly larger than the L2)
  dim3 grid((unsigned)((N_q + 128 * NCOL - 1) / (128 * NCOL) * splits), (unsigned)H_q, (unsigned)L_s);
#define PKV_LSE(D, MINB, SPLIT)                                                                                          \
  score_lse_kernel<D, NCOL, MINB, SPLIT><<<grid, 256, 0, stream>>>(q, k_ctx, k_rec, neg_lse, H_q, G, (int)N, (int)N_q, chunk, \
                                                                   c, inv_c, splits, x, n_x)
  if (d == 64) {
    if (splits > 1) PKV_LSE(64, 3, true);
    else PKV_LSE(64, 3, false);
  } else {
    if (splits > 1) PKV_LSE(128, 2, true);
    else PKV_LSE(128, 2, false);
  }
#undef PKV_LSE
  return hipGetLastError();
}

}  // namespace pkv
