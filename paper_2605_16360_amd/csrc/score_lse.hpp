// Proxy importance scoring, pass 1 (paper Sec. 3: softmax of Q K^T / sqrt(d) per query row): the
// row log-sum-exp of every reconstruction query over the N context keys plus the reconstruction
// keys of its own chunk up to and including itself.
//
// The logit matrix is never stored: K Q^T tiles are computed with v_mfma_f32_32x32x16_bf16 or v_mfma_f32_16x16x32_bf16.  The
// queries of a workgroup (the "columns", 32*NCOL per wave) stay in registers as the MFMA B operand
// for the whole kernel; the keys (the "rows") stream through 16 KB LDS tiles.  With rows on the
// MFMA M axis a lane owns a query column and some key rows of every tile, so the sum over keys runs
// inside a lane and needs one or two cross-lane steps at the end.
//
// With c = log2(e) / sqrt(d) the kernel accumulates lsum = sum 2^(c*s - m_ref) per lane and column.
// The vector ALU, not the matrix pipe, bounds this pass (one v_exp_f32 costs two ALU slots), so the
// work per element is cut to the three instructions that cannot be avoided (fma, exp2, add): no
// running maximum is tracked.  The reference m_ref is an attained logit of the column; it is only
// replaced when the sum of one chain of 8 or 16 elements leaves [0, 2^64), which the first chain of every
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
#pragma once
#include "kernels.hpp"
#include "score_common.hpp"

namespace pkv {
namespace {

// A chain's sum outside [0, kRebase) makes its lanes take a new reference.
constexpr float kRebase = 1.8446744e19f;  // 2^64
// Interior tiles are summed without any check; a column's running sum outside [0, kTileRedo) afterwards
// undoes the tile and sums it again chain by chain with the check.
constexpr float kTileRedo = 1.2676506e30f;  // 2^100

// Query block of place x of nb in head g.  Workgroups go round the eight XCDs in launch order, and a block is the longer the further back
// in its chunk it lies: where nb is a multiple of eight, an XCD would meet the same places of a chunk in every head (8192 tokens in chunks
// of 2048: XCD 7 only blocks of 80 tiles, XCD 0 of 66), and all wait for the one with the longest.  So the blocks of a head are
// turned, by as much as moves a block's XCD on by one from head to head.  Both passes: 16 x 32 heads, 2000 queries and keys 783 -> 725 us,
// 8192 9067 -> 8463; 24 x 14 heads, 6001, sum form 4295 -> 4065; 28 x 12 heads of 128, 10 007 17 065 -> 16 270; with four blocks, where a place
// has two XCDs, 16 x 32 heads of 900 196 -> 193.  Other numbers of blocks spread by themselves (six, turned: 24 x 14 heads of 1400 271 ->
// 277), and workgroups that share a block are few and short (one layer of 512 keys 15.9 -> 16.2).
__device__ __forceinline__ int turned_block(int x, int nb, int g) { return (x + (nb + 7) % 8 * (g % 8)) % nb; }

// SPLIT: `splits` workgroups per query block; with more than one neg_lse holds (reference, sum) pairs [splits][L_s * H_q * N_q].
// x [n_x] (n_x may be 0) is cleared for a pass 2 whose workgroups raise it.
// In: what q, k_ctx and k_rec hold.  With fp32 the kernel rounds them itself and leaves bf16 copies of the queries and of the keys that
// pass 2 reads (the context's, or the sequence's own) in q16 and k16.
template <int D, int NCOL, int W, int MINB, bool SPLIT, class In = uint16_t, bool PIPE = false>
__global__ __launch_bounds__(256, MINB) void score_lse_kernel(const In* __restrict__ q,
                                                               const In* __restrict__ k_ctx,
                                                               const In* __restrict__ k_rec,
                                                               float* __restrict__ neg_lse, int H_q, int G, int N,
                                                               int N_q, int chunk, float c, float inv_c, int splits,
                                                               float* __restrict__ x, int64_t n_x, uint16_t* __restrict__ q16,
                                                               uint16_t* __restrict__ k16) {
  using C = ScoreCfg<D>;
  using R = Rows32<D, W>;
  constexpr bool kRound = sizeof(In) == 4;
  using Regs = std::conditional_t<kRound, TileRegsF32<D>, TileRegs<D>>;
  using Acc = typename R::Acc;
  __shared__ u32x4 lds[kNBuf * C::TILE_U4];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, rows4 = lane / W * 4;
  constexpr int QB = 128 * NCOL;
  const int split = SPLIT ? blockIdx.x % splits : 0;
  int h = blockIdx.y, l = blockIdx.z, qb = SPLIT ? blockIdx.x / splits : blockIdx.x;
  if (!SPLIT && N == 0) {
    // causal over the whole sequence: the last query block has the most keys; 64 heads (or as many as fill the chip) at a time
    // (16 x 32 heads of 64, 4097 tokens, both passes: 1625 -> 1590 us; 1000 tokens: 173 -> 156)
    const int nb = gridDim.x, id = ((int)blockIdx.z * gridDim.y + blockIdx.y) * nb + blockIdx.x;
    const SetItem it = longest_first(id, gridDim.y * gridDim.z, nb, nb < 16 ? 1024 / nb : 64);
    qb = nb - 1 - it.item;
    h = it.set % H_q;
    l = it.set / H_q;
  }
  if constexpr (!SPLIT || D == 128) {
    if (N > 0 && gridDim.x % 4 == 0 && (!SPLIT || splits == 1)) qb = turned_block(qb, gridDim.x, l * H_q + h);
  }
  const int H_kv = H_q / G, hs = h / G, i0 = qb * QB;
  // where the part's results start: at the end the grid's size would be waited for (causal, 256 tokens of 28 x 12 heads of 128 34.3 -> 33.6 us)
  const size_t split0 = SPLIT ? (size_t)split * gridDim.z * H_q * N_q : 0;
  if (n_x > 0) {
    const int64_t wg = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const int64_t stride = (int64_t)gridDim.x * gridDim.y * gridDim.z * 256;
    for (int64_t i = wg * 256 + tid; i < n_x; i += stride) x[i] = 0.0f;
  }
  const In* qh = q + (size_t)(l * H_q + h) * N_q * D;
  const In* kc = k_ctx + (size_t)(l * H_kv + hs) * N * D;
  const In* kr = k_rec + (size_t)(l * H_kv + hs) * N_q * D;

  // resident B operand: the wave's queries, NT tiles of W, NS to 32 columns
  constexpr int NT = 32 * NCOL / W, NS = 32 / W;
  bf16x8 b[NT][R::KK];
  int qi[NT], qlo[NT];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    qi[ct] = i0 + (wave * NT + ct) * W + lane % W;
    const int row = qi[ct] < N_q ? qi[ct] : N_q - 1;
    qlo[ct] = (row / chunk) * chunk;  // (a column past the last query sees that query's chunk, so that it has a reference too)
    R::columns(b[ct], qh, row, lane);
    if constexpr (kRound) {
      if (split == 0 && qi[ct] < N_q) R::keep_columns(b[ct], q16 + (size_t)(l * H_q + h) * N_q * D, row, lane);
    }
  }
  float nref[NT], lsum[NT];  // nref = -m_ref
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    nref[ct] = 1.0e30f;
    lsum[ct] = 0.0f;
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
  // the copy of the keys is the group's first head's to make: the first query block's workgroups meet all context tiles, in the causal form
  // (N = 0) the last one's all tiles
  const bool keeps = kRound && h % G == 0 && i0 == (N > 0 ? 0 : (N_q - 1) / QB * QB);
  auto store_rounded = [&](const auto& r, u32x4* dst, int t) {
    const int row0 = (t0 + t) * C::ROWS, rows = N > 0 ? N : N_q;
    uint16_t* copy = keeps && row0 < rows ? k16 + ((size_t)(l * H_kv + hs) * rows + row0) * D : nullptr;
    tile_store<D>(r, dst, tid, copy, rows - row0);
  };
#define PKV_STORE(regs, dst, t)                            \
  do {                                                     \
    if constexpr (kRound) store_rounded(regs, dst, t);     \
    else tile_store<D>(regs, dst, tid);                    \
  } while (0)
  Regs regs;
  auto fetch_to = [&](Regs& r, int t) {
    t += t0;
    if (t < n_ctx) tile_fetch<D>(r, kc, t * C::ROWS, N, tid);
    else tile_fetch<D>(r, kr, rec_lo + (t - n_ctx) * C::ROWS, i_end, tid);
  };
  auto fetch = [&](int t) { fetch_to(regs, t); };

  // sum of one chain (32 keys, of which a lane has R::E, and one column tile), no check: fma, exp2, add per element
  auto fast_sum = [&](const Acc& acc, int ct) {
    float s[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(acc.get(r), c, nref[ct]));
#pragma unroll
    for (int r = 4; r < R::E; ++r) s[r & 3] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc.get(r), c, nref[ct]));
    return (s[0] + s[1]) + (s[2] + s[3]);
  };
  // the same, re-based when it leaves [0, 2^64)
  auto accumulate = [&](const Acc& acc, int ct) {
    float sum = fast_sum(acc, ct);
    const bool bad = !(sum < kRebase);  // too large, infinite or NaN
    if (__builtin_amdgcn_ballot_w64(bad)) {
      if (bad) {
        const float tm = max_of<R>(acc, kNegInf) * c;
        // all rows masked: keep the reference (their terms are zero under any finite reference)
        const float nm = tm > -1.0e30f ? tm : -nref[ct];
        lsum[ct] *= __builtin_amdgcn_exp2f(-nref[ct] - nm);
        nref[ct] = -nm;
        sum = fast_sum(acc, ct);
      }
    }
    lsum[ct] += sum;
  };
  // The keys of an interior tile, visible to every query of the block, summed without checks.  At d = 128, where matrix and vector
  // work take nearly as long, the products of one sub-tile are issued between the exponentials of the one before (28 x 12 heads,
  // 10 007 keys, both passes: 17 190 -> 16 890 us); at d = 64 the compiler's own order is the faster one (8192 keys, 16 x 32 heads:
  // 9030 and 9100 us).
  auto interior_tile = [&](const u32x4* buf) {
    if constexpr (D == 128) {
      Acc acc[2][NT];
      R a[2];
      a[0].read(buf, 0, lane);
      a[0].products(acc[0], b, R::zero());
      a[1].read(buf, 32, lane);
      static_for<C::SUB>([&](auto sc) {
        constexpr int s = decltype(sc)::value, cur = s & 1, nxt = cur ^ 1;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (s + 1 < C::SUB) a[nxt].products(acc[nxt], b, R::zero());
        if constexpr (s + 2 < C::SUB) a[cur].read(buf, (s + 2) * 32, lane);
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) lsum[ct] += fast_sum(acc[cur][ct], ct);
        if constexpr (s + 1 < C::SUB) {
#pragma unroll
          for (int i = 0; i < R::RT * NT * R::KK; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x402, 3, 0);  // three vector instructions, exponentials among them
          }
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    } else {
#pragma unroll
      for (int s = 0; s < C::SUB; ++s) {
        R a;
        a.read(buf, s * 32, lane);
        Acc acc[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) acc[ct] = a.product(b[ct], R::zero());
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) lsum[ct] += fast_sum(acc[ct], ct);
      }
    }
  };

  // PIPE (32-column tiles): the same, a unit of one column tile and 32 keys at a time: its 16 fma, its 16 exponentials with the next unit's
  // products between them, its 16 adds.  Two waves of a SIMD issue full-rate vector instructions (fma, add) in the same cycles, exponentials and
  // products hold it alone, so the waves are kept in step: exponentials go first, and a wave that has done its own finds the other one
  // at its fma and adds too.  (Out of registers with the products, three waves per SIMD, ns per logit of a lane: 8.35 in the compiler's order and
  // 6.91 so on zeros, 9.01 and 8.19 on random numbers, where power sets the clock: microbench/score_mix.hip.)  `ready`: units[0] holds the first unit's products; afterwards it holds those of `next`, the tile behind it.
  constexpr int UNITS = C::SUB * NT;
  Acc units[2];
  R keys;
  auto unit_step = [&](Acc& unit, auto uc, auto kc) __attribute__((always_inline)) {  // k-step kc of unit u
    constexpr int u = decltype(uc)::value % UNITS, kk = decltype(kc)::value;
    if constexpr (kk == 0) unit = R::zero();
    keys.step(unit, b[u % NT], 0, kk);
  };
  auto first_unit = [&](const u32x4* buf) __attribute__((always_inline)) {
    keys.read(buf, 0, lane);
    static_for<R::KK>([&](auto kc) { unit_step(units[0], std::integral_constant<int, 0>{}, kc); });
  };
  auto piped_tile = [&](const u32x4* buf, const u32x4* next) __attribute__((always_inline)) {
    static_for<UNITS>([&](auto uc) {
      constexpr int u = decltype(uc)::value, cur = u & 1, ct = u % NT, per = R::E / R::KK;
      float e[R::E], sum[4];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < R::E; ++r) e[r] = __builtin_fmaf(units[cur].get(r), c, nref[ct]);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(2);
      static_for<R::KK>([&](auto kc) {
        unit_step(units[cur ^ 1], std::integral_constant<int, u + 1>{}, kc);
#pragma unroll
        for (int r = decltype(kc)::value * per; r < (decltype(kc)::value + 1) * per; ++r) e[r] = __builtin_amdgcn_exp2f(e[r]);
        __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_s_setprio(0);
      // the products of the sub-tile's last unit are issued: its fragments make way for the next one's
      if constexpr (ct == NT - 2) {
        constexpr int s = u / NT + 1;
        if constexpr (s < C::SUB) keys.read(buf, s * 32, lane);
        else keys.read(next, 0, lane);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] = e[r];
#pragma unroll
      for (int r = 4; r < R::E; ++r) sum[r & 3] += e[r];
      lsum[ct] += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  // Where a chain of the tile at row0 (32 keys from jbase on, the wave's 32 columns cs) stands: nothing of it is visible,
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
  auto mask_chain = [&](Acc& acc, bool is_rec, int jbase, int ct) {
    const int first = is_rec ? qlo[ct] : 0, last = is_rec ? qi[ct] : N - 1;
    const int from = first - (jbase + rows4);
    const uint32_t span = (uint32_t)(last - first);
#pragma unroll
    for (int r = 0; r < R::E; ++r) acc.set(r, (uint32_t)(R::acc_row(r) - from) <= span ? acc.get(r) : kNegInf);
  };
  // one sub-tile of 32 keys: its visible chains, masked where they are cut, go to `sum`; false: nothing of it or behind it is visible
  auto cut_rows = [&](const u32x4* buf, bool is_rec, int s, int row0, int limit, auto&& sum) {
    const int jbase = row0 + s * 32;
    if (hidden(is_rec, jbase, limit, NCOL - 1)) return false;
    R a;
    a.read(buf, s * 32, lane);
#pragma unroll
    for (int cs = 0; cs < NCOL; ++cs) {
      if (hidden(is_rec, jbase, limit, cs)) continue;
      Acc acc[NS];
#pragma unroll
      for (int e = 0; e < NS; ++e) acc[e] = a.product(b[NS * cs + e], R::zero());
      if (cut(is_rec, jbase, limit, cs)) {
#pragma unroll
        for (int e = 0; e < NS; ++e) mask_chain(acc[e], is_rec, jbase, NS * cs + e);
      }
#pragma unroll
      for (int e = 0; e < NS; ++e) sum(acc[e], NS * cs + e);
    }
    return true;
  };
  // a tile that causality, a chunk boundary or the end of the context cuts: its visible chains, summed without checks
  auto cut_tile = [&](const u32x4* buf, bool is_rec, int row0, int limit) {
#pragma unroll 1
    for (int s = 0; s < C::SUB; ++s)
      if (!cut_rows(buf, is_rec, s, row0, limit, [&](const Acc& acc, int ct) { lsum[ct] += fast_sum(acc, ct); })) break;
  };
  // the first reference of every column: the largest visible logit that the lane has of the first 32 keys of a tile (if any is visible)
  auto first_reference = [&](const u32x4* buf, bool interior, bool is_rec, int row0) {
    R a;
    a.read(buf, 0, lane);
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
      Acc acc = a.product(b[ct], R::zero());
      if (!interior) mask_chain(acc, is_rec, row0, ct);
      const float tm = max_of<R>(acc, kNegInf) * c;
      if (tm > -1.0e30f) nref[ct] = -tm;
    }
  };

  // sums a tile without checks; false, and the sums as they were, if one of them went out of range
  auto sum_unchecked = [&](auto&& sum_tile) {
    float before[NT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) before[ct] = lsum[ct];
    sum_tile();
    bool bad = false;
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) bad |= !(lsum[ct] < kTileRedo);
    if (__builtin_amdgcn_ballot_w64(bad) == 0) return true;
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) lsum[ct] = before[ct];
    return false;
  };

  if (total > 0) {
    Regs second;  // the first two tiles are asked for together
    fetch(0);
    if (total > 1) fetch_to(second, 1);
    PKV_STORE(regs, lds, 0);
    if (total > 1) PKV_STORE(second, lds + C::TILE_U4, 1);
  }
  // Every load so far (the wave's queries among them) has landed before the loop: a share without tiles skips the stores that
  // wait for them, so without this the compiler cannot tell that they arrived long ago, and waits in front of the MFMAs of
  // every tile for the prefetch just issued (16 layers of 32 heads, 64 queries of 9000 keys, both passes: 262 -> 253 us).
  __builtin_amdgcn_s_waitcnt(kVmcnt0);
  if (total > 2) fetch(2);

  bool ready = false;
  for (int t = 0; t < total; ++t) {
    // every wave has finished tile t-1: its buffer takes tile t+2, the registers take tile t+3
    __syncthreads();
    if (t + 2 < total) PKV_STORE(regs, lds + ((t + 2) % kNBuf) * C::TILE_U4, t + 2);
    if (t + 3 < total) fetch(t + 3);
    // a wave without a query helps with the tiles only (as in pass 2 one without a key; both passes: 16 x 32 heads of 300 queries and keys 49.5 ->
    // 47.1 us, causal 42.2 -> 40.3, 28 x 12 heads of 128, 1100 334 -> 326)
    if (wave_i_lo >= N_q) continue;
    const u32x4* buf = lds + (t % kNBuf) * C::TILE_U4;
    const int tg = t0 + t;
    if constexpr (PIPE) {
      static_assert(W == 32 && NT >= 2 && NT % 2 == 0, "units of a column tile, two at a time");
      const bool is_rec = tg >= n_ctx;
      const int row0 = is_rec ? rec_lo + (tg - n_ctx) * C::ROWS : tg * C::ROWS, limit = is_rec ? i_end : N;
      const bool interior = is_rec ? row0 + C::ROWS - 1 <= i0 && row0 >= ((i_end - 1) / chunk) * chunk : row0 + C::ROWS <= N;
      if (t == 0) first_reference(buf, interior, is_rec, row0);
      if (interior) {
        if (!ready) first_unit(buf);
        ready = sum_unchecked([&]() __attribute__((always_inline)) { piped_tile(buf, lds + ((t + 1) % kNBuf) * C::TILE_U4); });
        if (ready) continue;
      } else {
        ready = false;
        if (sum_unchecked([&]() __attribute__((always_inline)) { cut_tile(buf, is_rec, row0, limit); })) continue;
      }
#pragma unroll 1
      for (int s = 0; s < C::SUB; ++s)
        if (!cut_rows(buf, is_rec, s, row0, limit, accumulate)) break;
      continue;
    }
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
      for (int s = 0; s < C::SUB; ++s)
        if (!cut_rows(buf, is_rec, s, row0, limit, accumulate)) break;
    }
  }
  // a column's sums lie in 64 / W lanes, each with a reference of its own
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    float m = -nref[ct], tot = lsum[ct];
#pragma unroll
    for (int x = W; x < 64; x *= 2) {
      const float m2 = __shfl_xor(m, x, 64), l2 = __shfl_xor(tot, x, 64), mm = __builtin_fmaxf(m, m2);
      tot = tot * __builtin_amdgcn_exp2f(m - mm) + l2 * __builtin_amdgcn_exp2f(m2 - mm);
      m = mm;
    }
    const size_t at = split0 + (size_t)(l * H_q + h) * N_q + qi[ct];
    const float whole = -(m + __builtin_amdgcn_logf(tot)) * inv_c;
    if (lane < W && qi[ct] < N_q) {
      if constexpr (SPLIT && D == 64) {
        reinterpret_cast<LsePart*>(neg_lse)[at] = LsePart{m, tot};
      } else if constexpr (SPLIT) {  // also launched with one split
        if (splits > 1) reinterpret_cast<LsePart*>(neg_lse)[at] = LsePart{m, tot};
        else neg_lse[at] = whole;
      } else {
        neg_lse[at] = whole;
      }
    }
  }
}

}  // namespace

constexpr int kLseCols = 2;  // column sub-tiles per wave; 128 * kLseCols queries per workgroup

// the query blocks of a head are dealt over all XCDs (measured: fewer L2 misses than one KV group per XCD, whose
// blocks drift apart along a key stream slightly larger than the L2)
inline dim3 lse_grid(int L_s, int H_q, int64_t N_q, int splits) {
  return dim3((unsigned)((N_q + 128 * kLseCols - 1) / (128 * kLseCols) * splits), (unsigned)H_q, (unsigned)L_s);
}

}  // namespace pkv
