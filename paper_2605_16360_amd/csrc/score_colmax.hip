// Proxy importance scoring, pass 2 (paper Sec. 3: the softmax probabilities of Q K^T / sqrt(d),
// reduced over the query axis to one score per context key): per context key, the maximum over all
// reconstruction queries and over the query heads of the GQA group of exp(logit - lse).
//
// The logit matrix is never stored: Q K^T tiles are recomputed.  The
// context keys of a workgroup (the "columns", 32*NCOL per wave) stay in registers as the MFMA B
// operand for the whole kernel; the queries (the "rows") stream through 16 KB LDS tiles.  With
// rows on the MFMA M axis a lane owns a key column and some query rows of every tile, so the
// maximum over queries runs inside a lane and needs one or two cross-lane steps at the end.
//
// The max form keeps the matrix pipe busy 83 % of the cycles, so the chip's power sets its clock: it uses v_mfma_f32_16x16x32_bf16,
// which draw less per flop than 32 x 32 x 16.  Both passes, in steady repetition: 16 x 32 heads of 64, 8192 keys 9390 -> 9030 us;
// 28 x 12 heads of 128 (pass 1 with the same), 10 007 keys 18 440 -> 17 000.
//
// With c = log2(e) / sqrt(d) the probability is p = 2^(c*s - L2), L2 the row's log2-sum-exp2.
// Pass 1 stores -L2 / c per query row; it is fed to the MFMA as the accumulator's initial value,
// so tiles come out as s - L2/c and need nothing but a running maximum (v_max3); one exp2 per
// context key is taken at the very end (max and exp commute).  The result is a probability: rounding in
// s - L2/c can carry it a few ulp past one, so it is clamped to one.
//
// Streaming: three LDS buffers and one barrier per tile.  While tile t is computed, tile t+2 goes
// from registers to LDS and tile t+3 is fetched from global memory into registers, all issued
// behind the first MFMAs of the tile.  The issue order inside a tile is written out by hand and
// pinned with scheduling barriers: the MFMAs of one pair of column sub-tiles alternate with the
// v_max3 that reduce the previous pair.
#include "kernels.hpp"
#include "score_common.hpp"

namespace pkv {
namespace {

// ---------------------------------------------------------------------------------------------
// pass 2: x[l, hs, n] = 2^(c * max_{g, i} (<q^{(hs*G+g)}_i, k_n> + neg_lse[l, hs*G+g, i]))
// one-dimensional grid over (KV group, key block of 128*NCOL keys), 256 threads; wave w owns context keys
// [n0 + 32*NCOL*w, +32*NCOL) as the resident B operand and streams all G*N_q queries.
// Rows past N_q carry -inf as their initial value, so every sub-tile is processed without a branch.
// Chains are handled in pairs (two column sub-tiles): the MFMAs of pair i are issued while the
// VALU reduces the accumulators of pair i-1 (also across tile boundaries).
// ---------------------------------------------------------------------------------------------
// SPLIT (see score_lse.hpp): neg_lse holds shares.  QSPLIT: the query tiles of a key block are dealt to q_splits workgroups, and
// each raises x (cleared by pass 1; probabilities are not negative, so their bits compare like integers).
template <int D, int NCOL, bool SPLIT, bool QSPLIT>
__global__ __launch_bounds__(256, D == 128 ? 1 : 2) void score_colmax_kernel(const uint16_t* __restrict__ q,
                                                               const uint16_t* __restrict__ k_ctx,
                                                               const float* __restrict__ neg_lse,
                                                               float* __restrict__ x, int L_s, int H_q, int G, int N, int N_q,
                                                               float c, float inv_c, int splits, int q_splits) {
  using C = ScoreCfg<D>;
  using R = Rows32<D, 16>;
  static_assert(NCOL % 2 == 0, "column sub-tiles are processed in pairs");
  __shared__ u32x4 lds[kNBuf * C::TILE_U4];
  __shared__ __attribute__((aligned(16))) float lds_nl[kNBuf * C::ROWS];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, quad = lane >> 4;
  constexpr int KB = 128 * NCOL;
  const int H_kv = H_q / G;
  // a group's blocks: its key blocks (they stream the same queries), each in q_splits parts
  const GroupBlock gb = group_block(L_s * H_kv, (N + KB - 1) / KB * (QSPLIT ? q_splits : 1));
  if (gb.group >= L_s * H_kv) return;
  const int l = gb.group / H_kv, hs = gb.group % H_kv;
  const int n0 = (QSPLIT ? gb.item / q_splits : gb.item) * KB;
  const uint16_t* kc = k_ctx + (size_t)(l * H_kv + hs) * N * D;

  constexpr int NT = 2 * NCOL;  // column tiles of 16
  bf16x8 b[NT][R::KK];
  int kn[NT];
  float runmax[NT];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    kn[ct] = n0 + (wave * NT + ct) * 16 + (lane & 15);
    R::columns(b[ct], kc, kn[ct] < N ? kn[ct] : N - 1, lane);
    runmax[ct] = kNegInf;
  }

  // tiles are fetched in order: head g = 0..G-1 of the group, query tile qt = 0..nqt-1
  const int nqt = (N_q + C::ROWS - 1) / C::ROWS;
  const int part = QSPLIT ? gb.item % q_splits : 0;
  const int first = QSPLIT ? (int)((int64_t)G * nqt * part / q_splits) : 0;
  const int total = QSPLIT ? (int)((int64_t)G * nqt * (part + 1) / q_splits) - first : G * nqt;
  TileRegs<D> regs;
  LseRegs<SPLIT> nl_reg;
  nl_reg.none();
  int fg = QSPLIT ? first / nqt : 0, fqt = QSPLIT ? first % nqt : 0;
  auto fetch_next = [&]() {
    const size_t head = (size_t)(l * H_q + hs * G + fg);
    tile_fetch<D>(regs, q + head * N_q * D, fqt * C::ROWS, N_q, tid);
    if (tid < C::ROWS) {
      const int i = fqt * C::ROWS + tid;
      if (i < N_q) nl_reg.read(neg_lse, head * N_q + i, (size_t)L_s * H_q * N_q, splits);
      else nl_reg.none();
    }
    if (++fqt == nqt) {
      fqt = 0;
      ++fg;
    }
  };
  auto store = [&](int t) {
    tile_store<D>(regs, lds + (t % kNBuf) * C::TILE_U4, tid);
    if (tid < C::ROWS) lds_nl[(t % kNBuf) * C::ROWS + tid] = nl_reg.neg_lse(inv_c);
  };
  fetch_next();
  store(0);
  if (total > 1) {
    fetch_next();
    store(1);
  }
  if (total > 2) fetch_next();
  __syncthreads();

  // Fragments and initial values of the current 32-row sub-tile, refilled in place: a[rt][kk] right behind
  // the last MFMA that consumes it, init[rt] behind the last one that starts from it.
  bf16x8 a[2][R::KK];
  f32x4 init[2];
  auto load_a = [&](int t, int s, int rt, int kk) {
    a[rt][kk] = frag_read<D>(lds + (t % kNBuf) * C::TILE_U4, s * 32 + rt * 16 + (lane & 15), kk * 4 + quad);
  };
  auto load_init = [&](int t, int s, int rt) {
    init[rt] = *reinterpret_cast<const f32x4*>(&lds_nl[(t % kNBuf) * C::ROWS + s * 32 + rt * 16 + quad * 4]);
  };
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
    for (int kk = 0; kk < R::KK; ++kk) load_a(0, 0, rt, kk);
    load_init(0, 0, rt);
  }
  // accumulators of the four column tiles of the pair before
  f32x4 pend[2][4];
#pragma unroll
  for (int i = 0; i < 8; ++i) pend[i >> 2][i & 3] = f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
  // step v of 16: first all of the first sixteen rows, whose MFMAs were done first
  auto max_step = [&](auto vc, int pp) {
    constexpr int v = decltype(vc)::value, rt = v >> 3, ct = (v >> 1) & 3, e = (v & 1) * 2;
    runmax[pp * 4 + ct] = max3f(runmax[pp * 4 + ct], pend[rt][ct][e], pend[rt][ct][e + 1]);
  };
  constexpr int NP = NCOL / 2;  // pairs per sub-tile
  if (n0 + wave * NT * 16 >= N) {  // a wave without a key helps with the tiles only
    for (int t = 0; t < total; ++t) {
      __syncthreads();
      if (t + 2 < total) store(t + 2);
      if (t + 3 < total) fetch_next();
    }
    return;
  }
  for (int t = 0; t < total; ++t) {
    static_for<C::SUB * NP>([&](auto ic) {
      constexpr int i = decltype(ic)::value, s = i / NP, pr = i % NP;
      constexpr int pp = (pr + NP - 1) % NP;  // pair whose accumulators are pending
      constexpr int NM = 8 * R::KK;
      f32x4 acc[2][4];
      static_for<NM>([&](auto jc) {
        // of two MFMAs in a row one operand is the same: the less of their input changes, the less they draw
        constexpr int j = decltype(jc)::value, kk = j / 8, rt = (j >> 2) & 1, ct = rt ? 3 - (j & 3) : (j & 3);
        acc[rt][ct] = mfma_bf16_16x16x32(a[rt][kk], b[4 * pr + ct][kk], kk == 0 ? init[rt] : acc[rt][ct]);
        if constexpr (i == 0 && j == 1) {
          // every wave has finished tile t-1: its buffer takes tile t+2, the registers take tile t+3
          __syncthreads();
          if (t + 2 < total) store(t + 2);
          if (t + 3 < total) fetch_next();
        }
        if constexpr (pr == NP - 1 && (j & 3) == 3) {
          // last pair of the sub-tile: refill from the next sub-tile (sub-tile 0 of the next tile after the last;
          // past the last tile this reads a stale buffer, harmlessly)
          constexpr int next = s + 1 < C::SUB ? 0 : 1, sn = s + 1 < C::SUB ? s + 1 : 0;
          load_a(t + next, sn, rt, kk);
          if constexpr (kk == 0) load_init(t + next, sn, rt);
        }
        // the 16 v_max3 of the pending pair behind MFMAs 2, 3, ... (its last MFMAs have retired by then)
        if constexpr (j >= 2) {
          constexpr int g = j - 2, lo = (16 * g) / (NM - 2), hi = (16 * (g + 1)) / (NM - 2);
          static_for<hi - lo>([&](auto vc) { max_step(std::integral_constant<int, lo + decltype(vc)::value>{}, pp); });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
      for (int e = 0; e < 8; ++e) pend[e >> 2][e & 3] = acc[e >> 2][e & 3];
    });
  }
  static_for<16>([&](auto vc) { max_step(vc, NP - 1); });
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    const float p = __builtin_fminf(__builtin_amdgcn_exp2f(c * quads_max(runmax[ct])), 1.0f);
    if (quad == 0 && kn[ct] < N) {
      float* dst = x + (size_t)(l * H_kv + hs) * N + kn[ct];
      if constexpr (QSPLIT) atomicMax(reinterpret_cast<unsigned int*>(dst), __float_as_uint(p));
      else *dst = p;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// pass 2, sum form (the accumulation over the query axis that Sec. 3 prints for the proxy feature):
//   x[l, hs, n] = sum over the heads g of the group and all queries i of 2^(c * (<q_i, k_n> + neg_lse[l, h, i]))
// Same geometry as the max form (a workgroup owns 128*NCOL context keys as the resident B operand and
// streams all G*N_q queries, -L2/c as the accumulator's initial value), but every element is exponentiated
// and added: mul, exp2, add per element, so this kernel is bound by the vector ALU like pass 1.  A probability
// never exceeds one, so there is no reference to track.  Rows past N_q carry -inf and add zero.
// ---------------------------------------------------------------------------------------------
//
// CAUSAL: the proxy's own prefill attention (N_q == N, the keys are the sequence's own): query i sees keys n <= i, so a
// workgroup starts at the query tile that holds its first key and masks the tiles that the diagonal cuts.
//
// With q_splits > 1 the query tiles of a key block are dealt to that many workgroups and x holds their sums one behind the
// other, [q_splits][L_s * H_kv * N]; sum_parts_kernel adds them up in that order.
template <int D, int NCOL, int W, bool CAUSAL, bool SPLIT>
__global__ __launch_bounds__(256, D == 64 && !(CAUSAL && SPLIT) ? 3 : 2) void score_colsum_kernel(const uint16_t* __restrict__ q,
                                                               const uint16_t* __restrict__ k_ctx,
                                                               const float* __restrict__ neg_lse,
                                                               float* __restrict__ x, int L_s, int H_q, int G, int N, int N_q,
                                                               float c, float inv_c, int splits, int q_splits) {
  using C = ScoreCfg<D>;
  using R = Rows32<D, W>;
  using Acc = typename R::Acc;
  __shared__ u32x4 lds[kNBuf * C::TILE_U4];
  __shared__ __attribute__((aligned(16))) float lds_nl[kNBuf * C::ROWS];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, rows4 = lane / W * 4;
  constexpr int KB = 128 * NCOL;
  const int H_kv = H_q / G;
  // a group's blocks: its key blocks (they stream the same queries), each in q_splits parts
  const int per_group = (N + KB - 1) / KB * q_splits;
  const int n_groups = L_s * H_kv;
  GroupBlock gb = group_block(n_groups, per_group);
  if constexpr (CAUSAL) {
    // the first key block has the most queries; an XCD takes four groups (or as many as fill its 96 places) at a time
    // (16 x 32 heads of 64, both passes: 4097 tokens 1590 -> 1582 us, 1000 tokens 156 -> 137; all 16 groups at once, whose queries
    // do not fit the L2, 4097 tokens 1602).  Groups that do not go round the XCDs evenly are dealt over
    // all of them (one layer of 4 heads, 11 000 tokens 260 -> 134 us).
    const int sets = per_group < 32 ? 128 / per_group : 4;
    const bool even = n_groups % kScoreXcds == 0;
    const int j = blockIdx.x / (even ? kScoreXcds : 1);
    if (j >= (even ? n_groups / kScoreXcds : n_groups) * per_group) return;
    const SetItem it = longest_first(j, even ? n_groups / kScoreXcds : n_groups, per_group, even ? sets : kScoreXcds * sets);
    gb = {even ? it.set * kScoreXcds + (int)blockIdx.x % kScoreXcds : it.set, it.item};
  }
  if (gb.group >= L_s * H_kv) return;
  const int l = gb.group / H_kv, hs = gb.group % H_kv;
  const int n0 = gb.item / q_splits * KB, part = gb.item % q_splits;
  const uint16_t* kc = k_ctx + (size_t)(l * H_kv + hs) * N * D;

  constexpr int NT = 32 * NCOL / W;  // column tiles
  bf16x8 b[NT][R::KK];
  int kn[NT];
  float colsum[NT];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    kn[ct] = n0 + (wave * NT + ct) * W + lane % W;
    R::columns(b[ct], kc, kn[ct] < N ? kn[ct] : N - 1, lane);
    colsum[ct] = 0.0f;
  }

  // tiles are fetched in order: head g = 0..G-1 of the group, query tile qt = 0..nqt-1
  const int nqt = (N_q + C::ROWS - 1) / C::ROWS;
  const int qt_first = CAUSAL ? n0 / C::ROWS : 0;  // KB is a multiple of ROWS
  const int nqg = nqt - qt_first;  // tiles per head
  const int first = (int)((int64_t)G * nqg * part / q_splits), total = (int)((int64_t)G * nqg * (part + 1) / q_splits) - first;
  TileRegs<D> regs;
  LseRegs<SPLIT> nl_reg;
  nl_reg.none();
  int fg = first / nqg, fqt = qt_first + first % nqg;
  auto fetch_next = [&]() {
    const size_t head = (size_t)(l * H_q + hs * G + fg);
    tile_fetch<D>(regs, q + head * N_q * D, fqt * C::ROWS, N_q, tid);
    if (tid < C::ROWS) {
      const int i = fqt * C::ROWS + tid;
      if (i < N_q) nl_reg.read(neg_lse, head * N_q + i, (size_t)L_s * H_q * N_q, splits);
      else nl_reg.none();
    }
    if (++fqt == nqt) {
      fqt = qt_first;
      ++fg;
    }
  };
  auto store = [&](int t) {
    tile_store<D>(regs, lds + (t % kNBuf) * C::TILE_U4, tid);
    if (tid < C::ROWS) lds_nl[(t % kNBuf) * C::ROWS + tid] = nl_reg.neg_lse(inv_c);
  };
  if (total > 0) {
    fetch_next();
    store(0);
  }
  if (total > 1) {
    fetch_next();
    store(1);
  }
  __builtin_amdgcn_s_waitcnt(kVmcnt0);  // the resident keys have landed: no tile waits for them (see score_lse.hpp)
  if (total > 2) fetch_next();

  const bool idle = n0 + wave * NCOL * 32 >= N;  // a wave without a key helps with the tiles only
  // As pass 1's piped tiles (score_lse.hpp): a unit of one column tile and 32 queries at a time, its exponentials between the next one's products
  // (24 x 14 heads of 64, 6001 keys, both passes 3862 -> 3793 us; 16 x 32, 2000 851 -> 835; not where there are few queries: one layer of 4 heads,
  // 300 queries of 500 keys 18.1 -> 18.4).
  constexpr bool kPiped = !CAUSAL && !SPLIT && W == 32;
  constexpr int UNITS = C::SUB * NT;
  Acc units[2], init;
  R rows;
  auto read_rows = [&](const u32x4* buf, const float* nl, int s) __attribute__((always_inline)) {
    rows.read(buf, s * 32, lane);
#pragma unroll
    for (int r = 0; r < R::E; r += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&nl[s * 32 + R::acc_row(r) + rows4]);
#pragma unroll
      for (int e = 0; e < 4; ++e) init.set(r + e, v[e]);
    }
  };
  auto unit_step = [&](Acc& unit, auto uc, auto kc) __attribute__((always_inline)) {
    constexpr int u = decltype(uc)::value % UNITS, kk = decltype(kc)::value;
    if constexpr (kk == 0) unit = init;
    rows.step(unit, b[u % NT], 0, kk);
  };
  auto first_unit = [&](const u32x4* buf, const float* nl) __attribute__((always_inline)) {
    read_rows(buf, nl, 0);
    static_for<R::KK>([&](auto kc) { unit_step(units[0], std::integral_constant<int, 0>{}, kc); });
  };
  auto piped_tile = [&](const u32x4* buf, const float* nl, const u32x4* next, const float* next_nl) __attribute__((always_inline)) {
    static_for<UNITS>([&](auto uc) {
      constexpr int u = decltype(uc)::value, cur = u & 1, ct = u % NT, per = R::E / R::KK;
      float e[R::E], sum[4];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < R::E; ++r) e[r] = units[cur].get(r) * c;
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(2);
      static_for<R::KK>([&](auto kc) {
        unit_step(units[cur ^ 1], std::integral_constant<int, u + 1>{}, kc);
#pragma unroll
        for (int r = decltype(kc)::value * per; r < (decltype(kc)::value + 1) * per; ++r) e[r] = __builtin_amdgcn_exp2f(e[r]);
        __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_s_setprio(0);
      if constexpr (ct == NT - 2) {
        constexpr int s = u / NT + 1;
        if constexpr (s < C::SUB) read_rows(buf, nl, s);
        else read_rows(next, next_nl, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] = e[r];
#pragma unroll
      for (int r = 4; r < R::E; ++r) sum[r & 3] += e[r];
      colsum[ct] += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  bool ready = false;
  int cqt = qt_first + first % nqg;  // query tile of step t
  for (int t = 0; t < total; ++t) {
    // every wave has finished tile t-1: its buffer takes tile t+2, the registers take tile t+3
    __syncthreads();
    if (t + 2 < total) store(t + 2);
    if (t + 3 < total) fetch_next();
    if (idle) continue;
    const u32x4* buf = lds + (t % kNBuf) * C::TILE_U4;
    const float* nl = lds_nl + (t % kNBuf) * C::ROWS;
    const int row0 = cqt * C::ROWS;
    const bool diag = CAUSAL && row0 < n0 + KB - 1;  // some query of the tile lies before some key of the block
    if (++cqt == nqt) cqt = qt_first;
    if constexpr (kPiped) {
      if (!ready) first_unit(buf, nl);
      ready = t + 1 < total;
      piped_tile(buf, nl, lds + ((t + 1) % kNBuf) * C::TILE_U4, lds_nl + ((t + 1) % kNBuf) * C::ROWS);
      continue;
    }
    // (unrolled, the four sub-tiles of the causal form take 256 registers and with them the third workgroup per CU)
    constexpr int kUnroll = CAUSAL ? 2 : C::SUB;
#pragma unroll kUnroll
    for (int s = 0; s < C::SUB; ++s) {
      R a;
      a.read(buf, s * 32, lane);
      Acc init;
#pragma unroll
      for (int r = 0; r < R::E; r += 4) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(&nl[s * 32 + R::acc_row(r) + rows4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) init.set(r + e, v[e]);
      }
      Acc acc[NT];
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) acc[ct] = a.product(b[ct], init);
      if (diag) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
          for (int r = 0; r < R::E; ++r)
            acc[ct].set(r, row0 + s * 32 + rows4 + R::acc_row(r) >= kn[ct] ? acc[ct].get(r) : kNegInf);
      }
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = __builtin_amdgcn_exp2f(acc[ct].get(r) * c);
#pragma unroll
        for (int r = 4; r < R::E; ++r) v[r & 3] += __builtin_amdgcn_exp2f(acc[ct].get(r) * c);
        colsum[ct] += (v[0] + v[1]) + (v[2] + v[3]);
      }
    }
  }
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    float tot = colsum[ct];
#pragma unroll
    for (int o = W; o < 64; o *= 2) tot += __shfl_xor(tot, o, 64);
    if (lane < W && kn[ct] < N) x[((size_t)part * L_s * H_kv + l * H_kv + hs) * N + kn[ct]] = tot;
  }
}

__global__ __launch_bounds__(256) void sum_parts_kernel(const float* __restrict__ parts, int n_parts, int64_t n, float* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float v = parts[i];
  for (int p = 1; p < n_parts; ++p) v += parts[(size_t)p * n + i];
  x[i] = v;
}

// fp32 -> bf16 of up to three arrays in one launch, eight elements per thread (n counts eights; every array of queries or
// keys is a multiple of eight long)
struct ConvertArgs {
  const float* in[3];
  uint16_t* out[3];
  int64_t n[3];
};
__global__ __launch_bounds__(256) void f32_to_bf16_kernel(ConvertArgs a) {
  const int64_t stride = (int64_t)gridDim.x * 256, total = a.n[0] + a.n[1] + a.n[2];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
    const int64_t i1 = i - a.n[0], i2 = i1 - a.n[1];
    const float* in = i1 < 0 ? a.in[0] + i * 8 : (i2 < 0 ? a.in[1] + i1 * 8 : a.in[2] + i2 * 8);
    uint16_t* out = i1 < 0 ? a.out[0] + i * 8 : (i2 < 0 ? a.out[1] + i1 * 8 : a.out[2] + i2 * 8);
    const f32x4 v = *reinterpret_cast<const f32x4*>(in), w = *reinterpret_cast<const f32x4*>(in + 4);
    *reinterpret_cast<u32x4*>(out) = u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3])};
  }
}

}  // namespace

hipError_t launch_f32_to_bf16(const float* const in[3], uint16_t* const out[3], const int64_t n[3], hipStream_t stream) {
  ConvertArgs a;
  int64_t total = 0;
  for (int i = 0; i < 3; ++i) {
    if (n[i] % 8 != 0) return hipErrorInvalidValue;
    a.in[i] = in[i];
    a.out[i] = out[i];
    a.n[i] = n[i] / 8;
    total += a.n[i];
  }
  if (total <= 0) return hipSuccess;
  const int64_t blocks = (total + 255) / 256;
  f32_to_bf16_kernel<<<(unsigned)(blocks < 16384 ? blocks : 16384), 256, 0, stream>>>(a);
  return hipGetLastError();
}

// Columns of an MFMA tile in the sum form.  Where mul, exp2 and add take much longer than the products (d = 64) the wide tile's fewer
// instructions are level or ahead (24 x 14 heads, 6001 keys, both passes 4303 us, 4317 with 16; one layer of 3000 keys, 300 queries 24.8
// and 25.2); the causal form spills 20 registers with it (16 x 32 heads, 4097 tokens 1664, 1543 with 16).
constexpr int kSumW(int d, bool causal) { return d == 64 && !causal ? 32 : 16; }
constexpr int kMaxCols = 4, kSumCols = 2;  // column sub-tiles per wave of the two forms
constexpr int64_t kMaxSumParts = 16, kMaxTurns = 64;
static int64_t pass2_slots(bool sum, int d) { return 256 * (d == 64 ? (sum ? 3 : 2) : (sum ? 2 : 1)); }

// Workgroups per key block in pass 2.  All workgroups take equally long, so `blocks` of them on `slots` places take
// ceil(blocks / slots) turns, the last of which may be nearly empty (1152 on 768: two turns for one and a half's work);
// s workgroups per block take ceil(s * blocks / slots) turns of a part each.  A part takes its share of the block's query tiles
// and a start: the resident keys and the first tiles have to arrive, as long as four tiles take in the max form, whose part loads
// twice the keys of the sum form's two (one in the causal form, whose parts are not equally long: the late ones are short).
// Parts of fewer than two tiles would only wait for memory.
// Measured, without and with: 28 x 2 heads of 128, 10 007 keys (4.4 turns' work in 5) 7830 -> 7160 us; the sum form,
// 24 x 2 heads of 64, 6001 keys (1.5 in 2) 2212 -> 2060 us; causal, 16 x 8 heads, 4097 keys 1164 -> 950 us.  Short streams,
// with a start of one tile and as here, both passes: 28 x 2 heads of 128, 4096 keys, 200 queries 237 -> 224 us (217 before
// any were split), 2000 keys, 800 queries 436 -> 400 us (397); the sum form, 16 x 8 heads of 64, 2000 keys, 64 queries
// 84.5 -> 82 us; the causal form with a start of two tiles instead of one, 4097 keys, 1660 -> 1810 us.
int score_query_splits(bool sum, bool causal, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q) {
  const int cols = 128 * (sum ? kSumCols : kMaxCols);
  const int64_t slots = pass2_slots(sum, d);
  const int64_t blocks = (N + cols - 1) / cols * L_s * H_kv;
  const int64_t tiles = (int64_t)(H_q / H_kv) * ((N_q + 8192 / d - 1) / (8192 / d));
  int64_t most = slots / blocks > 8 ? slots / blocks : 8;
  if (sum && most > kMaxSumParts) most = kMaxSumParts;  // each part's sums are written and read again
  if (most > kMaxTurns * slots / blocks) most = kMaxTurns * slots / blocks;  // one more saves no more than a 64th
  if (most > tiles / 2) most = tiles / 2;
  const double start = causal ? 1.0 : (sum ? 2.0 : 4.0);
  int64_t best = 1;
  double best_cost = 1e30;
  for (int64_t s = 1; s <= most || s == 1; ++s) {
    const double cost = (double)((blocks * s + slots - 1) / slots) * ((double)tiles / (double)s + start);
    if (cost < best_cost * 0.985) {
      best = s;
      best_cost = cost;
    }
  }
  return (int)best;
}

// The most that the parts of any input of up to N keys take: at most kMaxSumParts per block, kMaxTurns * slots workgroups.
size_t score_parts_bytes(int L_s, int H_kv, int d, int64_t N) {
  const int64_t cols = 128 * kSumCols, blocks = (N + cols - 1) / cols * L_s * H_kv;
  const int64_t wgs = kMaxSumParts * blocks < kMaxTurns * pass2_slots(true, d) ? kMaxSumParts * blocks : kMaxTurns * pass2_slots(true, d);
  return (size_t)(wgs * cols) * 4;
}

hipError_t launch_score_colsum(const uint16_t* q, const uint16_t* k_ctx, const float* neg_lse, int splits, float* x, float* parts,
                               int q_splits, int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, bool causal,
                               hipStream_t stream) {
  const int G = H_q / H_kv;
  const float c = 1.4426950408889634f / sqrtf((float)d), inv_c = 1.0f / c;
  constexpr int NCOL = kSumCols;
  if ((causal && N != N_q) || q_splits < 1 || (q_splits > 1 && !parts)) return hipErrorInvalidValue;
  const unsigned grid = group_grid((int64_t)L_s * H_kv, (N + 128 * NCOL - 1) / (128 * NCOL) * q_splits);
  if (grid == 0) return hipErrorInvalidValue;
  float* out = q_splits > 1 ? parts : x;
  auto go = [&](auto dc, auto cc, auto sc) {
    score_colsum_kernel<decltype(dc)::value, NCOL, kSumW(decltype(dc)::value, decltype(cc)::value), decltype(cc)::value, decltype(sc)::value>
        <<<grid, 256, 0, stream>>>(q, k_ctx, neg_lse, out, L_s, H_q, G, (int)N, (int)N_q, c, inv_c, splits, q_splits);
  };
  auto pick = [&](auto dc) {
    if (causal && splits > 1) go(dc, std::true_type{}, std::true_type{});
    else if (causal) go(dc, std::true_type{}, std::false_type{});
    else if (splits > 1) go(dc, std::false_type{}, std::true_type{});
    else go(dc, std::false_type{}, std::false_type{});
  };
  if (d == 64) pick(std::integral_constant<int, 64>{});
  else pick(std::integral_constant<int, 128>{});
  if (q_splits > 1) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)L_s * H_kv * N;
    sum_parts_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(parts, q_splits, n, x);
  }
  return hipGetLastError();
}

hipError_t launch_score_colmax(const uint16_t* q, const uint16_t* k_ctx, const float* neg_lse, int splits, float* x, int q_splits,
                               int L_s, int H_q, int H_kv, int d, int64_t N, int64_t N_q, hipStream_t stream) {
  const int G = H_q / H_kv;
  const float c = 1.4426950408889634f / sqrtf((float)d), inv_c = 1.0f / c;
  // d = 64: two workgroups per CU.  d = 128: one (the resident keys of 4 column sub-tiles alone take 128 registers): a wave
  // has the SIMD's whole register file, and the pinned issue order keeps the matrix pipe fed without a second wave
  constexpr int NCOL = kMaxCols;
  const unsigned grid = group_grid((int64_t)L_s * H_kv, (N + 128 * NCOL - 1) / (128 * NCOL) * q_splits);
  if (grid == 0 || q_splits < 1) return hipErrorInvalidValue;
  auto go = [&](auto dc, auto sc, auto qc) {
    score_colmax_kernel<decltype(dc)::value, NCOL, decltype(sc)::value, decltype(qc)::value>
        <<<grid, 256, 0, stream>>>(q, k_ctx, neg_lse, x, L_s, H_q, G, (int)N, (int)N_q, c, inv_c, splits, q_splits);
  };
  auto pick = [&](auto dc) {
    if (splits > 1) go(dc, std::true_type{}, std::true_type{});  // (few blocks: always split both ways)
    else if (q_splits > 1) go(dc, std::false_type{}, std::true_type{});
    else go(dc, std::false_type{}, std::false_type{});
  };
  if (d == 64) pick(std::integral_constant<int, 64>{});
  else pick(std::integral_constant<int, 128>{});
  return hipGetLastError();
}

}  // namespace pkv
