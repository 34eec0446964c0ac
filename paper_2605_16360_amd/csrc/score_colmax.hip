// Proxy importance scoring, pass 2 (paper Sec. 3: the softmax probabilities of Q K^T / sqrt(d),
// reduced over the query axis to one score per context key): per context key, the maximum over all
// reconstruction queries and over the query heads of the GQA group of exp(logit - lse).
//
// The logit matrix is never stored: Q K^T tiles are recomputed with v_mfma_f32_32x32x16_bf16.  The
// context keys of a workgroup (the "columns", 32*NCOL per wave) stay in registers as the MFMA B
// operand for the whole kernel; the queries (the "rows") stream through 16 KB LDS tiles.  With
// rows on the MFMA M axis a lane owns ONE key column and 16 query rows of every tile, so the
// maximum over queries runs inside a lane and needs one cross-lane step (lane ^ 32) at the end.
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
// SPLIT (see score_lse.hip): neg_lse holds shares; the query tiles of a key block are dealt to q_splits workgroups as well, and
// each raises x (cleared by pass 1; probabilities are not negative, so their bits compare like integers).
template <int D, int NCOL, bool SPLIT>
__global__ __launch_bounds__(256, D == 128 ? 1 : 2) void score_colmax_kernel(const uint16_t* __restrict__ q,
                                                               const uint16_t* __restrict__ k_ctx,
                                                               const float* __restrict__ neg_lse,
                                                               float* __restrict__ x, int L_s, int H_q, int G, int N, int N_q,
                                                               float c, float inv_c, int splits, int q_splits) {
  using C = ScoreCfg<D>;
  static_assert(NCOL % 2 == 0, "column sub-tiles are processed in pairs");
  __shared__ u32x4 lds[kNBuf * C::TILE_U4];
  __shared__ __attribute__((aligned(16))) float lds_nl[kNBuf * C::ROWS];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  constexpr int KB = 128 * NCOL;
  const int H_kv = H_q / G;
  // a group's blocks: its key blocks (they stream the same queries), each in q_splits parts
  const GroupBlock gb = group_block((N + KB - 1) / KB * (SPLIT ? q_splits : 1));
  if (gb.group >= L_s * H_kv) return;
  const int l = gb.group / H_kv, hs = gb.group % H_kv;
  const int n0 = (SPLIT ? gb.item / q_splits : gb.item) * KB;
  const uint16_t* kc = k_ctx + (size_t)(l * H_kv + hs) * N * D;

  bf16x8 b[NCOL][C::KK];
  int kn[NCOL];
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) {
    kn[cs] = n0 + (wave * NCOL + cs) * 32 + l32;
    const int row = kn[cs] < N ? kn[cs] : N - 1;
#pragma unroll
    for (int kk = 0; kk < C::KK; ++kk)
      b[cs][kk] = as_bf16x8(*reinterpret_cast<const u32x4*>(kc + (size_t)row * D + kk * 16 + half * 8));
  }
  float runmax[NCOL];
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) runmax[cs] = kNegInf;

  // tiles are fetched in order: head g = 0..G-1 of the group, query tile qt = 0..nqt-1
  const int nqt = (N_q + C::ROWS - 1) / C::ROWS;
  const int part = SPLIT ? gb.item % q_splits : 0;
  const int first = SPLIT ? (int)((int64_t)G * nqt * part / q_splits) : 0;
  const int total = SPLIT ? (int)((int64_t)G * nqt * (part + 1) / q_splits) - first : G * nqt;
  TileRegs<D> regs;
  LseRegs<SPLIT> nl_reg;
  nl_reg.none();
  int fg = SPLIT ? first / nqt : 0, fqt = SPLIT ? first % nqt : 0;
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

  // Fragments and initial values of the current 32-row sub-tile, refilled in place: a[kk] right behind
  // the last MFMA that consumes it, init behind the pair's second MFMA (the last one that reads it).
  bf16x8 a[C::KK];
  f32x16 init;
  auto load_a = [&](int t, int s, int kk) {
    a[kk] = frag_read<D>(lds + (t % kNBuf) * C::TILE_U4, s * 32 + l32, kk * 2 + half);
  };
  auto load_init = [&](int t, int s) {
    const float* nl = lds_nl + (t % kNBuf) * C::ROWS;
    // accumulator rows of this lane: (r/4)*8 + half*4 + r%4
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&nl[s * 32 + j * 8 + half * 4]);
      init[4 * j + 0] = v[0];
      init[4 * j + 1] = v[1];
      init[4 * j + 2] = v[2];
      init[4 * j + 3] = v[3];
    }
  };
#pragma unroll
  for (int kk = 0; kk < C::KK; ++kk) load_a(0, 0, kk);
  load_init(0, 0);
  f32x16 pend0 = splat16(kNegInf), pend1 = splat16(kNegInf);
  constexpr int NP = NCOL / 2;  // pairs per sub-tile
  for (int t = 0; t < total; ++t) {
    static_for<C::SUB * NP>([&](auto ic) {
      constexpr int i = decltype(ic)::value, s = i / NP, pr = i % NP;
      constexpr int pp = (pr + NP - 1) % NP;  // pair whose accumulators are pending
      constexpr int NM = 2 * C::KK;
      f32x16 c0, c1;
      MaxTree w0, w1;
      static_for<NM>([&](auto jc) {
        constexpr int j = decltype(jc)::value, kk = j / 2;
        if constexpr (j == 0) c0 = mfma_32x32x16(a[0], b[2 * pr][0], init);
        else if constexpr (j == 1) c1 = mfma_32x32x16(a[0], b[2 * pr + 1][0], init);
        else if constexpr (j % 2 == 0) c0 = mfma_32x32x16(a[kk], b[2 * pr][kk], c0);
        else c1 = mfma_32x32x16(a[kk], b[2 * pr + 1][kk], c1);
        if constexpr (i == 0 && j == 1) {
          // every wave has finished tile t-1: its buffer takes tile t+2, the registers take tile t+3
          __syncthreads();
          if (t + 2 < total) store(t + 2);
          if (t + 3 < total) fetch_next();
        }
        if constexpr (pr == NP - 1 && (j & 1)) {
          // last pair of the sub-tile: refill from the next sub-tile (sub-tile 0 of the next tile after the last)
          if constexpr (s + 1 < C::SUB) {
            load_a(t, s + 1, kk);
            if constexpr (j == 1) load_init(t, s + 1);
          } else {  // past the last tile this reads a stale buffer, harmlessly
            load_a(t + 1, 0, kk);
            if constexpr (j == 1) load_init(t + 1, 0);
          }
        }
        // the 16 v_max3 of the pending pair behind MFMAs 2, 3, ... (its last MFMA has retired by then)
        if constexpr (j >= 2) {
          constexpr int g = j - 2, lo = (16 * g) / (NM - 2), hi = (16 * (g + 1)) / (NM - 2);
          static_for<hi - lo>([&](auto vc) {
            constexpr int v = lo + decltype(vc)::value;
            if constexpr (v < 8) max_step<v>(pend0, w0, runmax[2 * pp]);
            else max_step<v - 8>(pend1, w1, runmax[2 * pp + 1]);
          });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      pend0 = c0;
      pend1 = c1;
    });
  }
  runmax[NCOL - 2] = max16_tree(pend0, runmax[NCOL - 2]);
  runmax[NCOL - 1] = max16_tree(pend1, runmax[NCOL - 1]);
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) {
    const float m = __builtin_fmaxf(runmax[cs], swap_halves(runmax[cs]));
    const float p = __builtin_fminf(__builtin_amdgcn_exp2f(c * m), 1.0f);
    if (half == 0 && kn[cs] < N) {
      float* dst = x + (size_t)(l * H_kv + hs) * N + kn[cs];
      if constexpr (SPLIT) atomicMax(reinterpret_cast<unsigned int*>(dst), __float_as_uint(p));
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
template <int D, int NCOL, bool CAUSAL, bool SPLIT>
__global__ __launch_bounds__(256, 2) void score_colsum_kernel(const uint16_t* __restrict__ q,
                                                               const uint16_t* __restrict__ k_ctx,
                                                               const float* __restrict__ neg_lse,
                                                               float* __restrict__ x, int L_s, int H_q, int G, int N, int N_q,
                                                               float c, float inv_c, int splits) {
  using C = ScoreCfg<D>;
  __shared__ u32x4 lds[kNBuf * C::TILE_U4];
  __shared__ __attribute__((aligned(16))) float lds_nl[kNBuf * C::ROWS];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  constexpr int KB = 128 * NCOL;
  const int H_kv = H_q / G;
  const GroupBlock gb = group_block((N + KB - 1) / KB);  // a group's blocks: its key blocks (they stream the same queries)
  if (gb.group >= L_s * H_kv) return;
  const int l = gb.group / H_kv, hs = gb.group % H_kv;
  const int n0 = gb.item * KB;
  const uint16_t* kc = k_ctx + (size_t)(l * H_kv + hs) * N * D;

  bf16x8 b[NCOL][C::KK];
  int kn[NCOL];
  float colsum[NCOL];
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) {
    kn[cs] = n0 + (wave * NCOL + cs) * 32 + l32;
    const int row = kn[cs] < N ? kn[cs] : N - 1;
#pragma unroll
    for (int kk = 0; kk < C::KK; ++kk)
      b[cs][kk] = as_bf16x8(*reinterpret_cast<const u32x4*>(kc + (size_t)row * D + kk * 16 + half * 8));
    colsum[cs] = 0.0f;
  }

  // tiles are fetched in order: head g = 0..G-1 of the group, query tile qt = 0..nqt-1
  const int nqt = (N_q + C::ROWS - 1) / C::ROWS;
  const int qt_first = CAUSAL ? n0 / C::ROWS : 0;  // KB is a multiple of ROWS
  const int total = G * (nqt - qt_first);
  TileRegs<D> regs;
  LseRegs<SPLIT> nl_reg;
  nl_reg.none();
  int fg = 0, fqt = qt_first;
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
  fetch_next();
  store(0);
  if (total > 1) {
    fetch_next();
    store(1);
  }
  if (total > 2) fetch_next();

  int cqt = qt_first;  // query tile of step t
  for (int t = 0; t < total; ++t) {
    // every wave has finished tile t-1: its buffer takes tile t+2, the registers take tile t+3
    __syncthreads();
    if (t + 2 < total) store(t + 2);
    if (t + 3 < total) fetch_next();
    const u32x4* buf = lds + (t % kNBuf) * C::TILE_U4;
    const float* nl = lds_nl + (t % kNBuf) * C::ROWS;
    const int row0 = cqt * C::ROWS;
    const bool diag = CAUSAL && row0 < n0 + KB - 1;  // some query of the tile lies before some key of the block
    if (++cqt == nqt) cqt = qt_first;
#pragma unroll
    for (int s = 0; s < C::SUB; ++s) {
      bf16x8 a[C::KK];
#pragma unroll
      for (int kk = 0; kk < C::KK; ++kk) a[kk] = frag_read<D>(buf, s * 32 + l32, kk * 2 + half);
      // accumulator rows of this lane: (r/4)*8 + half*4 + r%4
      f32x16 init;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(&nl[s * 32 + j * 8 + half * 4]);
        init[4 * j + 0] = v[0];
        init[4 * j + 1] = v[1];
        init[4 * j + 2] = v[2];
        init[4 * j + 3] = v[3];
      }
#pragma unroll
      for (int cp = 0; cp < NCOL; cp += 2) {
        f32x16 acc[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          acc[e] = init;
#pragma unroll
          for (int kk = 0; kk < C::KK; ++kk) acc[e] = mfma_32x32x16(a[kk], b[cp + e][kk], acc[e]);
        }
        if (diag) {
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int i = row0 + s * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
              acc[e][r] = i >= kn[cp + e] ? acc[e][r] : kNegInf;
            }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          float s0 = __builtin_amdgcn_exp2f(acc[e][0] * c), s1 = __builtin_amdgcn_exp2f(acc[e][1] * c);
          float s2 = __builtin_amdgcn_exp2f(acc[e][2] * c), s3 = __builtin_amdgcn_exp2f(acc[e][3] * c);
#pragma unroll
          for (int r = 4; r < 16; r += 4) {
            s0 += __builtin_amdgcn_exp2f(acc[e][r + 0] * c);
            s1 += __builtin_amdgcn_exp2f(acc[e][r + 1] * c);
            s2 += __builtin_amdgcn_exp2f(acc[e][r + 2] * c);
            s3 += __builtin_amdgcn_exp2f(acc[e][r + 3] * c);
          }
          colsum[cp + e] += (s0 + s1) + (s2 + s3);
        }
      }
    }
  }
#pragma unroll
  for (int cs = 0; cs < NCOL; ++cs) {
    const float tot = colsum[cs] + swap_halves(colsum[cs]);
    if (half == 0 && kn[cs] < N) x[(size_t)(l * H_kv + hs) * N + kn[cs]] = tot;
  }
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

hipError_t launch_score_colsum(const uint16_t* q, const uint16_t* k_ctx, const float* neg_lse, int splits, float* x, int L_s,
                               int H_q, int H_kv, int d, int64_t N, int64_t N_q, bool causal, hipStream_t stream) {
  const int G = H_q / H_kv;
  const float c = 1.4426950408889634f / sqrtf((float)d), inv_c = 1.0f / c;
  constexpr int NCOL = 2;
  if (causal && N != N_q) return hipErrorInvalidValue;
  const unsigned grid = group_grid((int64_t)L_s * H_kv, (N + 128 * NCOL - 1) / (128 * NCOL));
  if (grid == 0) return hipErrorInvalidValue;
  auto go = [&](auto dc, auto cc, auto sc) {
    score_colsum_kernel<decltype(dc)::value, NCOL, decltype(cc)::value, decltype(sc)::value>
        <<<grid, 256, 0, stream>>>(q, k_ctx, neg_lse, x, L_s, H_q, G, (int)N, (int)N_q, c, inv_c, splits);
  };
  auto pick = [&](auto dc) {
    if (causal && splits > 1) go(dc, std::true_type{}, std::true_type{});
    else if (causal) go(dc, std::true_type{}, std::false_type{});
    else if (splits > 1) go(dc, std::false_type{}, std::true_type{});
    else go(dc, std::false_type{}, std::false_type{});
  };
  if (d == 64) pick(std::integral_constant<int, 64>{});
  else pick(std::integral_constant<int, 128>{});
  return hipGetLastError();
}

hipError_t launch_score_colmax(const uint16_t* q, const uint16_t* k_ctx, const float* neg_lse, int splits, float* x, int L_s,
                               int H_q, int H_kv, int d, int64_t N, int64_t N_q, hipStream_t stream) {
  const int G = H_q / H_kv;
  const float c = 1.4426950408889634f / sqrtf((float)d), inv_c = 1.0f / c;
  // d = 64: two workgroups per CU.  d = 128: one (the resident keys of 4 column sub-tiles alone take 128 registers): a wave
  // has the SIMD's whole register file, and the pinned issue order keeps the matrix pipe fed without a second wave
  constexpr int NCOL = 4;
  const int64_t key_blocks = (N + 128 * NCOL - 1) / (128 * NCOL), q_tiles = G * ((N_q + 8192 / d - 1) / (8192 / d));
  int64_t q_splits = 1;
  if (splits > 1) {
    // as many parts of the query tiles as fill the chip, two tiles or more each (the first tile of a part waits for memory)
    q_splits = (d == 64 ? 512 : 256) / (key_blocks * L_s * H_kv);
    q_splits = q_splits < q_tiles / 2 ? q_splits : q_tiles / 2;
    q_splits = q_splits < 1 ? 1 : q_splits;
  }
  const unsigned grid = group_grid((int64_t)L_s * H_kv, key_blocks * q_splits);
  if (grid == 0) return hipErrorInvalidValue;
  auto go = [&](auto dc, auto sc) {
    score_colmax_kernel<decltype(dc)::value, NCOL, decltype(sc)::value>
        <<<grid, 256, 0, stream>>>(q, k_ctx, neg_lse, x, L_s, H_q, G, (int)N, (int)N_q, c, inv_c, splits, (int)q_splits);
  };
  if (d == 64 && splits > 1) go(std::integral_constant<int, 64>{}, std::true_type{});
  else if (d == 64) go(std::integral_constant<int, 64>{}, std::false_type{});
  else if (splits > 1) go(std::integral_constant<int, 128>{}, std::true_type{});
  else go(std::integral_constant<int, 128>{}, std::false_type{});
  return hipGetLastError();
}

}  // namespace pkv
