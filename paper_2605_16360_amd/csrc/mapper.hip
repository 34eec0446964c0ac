// HybridAxialMapper forward (paper Sec. 4.1) for a batch of proxy layers at a time:
//   stage 1  conv stem            stem_conv1_kernel (fp32 ALU) + conv 2 as an fp16 MFMA GEMM whose A rows
//                                 are overlapping 3-token spans of the padded conv-1 output
//   stage 2  time-axis encoder    per encoder layer: encoder_block_kernel (mapper_block.hip; everything beside the attention, up to the
//                                 next layer's q, k and v) -> window attention; the sliding windows of all proxy layers of
//                                 the batch lie on one axis of rows
//            overlap averaging    overlap_avg_kernel
//   stage 3  head-axis attention  K/V projection GEMM (inner products with queries / output weights in its epilogue)
//                                  + stage3_kernel (softmax over the slots per token and head, fp32 ALU)
// Matrix products take IEEE half (fp16) operands and accumulate in fp32, the two here on v_mfma_f32_32x32x16_f16, the encoder
// and its attention on v_mfma_f32_16x16x32_f16, which draws less power per flop where the chip's power sets its clock; the
// residual stream, normalisation, softmax and GELU are fp32.
#include "common.hpp"
#include "context.hpp"
#include "kernels.hpp"
#include "mapper.hpp"

namespace pkv {
namespace {

// partial maxima of |x| of every layer's scores (n per layer), as bits; grid (kRangeWords, layers)
__global__ __launch_bounds__(1024) void absmax_kernel(const float* __restrict__ x, int64_t n, LayerBatch lb,
                                                      uint32_t* __restrict__ words) {
  __shared__ uint32_t part[16];
  x += (size_t)lb.ls[blockIdx.y] * n;
  uint32_t m = 0;
  for (int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x; i < n; i += (int64_t)kRangeWords * 1024) {
    const uint32_t a = __float_as_uint(x[i]) & 0x7fffffffu;
    m = a > m ? a : m;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t o = __shfl_xor(m, off, 64);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < 16; ++w) m = part[w] > m ? part[w] : m;
    words[blockIdx.y * kRangeWords + blockIdx.x] = m;
  }
}

// ------------------------------------------------------------------------------------------
// stage 1, first convolution: h1[t+1, c] = half(2^-s * GELU(scale[c] * sum_{h,tap} w[c,h,tap] * x[h, t+tap-1] + shift[c]))
// rows 0 and N+1 of h1 are zero (the padding of the second convolution).
// grid (ceil(N / tok), layers), 256 threads; thread owns channels tid, tid+256, ...  tok <= 64 tokens per workgroup: a
// workgroup's tokens are a serial chain, so short inputs take fewer of them (512 tokens of one layer: 23.6 us with 64
// tokens per workgroup, eight workgroups on 256 CUs, 8.3 with 16 and 5.0 with 4; from 8192 tokens on 16 give every CU two).
// The weights lie [H_s * 3][c_mid], so a wave's load is 256 bytes in one piece; with a channel's side by side each touched 48 lines, and
// eight layers of 600 tokens, 1200 workgroups of four tokens, took 22.1 us instead of 11.0, of 1500 21.0 / 14.4.
// ------------------------------------------------------------------------------------------
constexpr int kStemTok = 64;
constexpr int kMaxHs = 16;

__global__ __launch_bounds__(256) void stem_conv1_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                          const float* __restrict__ scale,
                                                          const float* __restrict__ shift,
                                                          const uint32_t* __restrict__ range, float cw, float cs, LayerBatch lb,
                                                          uint16_t* __restrict__ h1, int H_s, int N, int c_mid, int tok) {
  __shared__ float xs[kMaxHs][kStemTok + 2];
  const float down = exp2_int(-stem_exponent(range + blockIdx.y * kRangeWords, cw, cs));
  x += (size_t)lb.ls[blockIdx.y] * H_s * N;
  h1 += (size_t)blockIdx.y * (N + 2) * c_mid;
  const int t0 = blockIdx.x * tok;
  for (int i = threadIdx.x; i < H_s * (tok + 2); i += 256) {
    const int h = i / (tok + 2), tt = i % (tok + 2);
    const int t = t0 + tt - 1;
    xs[h][tt] = (t >= 0 && t < N) ? x[(size_t)h * N + t] : 0.0f;
  }
  __syncthreads();
  for (int c = threadIdx.x; c < c_mid; c += 256) {
    float wr[kMaxHs * 3];
#pragma unroll
    for (int i = 0; i < kMaxHs * 3; ++i) wr[i] = (i < H_s * 3) ? w[i * c_mid + c] : 0.0f;
    const float sc = scale[c], sh = shift[c];
    for (int tt = 0; tt < tok && t0 + tt < N; ++tt) {
      float acc = 0.0f;
#pragma unroll
      for (int h = 0; h < kMaxHs; ++h) {
        if (h < H_s) {
          acc = __builtin_fmaf(wr[h * 3 + 0], xs[h][tt + 0], acc);
          acc = __builtin_fmaf(wr[h * 3 + 1], xs[h][tt + 1], acc);
          acc = __builtin_fmaf(wr[h * 3 + 2], xs[h][tt + 2], acc);
        }
      }
      h1[(size_t)(t0 + tt + 1) * c_mid + c] = to_h(gelu_erf(__builtin_fmaf(acc, sc, sh)) * down);
    }
    if (blockIdx.x == 0) h1[c] = 0;
    if (blockIdx.x == gridDim.x - 1) h1[(size_t)(N + 1) * c_mid + c] = 0;
  }
}

// ------------------------------------------------------------------------------------------
// fp16 GEMM  C[M, Nn] = A[M, K] * W[Nn, K]^T  (+ epilogue), fp32 accumulation.
// A rows start lda elements apart (lda < K gives the overlapping rows of the second convolution).
//
// The stage-3 projection where it has many tiles (where it has few, and for the second convolution: gemm_f16_tile_kernel).
// Persistent kernel, one 512-thread workgroup per CU.  Block tile BM (rows of A) x BN (rows of W) = 256 x 256, K step 64 (full
// 128-byte lines per row), 8 waves, each 64 x 128 = 2 x 4 MFMA tiles.  A tile of this size needs 1 byte from L2 per 128 flop.
//
// The A rows go on the MFMA M axis and the W rows on the N axis, so a lane owns output COLUMNS.  The
// W rows of a wave's 128-column block are staged in the order n = 4*l + jn (l = lane & 31, jn = MFMA
// tile), so a lane holds four adjacent columns in its four tiles and every store instruction writes
// whole 512-byte row segments, 16 bytes per lane.  Rows past a layer's last are not written.
//
// The K steps of all tiles of a workgroup form one stream: two LDS stages (64 KB each) and ONE barrier
// per step.  A step is four phases of 8 MFMAs; the fragments of phase kk+1 are read from LDS between
// the MFMAs of phase kk (phase 3 reads phase 0 of the next step, behind the barrier), step s+1 goes
// from registers to LDS during phase 2 and each register is refilled with its part of step s+2 right
// behind that -- across tile boundaries, so the next tile's loads are in flight during an epilogue.
// The issue order is written out and pinned with scheduling barriers.
//
// Tile order: blocks are dealt round-robin to the 8 XCDs by the hardware, so XCD x = block % 8 takes the
// row tiles x, x+8, ... and its workgroups take that list's (row tile, column tile) pairs round-robin:
// the Nn / BN column tiles of one row tile run at the same time on one XCD and share its L2 copy of
// the A rows.
// The M axis holds the rows of all layers of a batch: layer b owns rows [b * row_stride, b * row_stride + rows), its A
// rows start a_layer elements after those of layer b - 1, and row_stride is a multiple of 256, so a tile never spans two
// layers; tile rows past a layer's last one re-read that row.
// K % 64 == 0, Nn % BN == 0.
// ------------------------------------------------------------------------------------------
enum Epilogue {
  kEpiGeluPeWin,      // z = GELU(acc * (p0[n] * 2^s) + p1[n]), s from `range`, of token m goes, plus the positional row of its place, into the
                      // row of every window that holds the token: out_f32, in blocks as block_x4 lays them (second stem convolution ->
                      // stage-2 input)
  kEpiStage3          // columns = stage-3 key and value slots of 64: per token and slot the inner products of
                      // acc + p0 with the learned queries (p1, n_head of them, times 1/8) or with the output weights (g)
};

struct EpiArgs {
  const float* p0;
  const float* p1;
  const uint32_t* range;  // kEpiGeluPeWin: partial maxima per layer, cw and cs as in stem_exponent
  float cw, cs;
  const float* g;
  float* out_f32;
  int ldc;  // kEpiStage3: elements between output rows
  int out_stride;  // kEpiGeluPeWin: output rows between layers
  const float* pe;  // kEpiGeluPeWin: positional table [kWin, d_time]
  int n_win;        // kEpiGeluPeWin: windows per layer
  int n_slot, n_head;  // kEpiStage3: slots H_s (keys in columns [0, 64 H_s), values in [64 H_s, 128 H_s)) and queries H_l
};

constexpr int kGemmTile = 256, kGemmBK = 64;

// Sum of v[0..15] over the 16 lanes that share the upper bits of the lane number, sixteen sums at once: in every step a lane
// keeps the half of its values that its own lane bit selects, hands the other half to the partner and adds what it
// receives; afterwards lane j (lane & 15) holds the sum of v[j].  15 exchanges.
__device__ __forceinline__ float reduce16_over_16_lanes(float (&v)[16], int lane) {
  static_for<4>([&](auto sc) {
    constexpr int step = decltype(sc)::value, n = 8 >> step, mask = 8 >> step;
    const bool up = (lane & mask) != 0;
#pragma unroll
    for (int j = 0; j < n; ++j) {
      const float send = up ? v[j] : v[j + n];
      const float keep = up ? v[j + n] : v[j];
      v[j] = keep + __shfl_xor(send, mask, 64);
    }
  });
  return v[0];
}

// What follows a wave's 32 MI x 128 accumulators: rows m0 .. of the batch, r0 .. of their layer, columns c0 ..
template <int EPI, int MI>
__device__ __forceinline__ void gemm_epilogue(const f32x16 (&acc)[MI][4], const f32x4 p0, const f32x4 p1, const EpiArgs& ep, int m0, int r0,
                                              int layer, int rows, int c0, int lane) {
  // a lane holds columns n .. n+3; register r of tile (i, jn) holds row i*32 + half*4 + (r/4)*8 + r%4
  const int half = lane >> 5, l32 = lane & 31, n = c0 + 4 * l32;
  if constexpr (EPI == kEpiStage3) {
    // The 64 columns of a slot sit in 16 lanes (four columns each).  Per 32-row block: the lane's share of every row's
    // inner product with one coefficient vector, sixteen rows reduced over the 16 lanes at once, lane j keeps row j of
    // the sixteen that its half-wave holds.  Key slots take the n_head queries in turn, value slots the output weights.
    const int col = c0 + (l32 >> 4) * 64;  // first column of the lane group's slot
    const int slot = col >> 6, e0 = (l32 & 15) * 4;
    const bool is_k = slot < ep.n_slot, is_v = !is_k && slot < 2 * ep.n_slot;
    const int sv = is_k ? slot : slot - ep.n_slot;
    const int j16 = l32 & 15;
    const int n_pass = ep.n_head;  // uniform; value slots use pass 0 only
    const float* cf = is_k ? ep.p1 + e0 : ep.g + e0;
    f32x4 next = *reinterpret_cast<const f32x4*>(cf);  // coefficients of pass h, loaded a pass ahead
    for (int h = 0; h < n_pass; ++h) {
      const f32x4 c4 = next;
      next = *reinterpret_cast<const f32x4*>(cf + (is_k && h + 1 < n_pass ? (size_t)(h + 1) * 64 : 0));
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int row = m0 + i * 32 + (j16 >> 2) * 8 + half * 4 + (j16 & 3);  // the row this lane ends up with
        float* orow = ep.out_f32 + (size_t)row * ep.ldc;
        float part[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)
          part[r] = (acc[i][0][r] + p0[0]) * c4[0] + (acc[i][1][r] + p0[1]) * c4[1] + (acc[i][2][r] + p0[2]) * c4[2] +
                    (acc[i][3][r] + p0[3]) * c4[3];
        const float tot = reduce16_over_16_lanes(part, l32);
        if (row - m0 + r0 < rows) {
          if (is_k) orow[h * ep.n_slot + sv] = tot * 0.125f;
          else if (is_v && h == 0) orow[ep.n_head * ep.n_slot + sv] = tot;
        }
      }
    }
  } else {
    f32x4* xo = reinterpret_cast<f32x4*>(ep.out_f32);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      // Token t sits at place t - 1024 k of window k = min(t / 1024, n_win - 1) and, if that window is not the first and the token lies in
      // its first half, at place + 1024 of the window before: the same window for all 32 tokens, which lie in one 32nd of 1024.
      // The 32 places lie in the table whether the tokens are there or not.
      const int ti = r0 + i * 32, tl = half * 4;
      if (ti >= rows) break;
      const int kq = ti / kStride, k1 = kq < ep.n_win ? kq : ep.n_win - 1, place = ti - k1 * kStride + tl;
      const float* pe = ep.pe + (size_t)place * kDT + n;
      const int64_t row = (int64_t)layer * ep.out_stride + (int64_t)k1 * kWin + place;
      const bool second = k1 >= 1 && kq == k1;
      // Eight rows at a time, their positional rows loaded before the first GELU: a load behind each GELU would be waited for by itself.
#pragma unroll
      for (int g = 0; g < 16; g += 8) {
        f32x4 e0[8], e1[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) e0[r] = *reinterpret_cast<const f32x4*>(pe + (((g + r) >> 2) * 8 + (r & 3)) * kDT);
        if (second) {
#pragma unroll
          for (int r = 0; r < 8; ++r) e1[r] = *reinterpret_cast<const f32x4*>(pe + (kStride + ((g + r) >> 2) * 8 + (r & 3)) * kDT);
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const int t = ((g + r) >> 2) * 8 + (r & 3);
          f32x4 v = {acc[i][0][g + r], acc[i][1][g + r], acc[i][2][g + r], acc[i][3][g + r]};
#pragma unroll
          for (int c = 0; c < 4; ++c) v[c] = gelu_erf(__builtin_fmaf(v[c], p0[c], p1[c]));
          if (ti + tl + t < rows) {
            xo[block_x4(row + t, n)] = v + e0[r];
            if (second) xo[block_x4(row + t - (kWin - kStride), n)] = v + e1[r];
          }
        }
      }
    }
  }
}

__global__ __launch_bounds__(512, 1) void gemm_f16_kernel(const uint16_t* __restrict__ A, int lda, int64_t a_layer,
                                                          const uint16_t* __restrict__ W, int M, int rows, int row_stride,
                                                          int Nn, int K, EpiArgs ep) {
  constexpr int BM = kGemmTile, BN = kGemmTile, WM = BM / 64, WN = 8 / WM;  // waves along M and N
  constexpr int NA = BM / 64, NS = (BM + BN) / 64;  // 64-row parts of a stage: A parts, then W parts
  constexpr int kStageU4 = (BM + BN) * (kGemmBK / 8);  // 16-byte units per stage
  static_assert(WM * WN == 8 && BN / WN == 128, "a wave computes 64 x 128");
  extern __shared__ u32x4 lds[];  // 2 stages
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wm = wave / WN, wn = wave % WN;
  const int n_tiles = Nn / BN;
  const int nk = K / kGemmBK;
  const int xcd = blockIdx.x % kXcds, wg = blockIdx.x / kXcds, wg_per_xcd = gridDim.x / kXcds;
  // tile `it` of this workgroup: entry it * wg_per_xcd + wg of the XCD's list
  auto tile_of = [&](int it, int& m0, int& n0) {
    const int u = it * wg_per_xcd + wg;
    m0 = ((u / n_tiles) * kXcds + xcd) * BM;
    n0 = (u % n_tiles) * BN;
    return m0 < M;
  };
  int my_tiles = 0;
  {
    int a, b;
    while (tile_of(my_tiles, a, b)) ++my_tiles;
  }
  const int total = my_tiles * nk;
  if (total == 0) return;

  // staging: thread t moves chunk t % 8 of LDS rows t / 8 + 64 * i (i < NA: A rows, i >= NA: W rows).
  // LDS row wl = 64 (i - NA) + t / 8 of the W part holds W row n0 + 128 (wl / 128) + 4 (wl % 32) + (wl % 128) / 32.
  const int srow = tid >> 3, sch = tid & 7;
  const int sslot = srow * 8 + (sch ^ swz8(srow));  // swz8(srow + 64 * i) == swz8(srow)
  u32x4 rg[NS];
  int f_m0 = 0, f_n0 = 0, f_k = 0, f_it = 0;  // position of the next step to fetch
  const uint16_t* f_a = A;                    // first A row of the layer that tile f_it lies in; f_m0 counts from there
  auto fetch_tile = [&](int it) {
    tile_of(it, f_m0, f_n0);
    const int layer = f_m0 / row_stride;
    f_m0 -= layer * row_stride;
    f_a = A + (size_t)layer * a_layer;
  };
  fetch_tile(0);
  auto fetch_one = [&](int i) {
    const int k0 = f_k * kGemmBK + sch * 8;
    if (i < NA) {
      int m = f_m0 + srow + 64 * i;
      m = m < rows ? m : rows - 1;
      rg[i] = *reinterpret_cast<const u32x4*>(f_a + (size_t)m * lda + k0);
    } else {
      const int wl = srow + 64 * (i - NA);
      const int n = f_n0 + (wl & ~127) + 4 * (wl & 31) + ((wl & 127) >> 5);
      rg[i] = *reinterpret_cast<const u32x4*>(W + (size_t)n * K + k0);
    }
  };
  // moves on to the following step; past the end it stays on the last step (re-reads valid memory)
  auto fetch_advance = [&]() {
    if (++f_k == nk) {
      if (f_it + 1 < my_tiles) {
        f_k = 0;
        ++f_it;
        fetch_tile(f_it);
      } else {
        f_k = nk - 1;
      }
    }
  };

  f32x16 acc[2][4];
  auto zero_acc = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int jn = 0; jn < 4; ++jn) acc[i][jn] = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  };
  zero_acc();
  // bias of the current tile's columns n .. n+3, loaded when the tile starts: a load inside
  // the epilogue would have to wait for the prefetch of the next step as well
  f32x4 p0;
  auto load_bias = [&](int it) {
    int m0, n0;
    tile_of(it < my_tiles ? it : my_tiles - 1, m0, n0);
    const int n = n0 + wn * 128 + 4 * l32;
    p0 = *reinterpret_cast<const f32x4*>(ep.p0 + n);
  };
  load_bias(0);

  // prologue: step 0 to LDS, step 1 in registers, fragments of (step 0, phase 0) in registers
#pragma unroll
  for (int i = 0; i < NS; ++i) fetch_one(i);
  fetch_advance();
#pragma unroll
  for (int i = 0; i < NS; ++i) lds[sslot + 64 * 8 * i] = rg[i];
#pragma unroll
  for (int i = 0; i < NS; ++i) fetch_one(i);
  fetch_advance();
  __syncthreads();
  const int fsw = swz8(l32);  // all fragment rows of this lane are l32 plus a multiple of 32
  const int xrow = (wm * 64 + l32) * 8, wrow = (BM + wn * 128 + l32) * 8;
  f16x8 fx[2][2], fw[2][4];
  auto read_frag = [&](const u32x4* st, int kk, int set, int which) {
    const int slot = (kk * 2 + half) ^ fsw;
    if (which < 2) fx[set][which] = as_f16x8(st[xrow + which * 32 * 8 + slot]);
    else fw[set][which - 2] = as_f16x8(st[wrow + (which - 2) * 32 * 8 + slot]);
  };
#pragma unroll
  for (int wh = 0; wh < 6; ++wh) read_frag(lds, 0, 0, wh);

  for (int s = 0; s < total; ++s) {
    u32x4* st = lds + (s & 1) * kStageU4;
    u32x4* st_next = lds + ((s + 1) & 1) * kStageU4;
    static_for<4>([&](auto kc) {
      constexpr int kk = decltype(kc)::value, cur = kk & 1, nxt = cur ^ 1;
      if constexpr (kk == 3) {
        // every wave has read the last fragments of this step and written its part of step s+1
        __syncthreads();
      }
      static_for<8>([&](auto jc) {
        constexpr int j = decltype(jc)::value, i = j >> 2, jn = j & 3;
        acc[i][jn] = mfma_f16_32x32x16(fx[cur][i], fw[cur][jn], acc[i][jn]);
        if constexpr (j < 6) {
          if constexpr (kk < 3) read_frag(st, kk + 1, nxt, j);
          else read_frag(st_next, 0, nxt, j);
        }
        if constexpr (kk == 2) {
          // the register is refilled as soon as it is free: a whole step lies between a load and its use
          st_next[sslot + 64 * 8 * j] = rg[j];
          fetch_one(j);
          if constexpr (j + 8 < NS) {
            st_next[sslot + 64 * 8 * (j + 8)] = rg[j + 8];
            fetch_one(j + 8);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    fetch_advance();
    if (s % nk != nk - 1) continue;

    int m0, n0;
    tile_of(s / nk, m0, n0);
    const int layer = m0 / row_stride;
    gemm_epilogue<kEpiStage3, 2>(acc, p0, p0, ep, m0 + wm * 64, m0 - layer * row_stride + wm * 64, layer, rows, n0 + wn * 128, lane);
    zero_acc();
    load_bias(s / nk + 1);
  }
}

// ------------------------------------------------------------------------------------------
// The same product, sum for sum, in tiles of 128 x 128: the second convolution, and the projection where it has few tiles (kTileProducts).
// 256 threads, a wave computes 32 x 128; two stages of 32 KB, so two workgroups share a CU and one's products run beside the other's epilogue,
// which in the convolution (a GELU per element, two stores) takes longer than its 12 K steps: with one 256 x 256 tile per CU
// nothing stood beside it.  One layer of 3500 tokens, 28 large tiles or 112 of these: 52.5 us and 21.3 (25.6 with a
// positional row loaded behind each GELU); eight layers of 600 tokens 40.8 / 19.9, one of 8192 beside another lane 134 / 123.  Loads write LDS
// directly, a stage as the fragments are read (row r's unit u at place u ^ swz8(r)).  Four stages and one workgroup per CU are up to
// 4 % of the mapper slower.
// XCD x = block % 8 takes the row tiles x, x + 8, ..., a row's column tiles one after another.  layer_tiles row tiles per layer, row_tiles
// in all; a layer's last tile re-reads its last row.
// ------------------------------------------------------------------------------------------
template <int EPI>
__global__ __launch_bounds__(256, 2) void gemm_f16_tile_kernel(const uint16_t* __restrict__ A, int lda, int64_t a_layer,
                                                                const uint16_t* __restrict__ W, int row_tiles, int layer_tiles,
                                                                int rows, int row_stride, int n_tiles, int K, EpiArgs ep) {
  constexpr int kStageU4 = 256 * (kGemmBK / 8);
  __shared__ u32x4 lds[2 * kStageU4];  // a stage: 128 rows of A, then 128 of W, in the order n = 4 * l + jn
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int bj = blockIdx.x / kXcds, rt = (bj / n_tiles) * kXcds + blockIdx.x % kXcds, n0 = (bj % n_tiles) * 128;
  if (rt >= row_tiles) return;
  const int layer = rt / layer_tiles, r0 = (rt % layer_tiles) * 128;
  const int nk = K / kGemmBK;
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  const int srow = tid >> 3, sch = ((tid & 7) ^ swz8(srow)) * 8;
  const uint16_t *pa[4], *pw = W + (size_t)(n0 + 4 * srow) * K + sch;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int m = r0 + srow + 32 * i;
    m = m < rows ? m : rows - 1;
    pa[i] = A + (size_t)layer * a_layer + (size_t)m * lda + sch;
  }
  // past the last step that one is copied again, so that every step has the same loads behind it
  auto fetch = [&](int s, int stage) __attribute__((always_inline)) {
    const int k0 = (s < nk ? s : nk - 1) * kGemmBK;
    u32x4* st = lds + stage * kStageU4 + wave * 64;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_global_load_lds((gptr_t)(pa[i] + k0), (lptr_t)(st + i * 256), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((gptr_t)(pw + (size_t)i * K + k0), (lptr_t)(st + (4 + i) * 256), 16, 0, 0);
    }
  };
  const int n = n0 + 4 * l32;
  f32x4 p0 = *reinterpret_cast<const f32x4*>(ep.p0 + n), p1 = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (EPI == kEpiGeluPeWin) {
    p0 *= exp2_int(stem_exponent(ep.range + layer * kRangeWords, ep.cw, ep.cs));
    p1 = *reinterpret_cast<const f32x4*>(ep.p1 + n);
  }
  f32x16 acc[1][4];
#pragma unroll
  for (int jn = 0; jn < 4; ++jn) acc[0][jn] = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  fetch(0, 0);
  fetch(1, 1);
  __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt(8): step 0
  __syncthreads();
  const int fsw = swz8(l32), xrow = (wave * 32 + l32) * 8, wrow = (128 + l32) * 8;
  f16x8 fx[2], fw[2][4];
  auto read_frags = [&](const u32x4* st, int kk, int set) __attribute__((always_inline)) {
    const int slot = (kk * 2 + half) ^ fsw;
    fx[set] = as_f16x8(st[xrow + slot]);
#pragma unroll
    for (int j = 0; j < 4; ++j) fw[set][j] = as_f16x8(st[wrow + j * 32 * 8 + slot]);
  };
  read_frags(lds, 0, 0);
  for (int s = 0; s < nk; ++s) {
    const u32x4 *st = lds + (s & 1) * kStageU4, *st_next = lds + ((s + 1) & 1) * kStageU4;
    static_for<4>([&](auto kc) {
      constexpr int kk = decltype(kc)::value, cur = kk & 1, nxt = cur ^ 1;
      if constexpr (kk == 3) {
        // this wave's part of step s + 1 has landed; behind the barrier everyone's has, and every wave has read the last of step s
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();
        fetch(s + 2, s & 1);
        read_frags(st_next, 0, nxt);
      } else {
        read_frags(st, kk + 1, nxt);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[0][j] = mfma_f16_32x32x16(fx[cur], fw[cur][j], acc[0][j]);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing of this workgroup writes LDS that anyone may have by then
  gemm_epilogue<EPI, 1>(acc, p0, p1, ep, layer * row_stride + r0 + wave * 32, r0 + wave * 32, layer, rows, n0, lane);
}

// ------------------------------------------------------------------------------------------
// Window attention (8 heads x 64, full bidirectional attention inside each window).
// qkv [block of 128 rows][head][q, k, v][16 KB] as encoder_block_kernel leaves it: MFMA fragments of 1 KB, a lane's 16 bytes each.  q and k:
// [16 rows][32 of d]; v: [32 keys][16 of d].  ao: [block][16 rows][32 columns], the next product's fragments.
// Computes S^T = K Q^T so that a lane owns one query column; P^T then feeds the second MFMA as its
// B operand straight from the accumulator registers, with V^T fragments as the A operand.
// 256 threads; a workgroup owns 64 QT queries of one (window, head), a wave 16 QT of them (QT 16-column
// sub-tiles: four, or two, narrow_attention_pays); keys stream in tiles of 64, copied as they lie, by loads that write LDS, into four LDS stages (K, then V, 8 KB
// each) with one barrier per tile: while tile t is computed, tile t+1 lies there and t+2 and t+3 are on their way.
// A column's reference is the largest logit of its first 64 keys, raised in any later tile whose largest exceeds it by more than 2^8, so a
// tile costs the same wherever the sharp keys lie.  (Left out of the later tiles, with a second pass over the keys where a row sum
// overflows half, the maxima save up to 1 %: 16 layers of 20 000 tokens 35 766 us and 36 114 here, of 8192 13 768 and 13 551, 28 of 1500
// 2401 and 2404; but logits five times as wide, beyond that in every workgroup, then take 51 179, 19 260 and 3149 us, here
// 36 843, 14 122 and 2476.)
// Layer b of the batch owns rows [b * Tp, b * Tp + T); its windows start every 2048 rows.  What the 64 rows of a layer's last row hold beyond
// it is finite, and keys there are masked; rows behind are not read as keys, and queries there are computed and dropped.
// Block -> work mapping: blocks are dealt round-robin to the 8 XCDs, so with n_qb workgroups per window block
// b takes q-block (b / 8) % n_qb of item (b / 8 / n_qb) * 8 + b % 8: the q-blocks of one (window, head) run on one XCD
// and share its L2 copy of that head's K and V.
// ------------------------------------------------------------------------------------------
template <int QT>
__global__ __launch_bounds__(256, 2) void window_attention_kernel(const u32x4* __restrict__ qkv,
                                                                   u32x4* __restrict__ ao, int T, int Tp, int n_win, int n_qb) {
  __shared__ u32x4 lds[4 * 1024];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, quad = lane >> 4;
  const int bj = blockIdx.x >> 3, item = (bj / n_qb) * kXcds + (blockIdx.x & 7);
  const int wg = item / kHeads, hd = item % kHeads;  // wg: window of the batch
  const int layer = wg / n_win, wk = wg % n_win;
  const size_t blk0 = ((size_t)layer * Tp + (size_t)wk * kWin) / kBlk;  // the window's first block of rows
  const int len = (wk < n_win - 1) ? kWin : T - wk * kWin;
  const int i0 = (bj % n_qb) * (64 * QT);
  if (i0 >= len) return;
  constexpr float c = 1.4426950408889634f * 0.125f;  // log2(e) / sqrt(64)

  const u32x4* hbase = qkv + (blk0 * kHeads + hd) * 3 * 1024;
  constexpr size_t kBlkStride = kHeads * 3 * 1024;
  const int q0 = (i0 >> 4) + wave * QT;  // the wave's first tile of 16 queries; all of them lie in one block
  const u32x4* qb = hbase + (size_t)(q0 >> 3) * kBlkStride + (q0 & 7) * 2 * 64 + lane;
  f16x8 bq[QT][2];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) bq[qt][kk] = as_f16x8(qb[(qt * 2 + kk) * 64]);
  f32x4 o[4][QT];  // [16 of d][query sub-tile]
  // Row sums: one more product, ones times P^T, whose sixteen rows are all the sum.  (Two probabilities per v_dot2 took half as many vector
  // instructions as the exponentials.)  It takes the probabilities as the second product sees them, rounded to half.
  f32x4 ls[QT];
  const f16x8 ones = {(_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f};
  float m_run[QT], beyond[QT];  // reference, times c; the logit that raises it

  const int n_tiles = (len + 63) / 64;
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  // past the last tile the last one is copied again, so that every tile has the same number of loads behind it
  auto fetch = [&](int t, int stage) {
    const int tc = t < n_tiles ? t : n_tiles - 1;
    const u32x4* kb = hbase + (size_t)(tc >> 1) * kBlkStride + 1024 + (tc & 1) * 512 + wave * 64 + lane;
    u32x4* st = lds + stage * 1024 + wave * 64;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __builtin_amdgcn_global_load_lds((gptr_t)(kb + i * 256), (lptr_t)(st + i * 256), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((gptr_t)(kb + 1024 + i * 256), (lptr_t)(st + 512 + i * 256), 16, 0, 0);
    }
  };
  // LDS reads run ahead of their use: the first half of tile t+1's K fragments is read in the tail of tile t, the other half and
  // the first V fragments while the first products run.
  f16x8 fa[2][2], fb[2][2], fv[4];
  auto read_k = [&](const u32x4* st, int kt, f16x8 (&fk)[2][2]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) fk[i >> 1][i & 1] = as_f16x8(st[(kt * 2 + i) * 64]);
  };
  // one tile; `cut`: the keys end in it
  auto tile = [&](int t, auto cut) __attribute__((always_inline)) {
    // this wave's part of tile t+1 has landed (the four loads of tile t+2 may be outstanding); behind the barrier everyone's has, and
    // every wave has finished tile t-1, whose stage takes tile t+3
    __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4)
    __syncthreads();
    fetch(t + 3, (t + 3) & 3);
    const u32x4* st = lds + (t & 3) * 1024 + lane;
    const int j0 = t * 64;

    // S^T tiles: s[kt][qt] = K[kt] Q[qt]^T, 16 keys each
    f32x4 s[4][QT];
    read_k(st, 2, fb);
#pragma unroll
    for (int d = 0; d < 4; ++d) fv[d] = as_f16x8(st[512 + d * 64]);
    auto logits = [&](int kt, const f16x8 (&fk)[2]) {
#pragma unroll
      for (int q = 0; q < QT; ++q) s[kt][q] = mfma_f16_16x16x32(fk[0], bq[q][0], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
      for (int q = QT - 1; q >= 0; --q) s[kt][q] = mfma_f16_16x16x32(fk[1], bq[q][1], s[kt][q]);
    };
    logits(0, fa[0]);
    logits(1, fa[1]);
    __builtin_amdgcn_sched_barrier(0);
    logits(2, fb[0]);
    logits(3, fb[1]);
    if constexpr (decltype(cut)::value) {
      const int lim = len - j0 - quad * 4;  // element i of tile kt is key j0 + kt*16 + quad*4 + i
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[kt][qt][i] = kt * 16 + i < lim ? s[kt][qt][i] : kNegInf;
    }
    // the largest logits, or what they have to exceed: of the first 32 keys while the products of the others are on their way
    float tmax[QT];
    bool raise = false;
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      tmax[qt] = max3f(beyond[qt], s[0][qt][0], s[0][qt][1]);
      tmax[qt] = max3f(tmax[qt], s[0][qt][2], s[0][qt][3]);
      tmax[qt] = max3f(tmax[qt], s[1][qt][0], s[1][qt][1]);
    }
    if constexpr (!decltype(cut)::value) {
#pragma unroll
      for (int i = 0; i < 3 * QT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);  // one vector instruction
      }
      __builtin_amdgcn_sched_group_barrier(0x008, QT, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      tmax[qt] = max3f(tmax[qt], s[1][qt][2], s[1][qt][3]);
      tmax[qt] = max3f(tmax[qt], s[2][qt][0], s[2][qt][1]);
      tmax[qt] = max3f(tmax[qt], s[2][qt][2], s[2][qt][3]);
      tmax[qt] = max3f(tmax[qt], s[3][qt][0], s[3][qt][1]);
      tmax[qt] = max3f(tmax[qt], s[3][qt][2], s[3][qt][3]);
      raise |= tmax[qt] > beyond[qt];
    }
    // a column's logits lie in four lanes; only where one of them is beyond the reference do they have to agree on a new one
    if (__builtin_amdgcn_ballot_w64(raise)) {
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        const float tm = quads_max(tmax[qt]);
        const bool up = tm > beyond[qt];
        const float nm = up ? tm * c : m_run[qt];
        beyond[qt] = up ? tm + kAttnLazy / c : beyond[qt];
        const float alpha = __builtin_amdgcn_exp2f(m_run[qt] - nm);
        ls[qt] *= alpha;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[d][qt][i] *= alpha;
        m_run[qt] = nm;
      }
    }
    // Four (two) steps of 32 keys and 32 queries.  A wave issues in order, so an MFMA that finds the matrix pipe busy holds back the vector
    // instructions behind it: the ten MFMAs of step u-1 are therefore spread between the vector instructions of
    // step u (one MFMA, then a tenth of the step's exponentials and conversions), each finding the pipe free.
    constexpr int QH = QT / 2;
    f16x8 pb[2][2];  // [step parity][query sub-tile of the step]
    static_for<2 * QH + 1>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      if constexpr (u > 0) {
        constexpr int qh = (u - 1) % QH;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
#pragma unroll
          for (int i = 0; i < 2; ++i) o[d][qh * 2 + i] = mfma_f16_16x16x32(fv[d], pb[(u - 1) & 1][i], o[d][qh * 2 + i]);
          if constexpr (u == QH) fv[d] = as_f16x8(st[512 + (4 + d) * 64]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) ls[qh * 2 + i] = mfma_f16_16x16x32(ones, pb[(u - 1) & 1][i], ls[qh * 2 + i]);
      }
      if constexpr (u < 2 * QH) {
        constexpr int p = u / QH, qh = u % QH;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          constexpr int q2 = qh * 2;
          const float nref = -m_run[q2 + i];
          f32x8 e;
#pragma unroll
          for (int j = 0; j < 8; ++j) e[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[p * 2 + (j >> 2)][q2 + i][j & 3], c, nref));
          pb[u & 1][i] = __builtin_convertvector(e, f16x8);
        }
        if constexpr (u > 0) {
#pragma unroll
          for (int i = 0; i < 10; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // four vector instructions
          }
        }
      } else {
        read_k(lds + ((t + 1) & 3) * 1024 + lane, 0, fa);  // behind the last tile: of a copy that nobody uses
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
#pragma unroll
    for (int d = 0; d < 4; ++d) o[d][qt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    m_run[qt] = beyond[qt] = -1.0e30f;
    ls[qt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  fetch(0, 0);
  fetch(1, 1);
  fetch(2, 2);
  __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt(8): tile 0
  __syncthreads();
  read_k(lds + lane, 0, fa);
  const int whole = len / 64;
  for (int t = 0; t < whole; ++t) tile(t, std::false_type{});
  if (whole < n_tiles) tile(whole, std::true_type{});
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing of this workgroup writes LDS that anyone may have by then

  // output: O^T / row sum; a lane's eight accumulators are the unit that the next product's operand wants from it
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const float inv = 1.0f / ls[qt][0];
    const int tile = q0 + qt;
    if (tile * 16 >= n_tiles * 64) continue;
    u32x4* ob = ao + (blk0 + (tile >> 3)) * (kBlk * kDT / 8) + ((tile & 7) * 16 + hd * 2) * 64 + lane;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      f32x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = o[s * 2 + (e >> 2)][qt][e & 3] * inv;
      ob[s * 64] = __builtin_bit_cast(u32x4, __builtin_convertvector(v, f16x8));
    }
  }
}

// ------------------------------------------------------------------------------------------
// overlap averaging: zg[t] = half(mean over the windows covering token t of x[row of t in that window])
// grid (ceil(N / 32) * parts of 64 columns, layers).  x lies in blocks (block_x4): half a wave reads the same four columns of 32 tokens, 512
// bytes in one piece; the rows of zg are put together in LDS and leave as whole lines of 128 bytes.  A thread's four loads are all in
// flight at once: with all 512 columns, four turns behind one another, one layer of 3500 tokens made 110 workgroups and took 15.3 us,
// 5.1 here (128 columns 5.7), eight of 1500 13.6 / 10.4, one of 8192 beside another lane 58.7 / 37.6.
// ------------------------------------------------------------------------------------------
constexpr int kAvgCols = 64;  // a workgroup's columns
__global__ __launch_bounds__(256) void overlap_avg_kernel(const f32x4* __restrict__ x, uint16_t* __restrict__ zg,
                                                           int N, int n_win, int Tp, int Np) {
  __shared__ f16x4 rows[32][kAvgCols / 4 + 2];
  zg += (size_t)blockIdx.y * Np * kDT;
  const int t0 = (int)(blockIdx.x / (kDT / kAvgCols)) * 32, c0 = (int)(blockIdx.x % (kDT / kAvgCols)) * kAvgCols;
  const int l32 = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int khi = t0 / kStride;  // the same for all 32 tokens
  const bool second = khi < n_win, first = khi >= 1 && khi - 1 < n_win;
  const int64_t row1 = (int64_t)blockIdx.y * Tp + (int64_t)khi * kWin + (t0 - khi * kStride) + l32;  // in window khi
  const int64_t row0 = row1 - (kWin - kStride);                                                       // in window khi - 1
  if (t0 + l32 < N) {
    f32x4 sum[kAvgCols / 32], other[kAvgCols / 32];
#pragma unroll
    for (int it = 0; it < kAvgCols / 32; ++it) {
      const int n = c0 + (it * 8 + g) * 4;
      sum[it] = other[it] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (second) sum[it] = x[block_x4(row1, n)];
      if (first) other[it] = x[block_x4(row0, n)];
    }
#pragma unroll
    for (int it = 0; it < kAvgCols / 32; ++it) {
      const f32x4 mean = (0.0f + sum[it] + other[it]) / (first && second ? 2.0f : 1.0f);
      rows[l32][it * 8 + g] = __builtin_convertvector(mean, f16x4);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 32 * (kAvgCols / 4); i += 256) {
    const int r = i / (kAvgCols / 4), c4 = i % (kAvgCols / 4);
    if (t0 + r < N) *reinterpret_cast<f16x4*>(zg + (size_t)(t0 + r) * kDT + c0 + c4 * 4) = rows[r][c4];
  }
}

// ------------------------------------------------------------------------------------------
// stage 3 per token (Eq. 3), after the K/V projection GEMM whose epilogue has already taken the inner products:
// s3[t] = [ <Q_l[h], K[s]> / 8 for h < H_l, s < H_s | <w_o, V[s]> for s < H_s ];
// yhat[ll, h, t] = sum_s softmax_s(logit[h][s]) * u[s] + b_o for every paired target layer ll.
// Block = 256 threads = (256 / H_l) tokens x H_l target heads, token index fastest; grid.y = layers.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void stage3_kernel(const float* __restrict__ s3, float b_o, float* __restrict__ yhat,
                                                      int64_t N, int Np, int H_s, int H_l, LayerBatch lb) {
  const int ll_lo = lb.lo[blockIdx.y], ll_hi = lb.hi[blockIdx.y];
  s3 += (size_t)blockIdx.y * Np * ((H_l + 1) * H_s);
  const int tok_per_block = 256 / H_l;
  const int tt = threadIdx.x % tok_per_block, h = threadIdx.x / tok_per_block;
  const int64_t t = (int64_t)blockIdx.x * tok_per_block + tt;
  if (h >= H_l || t >= N) return;
  const float* row = s3 + (size_t)t * ((H_l + 1) * H_s);
  const float* lg = row + h * H_s;
  const float* u = row + H_l * H_s;
  float mx = kNegInf;
  for (int s = 0; s < H_s; ++s) mx = __builtin_fmaxf(mx, lg[s]);
  float den = 0.0f, num = 0.0f;
  for (int s = 0; s < H_s; ++s) {
    const float e = __expf(lg[s] - mx);
    den += e;
    num += e * u[s];
  }
  const float y = num / den + b_o;
  for (int ll = ll_lo; ll < ll_hi; ++ll) yhat[((size_t)ll * H_l + h) * N + t] = y;
}

// Up to so many large tiles (half the CUs) the projection takes the 128 x 128 tiles as well: 14 of them (one layer of 3500 tokens) 18.2 us, in
// small ones 9.9, 96 (8 layers of 600) 25.6 / 17.9; 192 (8 of 1500) 33.5 / 37.9, 128 in either lane (one of 8192) 100 / 125.  The large ones
// read half as much and sum a coefficient vector's 64 rows per load.  The convolution is faster in small ones at every size.
constexpr int kTileProducts = 128;
template <int EPI>
hipError_t launch_gemm(const uint16_t* A, int lda, const uint16_t* W, const RowSpace& rs, int Nn, int K, const EpiArgs& ep,
                       int n_cu, hipStream_t stream) {
  constexpr int BM = kGemmTile, BN = kGemmTile, kLdsBytes = 2 * (BM + BN) * (kGemmBK / 8) * 16;
  const int64_t M = (int64_t)rs.layers * rs.stride;
  if (Nn % BN != 0 || K % kGemmBK != 0 || rs.valid <= 0 || rs.valid > rs.stride || rs.stride % 256 != 0 || M > INT32_MAX)
    return hipErrorInvalidValue;
  const int m_tiles = (int)(M / BM), n_tiles = Nn / BN;
  if (EPI != kEpiStage3 || (int64_t)m_tiles * n_tiles <= kTileProducts) {
    const int layer_tiles = (rs.valid + 127) / 128, row_tiles = layer_tiles * rs.layers;
    const unsigned blocks = (unsigned)((row_tiles + kXcds - 1) / kXcds * kXcds) * (unsigned)(Nn / 128);
    gemm_f16_tile_kernel<EPI><<<blocks, 256, 0, stream>>>(A, lda, rs.a_layer, W, row_tiles, layer_tiles, rs.valid, rs.stride, Nn / 128, K, ep);
    return hipGetLastError();
  }
  if constexpr (EPI == kEpiStage3) {
    static bool attr_set = false;  // setting it again is harmless
    if (!attr_set) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f16_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
      if (e != hipSuccess) return e;
      attr_set = true;
    }
    // one workgroup per CU, a multiple of the XCD count, no more than there are tiles per XCD list
    const int per_xcd_tiles = ((m_tiles + kXcds - 1) / kXcds) * n_tiles;
    int wg_per_xcd = n_cu / kXcds;
    if (wg_per_xcd < 1) wg_per_xcd = 1;
    if (wg_per_xcd > per_xcd_tiles) wg_per_xcd = per_xcd_tiles;
    gemm_f16_kernel<<<kXcds * wg_per_xcd, 512, kLdsBytes, stream>>>(A, lda, rs.a_layer, W, (int)M, rs.valid, rs.stride, Nn, K, ep);
  }
  return hipGetLastError();
}

// 128 queries per workgroup instead of 256?  `wide` workgroups of 256 and `narrow` ones of 128 in all lanes.  Two narrow ones read twice the
// keys that one wide does and take up to a tenth longer, but a CU runs two side by side: where wide ones would have it to
// themselves, a wave per SIMD and nothing beside its chain of products and exponentials, or where one lane's leave half of the CUs one and
// half two, the narrow ones are faster; and where a window's last wide one is mostly beyond it, a tenth fewer are computed.  Mapper, us, wide /
// narrow: one layer of 2600 tokens (wide 120) 744 / 671, of 3500 (176) 753 / 715, of 7000 (376) 946 / 918, of 8000 (448) 987 / 1021; 16 of
// 600 (384, narrow 640) 714 / 696, of 800 (512, 896) 819 / 796, of 1100 (640, 1152) 1139 / 1112, of 1000 (512, 1024) 946 / 960.
inline bool narrow_attention_pays(int64_t wide, int64_t narrow, int lanes) {
  return wide <= (lanes == 1 ? 384 : 256) || 5 * narrow <= 9 * wide;
}

// Second stem convolution, encoder and stage-3 inner products of one batch with the large tiles: from h1 to s3.
hipError_t mapper_large_body(proxykv_ctx* ctx, const MapperWorkspace& ws, const MapPlan& p, int n_layers, int64_t N, int n_cu, hipStream_t stream) {
  const proxykv_config& c = ctx->cfg;
  const MapperWeights& w = ctx->w;
  const int T = (int)p.T, Tp = (int)p.Tp, Np = (int)p.Np, n_win = (int)p.n_win;
  const LanePointers m = lane_pointers(c, p, ws);
  uint16_t* zg = m.zg;
  const unsigned nl = (unsigned)n_layers;

  EpiArgs e2 = {};
  e2.p0 = w.bn2_scale;
  e2.p1 = w.bn2_shift;
  e2.range = m.range;
  e2.cw = w.stem_cw;
  e2.cs = w.stem_cs;
  e2.out_f32 = m.x;
  e2.pe = w.pe;
  e2.n_win = n_win;
  e2.out_stride = Tp;
  const RowSpace rows_conv = {n_layers, (int)N, Np, (int64_t)(N + 2) * c.c_mid};
  PKV_TRY(launch_gemm<kEpiGeluPeWin>(m.h1, c.c_mid, w.conv2_w, rows_conv, kDT, 3 * c.c_mid, e2, n_cu, stream));

  // stage 2 (the stem's epilogue has written its input rows)
  const int tail = T - (n_win - 1) * kWin;
  auto in_window = [](int len, int q) { return (len + q - 1) / q; };
  auto workgroups = [&](int q) { return (int64_t)nl * p.lanes * kHeads * ((n_win - 1) * in_window(kWin, q) + in_window(tail, q)); };
  const bool narrow = narrow_attention_pays(workgroups(256), workgroups(128), p.lanes);
  const int n_qb = in_window(T < kWin ? T : kWin, narrow ? 128 : 256);
  for (int li = 0; li < c.n_enc_layers; ++li) {
    PKV_TRY(launch_encoder_block(ctx, p, n_layers, li, m.x, m.xb, m.qk, stream));
    const u32x4* qkv = reinterpret_cast<const u32x4*>(m.qk);
    u32x4* ao = reinterpret_cast<u32x4*>(m.xb);
    auto* attention = narrow ? window_attention_kernel<2> : window_attention_kernel<4>;
    attention<<<nl * (unsigned)(n_win * kHeads * n_qb), 256, 0, stream>>>(qkv, ao, T, Tp, n_win, n_qb);
    PKV_TRY(hipGetLastError());
  }
  if (c.n_enc_layers > 0) PKV_TRY(launch_encoder_block(ctx, p, n_layers, c.n_enc_layers, m.x, m.xb, m.qk, stream));
  overlap_avg_kernel<<<dim3((unsigned)((N + 31) / 32 * (kDT / kAvgCols)), nl), 256, 0, stream>>>(reinterpret_cast<const f32x4*>(m.x), zg, (int)N, n_win, Tp, Np);
  PKV_TRY(hipGetLastError());

  // stage 3
  const int nkv = kv3_stride(c);
  EpiArgs e3 = {};
  e3.p0 = w.kv_b;
  e3.p1 = w.queries;
  e3.g = w.out_w;
  e3.out_f32 = m.s3;
  e3.ldc = (c.H_l + 1) * c.H_kv;
  e3.n_slot = c.H_kv;
  e3.n_head = c.H_l;
  const RowSpace rows_N = {n_layers, (int)N, Np, (int64_t)Np * kDT};
  return launch_gemm<kEpiStage3>(zg, kDT, w.kv_w, rows_N, nkv, kDT, e3, n_cu, stream);
}

// The network for the layers of one batch (x_in: all proxy layers' scores [L_s, H_kv, N]); writes the rows of every target
// layer that is paired with one of them.
hipError_t mapper_batch(proxykv_ctx* ctx, const MapperWorkspace& ws, const MapPlan& p, const LayerBatch& lb, const float* x_in, int64_t N, float* yhat,
                        int n_cu, hipStream_t stream) {
  const proxykv_config& c = ctx->cfg;
  const MapperWeights& w = ctx->w;
  const LanePointers m = lane_pointers(c, p, ws);
  const unsigned nl = (unsigned)lb.n;
  absmax_kernel<<<dim3(kRangeWords, nl), 1024, 0, stream>>>(x_in, (int64_t)c.H_kv * N, lb, m.range);
  PKV_TRY(hipGetLastError());
  const int tok = (int64_t)nl * N >= 64 * 512 ? kStemTok : ((int64_t)nl * N >= 16 * 512 ? 16 : 4);
  stem_conv1_kernel<<<dim3((unsigned)((N + tok - 1) / tok), nl), 256, 0, stream>>>(
      x_in, w.conv1_w, w.bn1_scale, w.bn1_shift, m.range, w.stem_cw, w.stem_cs, lb, m.h1, c.H_kv, (int)N, c.c_mid, tok);
  PKV_TRY(hipGetLastError());
  if (p.small) PKV_TRY(mapper_small_body(ctx, ws, p, lb.n, N, stream));
  else PKV_TRY(mapper_large_body(ctx, ws, p, lb.n, N, n_cu, stream));
  const int tok_per_block = 256 / c.H_l;
  stage3_kernel<<<dim3((unsigned)((N + tok_per_block - 1) / tok_per_block), nl), 256, 0, stream>>>(m.s3, w.out_b, yhat, N, (int)p.Np,
                                                                                                c.H_kv, c.H_l, lb);
  return hipGetLastError();
}

}  // namespace

hipError_t mapper_forward(proxykv_ctx* ctx, const MapPlan& p, const float* x_in, float* yhat, hipStream_t stream) {
  const proxykv_config& c = ctx->cfg;
  int n_cu = 0, dev = 0;
  PKV_TRY(hipGetDevice(&dev));
  PKV_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  // batches are dealt round-robin to the lanes; lane 0 is the caller's stream, the others start behind the work already
  // queued there and are joined into it at the end
  if (p.lanes > 1) {
    PKV_TRY(hipEventRecord(ctx->lane_fork, stream));
    for (int lane = 1; lane < p.lanes; ++lane) PKV_TRY(hipStreamWaitEvent(ctx->lane_stream[lane], ctx->lane_fork, 0));
  }
  LayerBatch lb = {};
  int lane = 0, done = 0, batches = 0;  // layers and batches so far
  for (int ll = 0; ll < c.L_l;) {
    int ll_hi = ll + 1;
    while (ll_hi < c.L_l && ctx->pairing[ll_hi] == ctx->pairing[ll]) ++ll_hi;
    lb.ls[lb.n] = ctx->pairing[ll];
    lb.lo[lb.n] = ll;
    lb.hi[lb.n] = ll_hi;
    ++lb.n;
    ll = ll_hi;
    if (++done == (int)((int64_t)ctx->distinct_layers * (batches + 1) / p.n_batches)) {
      PKV_TRY(mapper_batch(ctx, ctx->m[lane], p, lb, x_in, p.N, yhat, n_cu, lane == 0 ? stream : ctx->lane_stream[lane]));
      ++batches;
      lb.n = 0;
      lane = lane + 1 < p.lanes ? lane + 1 : 0;
    }
  }
  for (lane = 1; lane < p.lanes; ++lane) {
    PKV_TRY(hipEventRecord(ctx->lane_join[lane], ctx->lane_stream[lane]));
    PKV_TRY(hipStreamWaitEvent(stream, ctx->lane_join[lane], 0));
  }
  return hipSuccess;
}

}  // namespace pkv
