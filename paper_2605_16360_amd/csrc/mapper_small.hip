// The mapper's kernels for few rows (a short context, few proxy layers).  With the 256 x 256 tiles of mapper.hip a batch of
// 512 rows is 4 to 16 workgroups on 256 CUs, each a chain of up to 32 K steps: latency, not throughput, is what such an
// input costs.  These kernels cut the same products into small tiles, so that every CU has one, and shorten each chain:
//   small_wide_kernel  K = d_time (512): 64 x 64 tiles whose A and W rows are loaded into LDS whole, one round trip to memory.
//                      Its prologue can normalise the rows (LayerNorm) as it reads them, so that this needs no launch of
//                      its own: QKV projection, FFN-1, stage-3 K/V projection.
//   small_deep_kernel  32 x 32 tiles, the four waves of a workgroup share the K axis and meet in LDS: second stem
//                      convolution, out-projection, FFN-2.  It leaves the pre-norm sum to the next kernel's prologue.
//   small_attention_kernel  32 queries of one (layer, head) per workgroup, its four waves share the keys.
// A layer of more than one window has more rows than they take, so a layer's tokens, window rows and window are the same here.
// Results are rounded where the kernels of mapper.hip round; sums are fp32 in another order.
// Measured, one layer of 512 rows: 867 -> 231 us, and 226 with row statistics in place of the normalised rows and four tokens per workgroup
// of the first convolution; 2560 rows (kMapSmallRows) are their end.
#include "common.hpp"
#include "context.hpp"
#include "kernels.hpp"
#include "mapper.hpp"

namespace pkv {
namespace {

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

constexpr int kVmcnt0 = 0x0F70;  // s_waitcnt vmcnt(0)

static_assert(kMapSmallRows < kWin + kStride + 1, "a layer of two windows is not for these kernels");

// Tile of a block.  Blocks are dealt round-robin to the 8 XCDs; each XCD takes its own column tiles for all row tiles, so a
// weight row is fetched into one L2 only, and every activation into all of them.  (The weights outweigh the activations up to about 512 rows: the second FFN
// product's are 2 MB either way there.)
__device__ __forceinline__ void small_tile(int n_tiles, int& nt, int& mt) {
  const int b = (int)blockIdx.x;
  if (n_tiles % kXcds == 0) {
    const int j = b / kXcds, per = n_tiles / kXcds;
    nt = (j % per) * kXcds + b % kXcds;
    mt = j / per;
  } else {
    nt = b % n_tiles;
    mt = b / n_tiles;
  }
}

// Where the A rows of small_wide_kernel come from.
enum Prologue {
  kProHalf,    // fp16 rows as they are
  kProLn       // LayerNorm of fp32 rows; their means and scales also go to `stats`, for the residual of the next sum
};
enum WideEpilogue { kWideQkv, kWideRelu, kWideStage3 };

// mean and 1 / standard deviation of a row: the next sum takes its residual as the row normalised once more (the rows themselves,
// 1 MB per 512, took 0.8 us per launch to store)
struct RowStats {
  float mu, rstd;
};

struct WideArgs {
  const uint16_t* a_half;
  const float* pre;           // kProLn: rows to normalise
  const float *g, *b;         // LayerNorm scale and shift
  RowStats* stats;
  const uint16_t* w;          // [n_tiles * 64, 512]
  const float* bias;
  int n_tiles, tiles_per_layer;  // column tiles; row tiles of a layer
  int rows, stride;           // valid rows of a layer and rows between layers (A and outputs)
  uint16_t *out_h, *out_v;
  float* out_f32;
  int ldc;
  const float *queries, *out_w;  // kWideStage3
  int n_slot, n_head;
};

// One row of 512 fp32 over 16 lanes: lane j holds chunks (8 values) j, j + 16, j + 32, j + 48.
__device__ __forceinline__ void load_row16(const float* row, int j, f32x8 (&v)[4]) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const f32x4 lo = *reinterpret_cast<const f32x4*>(row + (c * 16 + j) * 8);
    const f32x4 hi = *reinterpret_cast<const f32x4*>(row + (c * 16 + j) * 8 + 4);
    v[c] = f32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  }
}
// sum over the 16 lanes that share a row, by lane permutes within the vector ALU: neighbours, pairs, then the mirrored
// half and the mirrored row, whose lanes hold the other four and the other eight
__device__ __forceinline__ float sum16(float v) {
  auto add = [&](auto ctrl) {
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  add(std::integral_constant<int, 0xB1>{});   // quad_perm 1 0 3 2
  add(std::integral_constant<int, 0x4E>{});   // quad_perm 2 3 0 1
  add(std::integral_constant<int, 0x141>{});  // row_half_mirror
  add(std::integral_constant<int, 0x140>{});  // row_mirror
  return v;
}
__device__ __forceinline__ RowStats layernorm_row16(f32x8 (&v)[4], const f32x8 (&g)[4], const f32x8 (&b)[4]) {
  float s = 0.0f;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int e = 0; e < 8; ++e) s += v[c][e];
  const float mu = sum16(s) * (1.0f / kDT);
  float q = 0.0f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    v[c] -= mu;
#pragma unroll
    for (int e = 0; e < 8; ++e) q += v[c][e] * v[c][e];
  }
  const float rstd = 1.0f / sqrtf(sum16(q) * (1.0f / kDT) + 1e-5f);
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = v[c] * rstd * g[c] + b[c];
  return {mu, rstd};
}

// grid n_tiles * layers * tiles_per_layer, 128 KB of LDS: 64 A rows, then 64 W rows, 64 chunks of 16 bytes each, chunk c
// of row r at c ^ (r & 15).  The normalisation of the 64 rows is a long chain of vector instructions, which one wave per
// SIMD issues at half the rate or less: kWideWaves waves, which also share the K axis of the products.
constexpr int kWideLds = 2 * 64 * 64 * 16;
constexpr int kWideWaves = 8, kWideRows = 64 / kWideWaves, kWideKs = kWideWaves / 4;

template <int PRO, int EPI>
__global__ __launch_bounds__(64 * kWideWaves, 1) void small_wide_kernel(WideArgs a) {
  extern __shared__ u32x4 lds[];
  u32x4* lw = lds + 64 * 64;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  int nt, mt;
  small_tile(a.n_tiles, nt, mt);
  const int layer = mt / a.tiles_per_layer, r0 = (mt % a.tiles_per_layer) * 64;

  // W rows: a wave instruction moves one row, every lane the chunk that its LDS place holds
  const uint16_t* wsrc = a.w + (size_t)(nt * 64 + wave * kWideRows) * kDT;
  if constexpr (PRO == kProHalf) {
#pragma unroll
    for (int i = 0; i < kWideRows; ++i) {
      const int row = wave * kWideRows + i, ch = lane ^ (row & 15);
      __builtin_amdgcn_global_load_lds((gptr_t)(wsrc + i * kDT + ch * 8), (lptr_t)(lw + row * 64), 16, 0, 0);
      const int m = r0 + row < a.rows ? r0 + row : a.rows - 1;
      const uint16_t* src = a.a_half + ((size_t)layer * a.stride + m) * kDT + ch * 8;
      __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(lds + row * 64), 16, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(kVmcnt0);
  } else {
    // The fp32 rows are asked for first and the W rows behind them (through registers: loads return in order), so that the
    // rows are normalised while the weights are on their way.
    const int j = lane & 15;
    constexpr int kIts = kWideRows / 4;  // rows per lane group
    u32x4 wr[kWideRows];
    f32x8 g[4], b[4], v[kIts][4];
#pragma unroll
    for (int it = 0; it < kIts; ++it) {
      const int row = wave * kWideRows + it * 4 + (lane >> 4);
      const int m = r0 + row < a.rows ? r0 + row : a.rows - 1;
      load_row16(a.pre + ((size_t)layer * a.stride + m) * kDT, j, v[it]);
    }
    load_row16(a.g, j, g);
    load_row16(a.b, j, b);
#pragma unroll
    for (int i = 0; i < kWideRows; ++i) wr[i] = *reinterpret_cast<const u32x4*>(wsrc + i * kDT + (lane ^ ((wave * kWideRows + i) & 15)) * 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = 0; it < kIts; ++it) {
      const int row = wave * kWideRows + it * 4 + (lane >> 4);
      const RowStats st = layernorm_row16(v[it], g, b);
      if (EPI != kWideStage3 && nt == 0 && j == 0 && r0 + row < a.rows) a.stats[(size_t)layer * a.stride + r0 + row] = st;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        lds[row * 64 + ((c * 16 + j) ^ (row & 15))] = __builtin_bit_cast(u32x4, __builtin_convertvector(v[it][c], f16x8));
    }
#pragma unroll
    for (int i = 0; i < kWideRows; ++i) lw[(wave * kWideRows + i) * 64 + lane] = wr[i];
  }
  __syncthreads();

  // wave (ks, wm, wn): rows 32 wm .. +31, columns 32 wn .. +31, part ks of the K axis
  const int ks = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1, sw = l32 & 15;
  const u32x4* fa = lds + (wm * 32 + l32) * 64;
  const u32x4* fb = lw + (wn * 32 + l32) * 64;
  f32x16 acc = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 8
  for (int k = 0; k < kDT / 16 / kWideKs; ++k) {
    const int slot = ((ks * (kDT / 16 / kWideKs) + k) * 2 + half) ^ sw;
    acc = mfma_f16_32x32x16(as_f16x8(fa[slot]), as_f16x8(fb[slot]), acc);
  }
  __syncthreads();  // the rows have been read: their place takes the partial sums and the output tile
  f32x4* part = reinterpret_cast<f32x4*>(lds);  // [ks - 1][wm, wn][register / 4][lane]
  if (ks > 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      part[(((ks - 1) * 4 + (wave & 3)) * 4 + r) * 64 + lane] = f32x4{acc[4 * r], acc[4 * r + 1], acc[4 * r + 2], acc[4 * r + 3]};
  }
  __syncthreads();
  if (ks == 0) {
#pragma unroll
    for (int o = 0; o < kWideKs - 1; ++o)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x4 v = part[((o * 4 + wave) * 4 + r) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * r + e] += v[e];
      }
  }
  // lane: column 32 wn + l32 of the tile, register r: row 32 wm + (r / 4) * 8 + half * 4 + r % 4
  const int n = nt * 64 + wn * 32 + l32;
  const float bias = a.bias[n];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] += bias;

  if constexpr (EPI == kWideQkv) {
    if (nt * 64 >= 2 * kDT) {
      if (ks > 0) return;
      // v transposed and key-permuted as the attention reads it: registers 8u .. 8u+7 are eight consecutive positions
      const int rg = r0 + wm * 32, vc = n - 2 * kDT;
      uint16_t* vb = a.out_v + ((size_t)(layer * kHeads + (vc >> 6)) * 64 + (vc & 63)) * a.stride + rg + half * 8;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f32x8 t;
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = acc[u * 8 + e];
        *reinterpret_cast<f16x8*>(vb + u * 16) = __builtin_convertvector(t, f16x8);
      }
      return;
    }
  }
  // the output tile takes the W rows' place
  if constexpr (EPI == kWideStage3) {
    // column tile = one slot: its 64 rows x 64 columns in LDS, then inner products with the learned queries (key slots,
    // a wave takes 64 rows of one query) or with the output weights (value slots)
    float* ct = reinterpret_cast<float*>(lw);
    if (ks == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) ct[(wm * 32 + (r >> 2) * 8 + half * 4 + (r & 3)) * 65 + wn * 32 + l32] = acc[r];
    }
    __syncthreads();
    const int slot = nt;
    const bool is_k = slot < a.n_slot;
    const int row = lane;
    for (int h = wave; h < (is_k ? a.n_head : 1); h += kWideWaves) {
      const float* cf = is_k ? a.queries + h * 64 : a.out_w;
      float t0 = 0.0f, t1 = 0.0f, t2 = 0.0f, t3 = 0.0f;
#pragma unroll
      for (int e = 0; e < 64; e += 4) {
        t0 = __builtin_fmaf(ct[row * 65 + e], cf[e], t0);
        t1 = __builtin_fmaf(ct[row * 65 + e + 1], cf[e + 1], t1);
        t2 = __builtin_fmaf(ct[row * 65 + e + 2], cf[e + 2], t2);
        t3 = __builtin_fmaf(ct[row * 65 + e + 3], cf[e + 3], t3);
      }
      const float tot = (t0 + t1) + (t2 + t3);
      if (r0 + row < a.rows) {
        float* orow = a.out_f32 + ((size_t)layer * a.stride + r0 + row) * a.ldc;
        if (is_k) orow[h * a.n_slot + slot] = tot * 0.125f;
        else orow[a.n_head * a.n_slot + slot - a.n_slot] = tot;
      }
    }
  } else {
    // through LDS, so that a row leaves as 128 contiguous bytes (the outputs' row count is padded: no predicate)
    uint16_t* ct = reinterpret_cast<uint16_t*>(lw);
    if (ks == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float v = EPI == kWideRelu ? __builtin_fmaxf(acc[r], 0.0f) : acc[r];
        ct[(wm * 32 + (r >> 2) * 8 + half * 4 + (r & 3)) * 72 + wn * 32 + l32] = to_h(v);
      }
    }
    __syncthreads();
    for (int id = tid; id < 512; id += 64 * kWideWaves) {
      const int row = id >> 3, ch = id & 7;
      *reinterpret_cast<u32x4*>(a.out_h + ((size_t)layer * a.stride + r0 + row) * a.ldc + nt * 64 + ch * 8) =
          *reinterpret_cast<const u32x4*>(ct + row * 72 + ch * 8);
    }
  }
}

// ------------------------------------------------------------------------------------------
// 32 x 32 tiles, N = 512.  Wave w of the four takes the K range [w K / 4, (w + 1) K / 4) in steps of 64 through LDS of its
// own (no barrier until the sums meet), four steps in flight in registers.  K a multiple of 256.
// ------------------------------------------------------------------------------------------
enum DeepEpilogue {
  kDeepRes,       // out_f32 = res + (sum + bias): the pre-norm row
  kDeepGeluPe     // the second stem convolution: GELU(sum * scale * 2^s + shift) + position
};
struct DeepArgs {
  const uint16_t* a;
  int lda;
  int64_t a_layer;
  const uint16_t* w;  // [512, K]
  int K, rows, tiles_per_layer;
  int out_stride;     // output rows between layers
  const float *p0, *p1;  // bias, or scale and shift
  const float* res;      // kDeepRes: the residual rows, as they are or, with `stats`, to be normalised; may be out_f32
  const RowStats* stats;
  const float *g, *b;    // LayerNorm scale and shift
  float* out_f32;
  uint16_t* out_h;
  const float* pe;
  const uint32_t* range;
  float cw, cs;
};

template <int EPI>
__global__ __launch_bounds__(256, 2) void small_deep_kernel(DeepArgs a) {
  __shared__ u32x4 lds[4 * 512];  // per wave: 32 A rows and 32 W rows of 8 chunks
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  int nt, mt;
  small_tile(kDT / 32, nt, mt);
  const int layer = mt / a.tiles_per_layer, r0 = (mt % a.tiles_per_layer) * 32;
  u32x4* la = lds + wave * 512;
  u32x4* lw = la + 256;
  const int n_steps = a.K / 256, kw = wave * (a.K / 4);
  const int srow = lane >> 3, sch = lane & 7;
  const uint16_t* arow[4];
  const uint16_t* wrow[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = r0 + srow + 8 * i < a.rows ? r0 + srow + 8 * i : a.rows - 1;
    arow[i] = a.a + (size_t)layer * a.a_layer + (size_t)m * a.lda + kw + sch * 8;
    wrow[i] = a.w + (size_t)(nt * 32 + srow + 8 * i) * a.K + kw + sch * 8;
  }
  constexpr int kDepth = 4;
  u32x4 ra[kDepth][4], rw[kDepth][4];
  auto fetch = [&](int s, u32x4 (&xa)[4], u32x4 (&xw)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      xa[i] = *reinterpret_cast<const u32x4*>(arow[i] + s * 64);
      xw[i] = *reinterpret_cast<const u32x4*>(wrow[i] + s * 64);
    }
  };
#pragma unroll
  for (int d = 0; d < kDepth; ++d)
    if (d < n_steps) fetch(d, ra[d], rw[d]);
  f32x16 acc = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  const int fsw = swz8(l32);
  for (int s0 = 0; s0 < n_steps; s0 += kDepth) {
    static_for<kDepth>([&](auto dc) {
      constexpr int d = decltype(dc)::value;
      if (s0 + d < n_steps) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = srow + 8 * i;
          la[row * 8 + (sch ^ swz8(row))] = ra[d][i];
          lw[row * 8 + (sch ^ swz8(row))] = rw[d][i];
        }
        if (s0 + d + kDepth < n_steps) fetch(s0 + d + kDepth, ra[d], rw[d]);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int slot = l32 * 8 + ((kk * 2 + half) ^ fsw);
          acc = mfma_f16_32x32x16(as_f16x8(la[slot]), as_f16x8(lw[slot]), acc);
        }
      }
    });
  }
  // the four partial tiles meet in LDS (each wave's in its own part), thread t sums row t / 8, columns 4 (t % 8) .. +3
  float* part = reinterpret_cast<float*>(la);
#pragma unroll
  for (int r = 0; r < 16; ++r) part[((r >> 2) * 8 + half * 4 + (r & 3)) * 36 + l32] = acc[r];
  __syncthreads();
  const int row = tid >> 3, c4 = (tid & 7) * 4, t = r0 + row, n = nt * 32 + c4;
  f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(lds + w * 512) + row * 36 + c4);
  if (t >= a.rows) return;
  const f32x4 p0 = *reinterpret_cast<const f32x4*>(a.p0 + n);
  const size_t o = ((size_t)layer * a.out_stride + t) * kDT + n;
  if constexpr (EPI == kDeepRes) {
    f32x4 r = *reinterpret_cast<const f32x4*>(a.res + o);
    if (a.stats != nullptr) {
      const RowStats st = a.stats[(size_t)layer * a.out_stride + t];
      r = (r - st.mu) * st.rstd * *reinterpret_cast<const f32x4*>(a.g + n) + *reinterpret_cast<const f32x4*>(a.b + n);
    }
    *reinterpret_cast<f32x4*>(a.out_f32 + o) = v + (r + p0);
  } else {
    const f32x4 p1 = *reinterpret_cast<const f32x4*>(a.p1 + n);
    const float up = exp2_int(stem_exponent(a.range + layer * kRangeWords, a.cw, a.cs));
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_erf(__builtin_fmaf(v[e], p0[e] * up, p1[e]));
    const f32x4 y = v + *reinterpret_cast<const f32x4*>(a.pe + (size_t)t * kDT + n);
    *reinterpret_cast<f32x4*>(a.out_f32 + o) = y;
    *reinterpret_cast<f16x4*>(a.out_h + o) = __builtin_convertvector(y, f16x4);
  }
}

// ------------------------------------------------------------------------------------------
// Window attention for few rows: a workgroup takes 32 queries of one (layer, head); wave w takes the 64-key tiles w, w + 4,
// ... through LDS of its own, each with an online softmax of its own, and the four meet in LDS at the end.  The products,
// the lazily raised reference and the layouts are those of window_attention_kernel (mapper.hip).
// grid layers * 8 heads * n_qb, n_qb = blocks of 32 queries per layer; block b: head b % 8 (one XCD per head).
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void small_attention_kernel(const uint16_t* __restrict__ qk, const uint16_t* __restrict__ vt,
                                                                  uint16_t* __restrict__ ao, int len, int Tp, int n_qb) {
  __shared__ u32x4 lds[4 * 1024];  // per wave: K tile (64 keys x 8 chunks), V^T tile (64 d rows x 8 chunks)
  __shared__ float ml[2][4][32];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int hd = blockIdx.x % kHeads, j8 = blockIdx.x / kHeads;
  const int layer = j8 / n_qb, i0 = (j8 % n_qb) * 32;
  const int64_t base = (int64_t)layer * Tp;
  constexpr float c = 1.4426950408889634f * 0.125f;  // log2(e) / sqrt(64)

  f16x8 bq[4];
  {
    const int row = i0 + l32 < len ? i0 + l32 : len - 1;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      bq[kk] = as_f16x8(*reinterpret_cast<const u32x4*>(qk + (size_t)(base + row) * (2 * kDT) + hd * 64 + kk * 16 + half * 8));
  }
  const uint16_t* kbase = qk + (size_t)base * (2 * kDT) + kDT + hd * 64;
  const uint16_t* vbase = vt + (size_t)(layer * kHeads + hd) * 64 * Tp;
  const int n_tiles = (len + 63) / 64;
  u32x4* lk = lds + wave * 1024;
  u32x4* lv = lk + 512;
  const int srow = lane >> 3, sch = lane & 7;
  u32x4 rk[8], rv[8];
  auto fetch = [&](int t) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = srow + 8 * i;
      int j = t * 64 + row;
      j = j < len ? j : len - 1;
      rk[i] = *reinterpret_cast<const u32x4*>(kbase + (size_t)j * (2 * kDT) + sch * 8);
      rv[i] = *reinterpret_cast<const u32x4*>(vbase + (size_t)row * Tp + t * 64 + sch * 8);
    }
  };
  f32x16 o[2];
#pragma unroll
  for (int ds = 0; ds < 2; ++ds) o[ds] = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  float m_run = -1.0e30f, l_run = 0.0f;
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  const f16x2 ones = {(_Float16)1.0f, (_Float16)1.0f};
  const int fsw = swz8(l32);
  if (wave < n_tiles) fetch(wave);
  for (int t = wave; t < n_tiles; t += 4) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = srow + 8 * i;
      lk[row * 8 + (sch ^ swz8(row))] = rk[i];
      lv[row * 8 + (sch ^ swz8(row))] = rv[i];
    }
    if (t + 4 < n_tiles) fetch(t + 4);
    f32x16 s[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      s[ks] = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) s[ks] = mfma_f16_32x32x16(as_f16x8(lk[(ks * 32 + l32) * 8 + ((kk * 2 + half) ^ fsw)]), bq[kk], s[ks]);
    }
    if (t * 64 + 64 > len) {
      const int lim = len - t * 64 - half * 4;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[ks][r] = (ks * 32 + (r >> 2) * 8 + (r & 3)) < lim ? s[ks][r] : kNegInf;
    }
    const float tmax = halves_max(max16_8(s[0], s[1])) * c;
    if (__builtin_amdgcn_ballot_w64(tmax > m_run + kAttnLazy)) {
      const float nm = tmax > m_run + kAttnLazy ? tmax : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - nm);
      l_run *= alpha;
#pragma unroll
      for (int ds = 0; ds < 2; ++ds)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[ds][r] *= alpha;
      m_run = nm;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      f32x8 p;
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u >> 1][(u & 1) * 8 + e], c, -m_run));
      const f16x8 pb = __builtin_convertvector(p, f16x8);
#pragma unroll
      for (int e = 0; e < 8; e += 2) l_run = __builtin_amdgcn_fdot2(f16x2{pb[e], pb[e + 1]}, ones, l_run, false);
#pragma unroll
      for (int ds = 0; ds < 2; ++ds)
        o[ds] = mfma_f16_32x32x16(as_f16x8(lv[(ds * 32 + l32) * 8 + ((u * 2 + half) ^ fsw)]), pb, o[ds]);
    }
  }
  // the waves' results meet: O^T [64 d][32 queries] of each in its own LDS part, references and sums beside them
  l_run = halves_sum(l_run);
  float* ow = reinterpret_cast<float*>(lk);
#pragma unroll
  for (int ds = 0; ds < 2; ++ds)
#pragma unroll
    for (int r = 0; r < 16; ++r) ow[l32 * 65 + ds * 32 + (r >> 2) * 8 + half * 4 + (r & 3)] = o[ds][r];
  if (half == 0) {
    ml[0][wave][l32] = m_run;
    ml[1][wave][l32] = l_run;
  }
  __syncthreads();
  const int qr = tid >> 3, d0 = (tid & 7) * 8;
  float m = ml[0][0][qr];
#pragma unroll
  for (int w = 1; w < 4; ++w) m = __builtin_fmaxf(m, ml[0][w][qr]);
  float l = 0.0f;
  f32x8 sum = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float f = __builtin_amdgcn_exp2f(ml[0][w][qr] - m);
    l += f * ml[1][w][qr];
    const float* orow = reinterpret_cast<const float*>(lds + w * 1024) + qr * 65 + d0;
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] += f * orow[e];
  }
  if (i0 + qr < len)
    *reinterpret_cast<f16x8*>(ao + (size_t)(base + i0 + qr) * kDT + hd * 64 + d0) = __builtin_convertvector(sum * (1.0f / l), f16x8);
}

template <int PRO, int EPI>
hipError_t launch_wide(const WideArgs& a, int layers, hipStream_t stream) {
  static bool attr_set = false;  // per instantiation; setting it again is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&small_wide_kernel<PRO, EPI>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kWideLds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  small_wide_kernel<PRO, EPI><<<(unsigned)(layers * a.tiles_per_layer * a.n_tiles), 64 * kWideWaves, kWideLds, stream>>>(a);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_deep(const DeepArgs& a, int layers, hipStream_t stream) {
  if (a.K % 256 != 0) return hipErrorInvalidValue;
  small_deep_kernel<EPI><<<(unsigned)(layers * a.tiles_per_layer * (kDT / 32)), 256, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t mapper_small_body(proxykv_ctx* ctx, const MapperWorkspace& ws, const MapPlan& p, int n_layers, int64_t N64, hipStream_t stream) {
  const proxykv_config& c = ctx->cfg;
  const MapperWeights& w = ctx->w;
  const int N = (int)N64, Np = (int)p.Np;  // a layer's rows, and padded
  const LanePointers m = lane_pointers(c, p, ws);
  float *x = m.x, *pre = m.pre;
  RowStats* stats = reinterpret_cast<RowStats*>(x);  // x is read for the last time before the first of them is written
  uint16_t *xb = m.xb, *qk = m.qk, *vt = m.vt, *ao = m.ao, *hid = m.hid;

  DeepArgs d = {};
  d.a = m.h1;
  d.lda = c.c_mid;
  d.a_layer = (int64_t)(N + 2) * c.c_mid;
  d.w = w.conv2_w;
  d.K = 3 * c.c_mid;
  d.rows = N;
  d.tiles_per_layer = (N + 31) / 32;
  d.out_stride = Np;
  d.p0 = w.bn2_scale;
  d.p1 = w.bn2_shift;
  d.out_f32 = x;
  d.out_h = xb;
  d.pe = w.pe;
  d.range = m.range;
  d.cw = w.stem_cw;
  d.cs = w.stem_cs;
  PKV_TRY(launch_deep<kDeepGeluPe>(d, n_layers, stream));

  // x: the encoder's first rows, the residual of the first sum; pre: the sum that the next kernel normalises, and the one behind it once
  // more for its residual
  const int n_qb = (N + 31) / 32;
  WideArgs a = {};
  a.tiles_per_layer = (N + 63) / 64;
  a.rows = N;
  a.stride = Np;
  a.pre = pre;
  a.stats = stats;
  d = DeepArgs{};
  d.rows = N;
  d.tiles_per_layer = (N + 31) / 32;
  d.out_stride = Np;
  d.res = x;
  d.out_f32 = pre;
  for (int li = 0; li < c.n_enc_layers; ++li) {
    const EncoderLayerWeights& e = w.enc[li];
    WideArgs q = a;
    q.w = e.in_w;
    q.bias = e.in_b;
    q.n_tiles = 3 * kDT / 64;
    q.out_h = qk;
    q.out_v = vt;
    q.ldc = 2 * kDT;
    if (li == 0) {
      q.a_half = xb;
      PKV_TRY((launch_wide<kProHalf, kWideQkv>(q, n_layers, stream)));
    } else {
      q.g = w.enc[li - 1].ln2_g;
      q.b = w.enc[li - 1].ln2_b;
      PKV_TRY((launch_wide<kProLn, kWideQkv>(q, n_layers, stream)));
    }
    small_attention_kernel<<<(unsigned)(n_layers * kHeads * n_qb), 256, 0, stream>>>(qk, vt, ao, N, Np, n_qb);
    PKV_TRY(hipGetLastError());
    if (li > 0) {
      d.stats = stats;
      d.g = w.enc[li - 1].ln2_g;
      d.b = w.enc[li - 1].ln2_b;
    }
    d.a = ao;
    d.lda = kDT;
    d.a_layer = (int64_t)Np * kDT;
    d.w = e.out_w;
    d.K = kDT;
    d.p0 = e.out_b;
    PKV_TRY(launch_deep<kDeepRes>(d, n_layers, stream));
    WideArgs f = a;
    f.w = e.ffn1_w;
    f.bias = e.ffn1_b;
    f.n_tiles = c.d_ffn / 64;
    f.g = e.ln1_g;
    f.b = e.ln1_b;
    f.out_h = hid;
    f.ldc = c.d_ffn;
    PKV_TRY((launch_wide<kProLn, kWideRelu>(f, n_layers, stream)));
    d.res = pre;
    d.stats = stats;
    d.g = e.ln1_g;
    d.b = e.ln1_b;
    d.a = hid;
    d.lda = c.d_ffn;
    d.a_layer = (int64_t)Np * c.d_ffn;
    d.w = e.ffn2_w;
    d.K = c.d_ffn;
    d.p0 = e.ffn2_b;
    PKV_TRY(launch_deep<kDeepRes>(d, n_layers, stream));
  }
  WideArgs h = a;
  h.w = w.kv_w;
  h.bias = w.kv_b;
  h.n_tiles = 2 * c.H_kv;
  h.g = w.enc[c.n_enc_layers - 1].ln2_g;
  h.b = w.enc[c.n_enc_layers - 1].ln2_b;
  h.out_f32 = m.s3;
  h.ldc = (c.H_l + 1) * c.H_kv;
  h.queries = w.queries;
  h.out_w = w.out_w;
  h.n_slot = c.H_kv;
  h.n_head = c.H_l;
  return launch_wide<kProLn, kWideStage3>(h, n_layers, stream);
}

}  // namespace pkv
