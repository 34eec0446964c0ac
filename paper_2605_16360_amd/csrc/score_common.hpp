// Helpers shared by the two scoring passes: tile geometry, the XOR-swizzled LDS tile layout, the
// global -> register -> LDS staging of a tile, MFMA fragment reads and products of 32 rows.
#pragma once
#include "common.hpp"

namespace pkv {
namespace {

template <int D>
struct ScoreCfg {
  static constexpr int CPR = D / 8;             // 16-byte chunks per row
  static constexpr int ROWS = 8192 / D;         // rows of one streamed tile (16 KB)
  static constexpr int SUB = ROWS / 32;         // 32-row sub-tiles per tile
  static constexpr int LOADS = ROWS * CPR / 256;  // 16-byte chunks staged per thread and tile
  static constexpr int TILE_U4 = ROWS * CPR;    // 16-byte units per tile
};
constexpr int kNBuf = 3;
constexpr int kVmcnt0 = 0x0F70;  // s_waitcnt vmcnt(0)

// Block -> (group, item) on a one-dimensional grid.  The hardware deals blocks round-robin to the 8 XCDs, so XCD x
// = block % 8 takes the x-th eighth of the groups' items, (layer, KV head) groups one after the other: the `per_group` blocks of a group run
// on one XCD at about the same time and share its L2 copy of the queries they all stream in pass 2 (measured: 4.9 GB
// leave the L2s per launch at N = 32k instead of 18.5 GB with the key blocks of a group dealt over all XCDs).  Eighths of the items, not of
// the groups: two groups kept two XCDs busy and six idle (one layer of 4 heads, 14 000 queries and keys, both passes 426 -> 229 us,
// the sum form with 6000 142 -> 74).
constexpr int kScoreXcds = 8;
struct GroupBlock {
  int group, item;  // group == n_groups: nothing to do
};
__device__ __forceinline__ GroupBlock group_block(int n_groups, int per_group) {
  const int xcd = blockIdx.x % kScoreXcds, j = blockIdx.x / kScoreXcds;
  const int total = n_groups * per_group, each = total / kScoreXcds, more = total % kScoreXcds;  // XCDs below `more` take one more
  if (j >= each + (xcd < more)) return {n_groups, 0};
  const int i = xcd * each + (xcd < more ? xcd : more) + j;
  return {i / per_group, i % per_group};
}
// number of blocks of such a grid; 0 if it does not fit a one-dimensional launch
inline unsigned group_grid(int64_t n_groups, int64_t per_group) {
  const int64_t blocks = kScoreXcds * ((n_groups * per_group + kScoreXcds - 1) / kScoreXcds);
  return blocks < (1ll << 31) ? (unsigned)blocks : 0u;
}

// Item j of n_sets sets of `per` items each, whose items get shorter with their number: `batch` sets at a time, first the longest items
// of all of them, so that what is left at the end is short.  Not all sets at once: those that run together share an L2.
struct SetItem {
  int set, item;
};
__device__ __forceinline__ SetItem longest_first(int j, int n_sets, int per, int batch) {
  const int b = j / (batch * per), r = j - b * (batch * per);
  const int n = n_sets - b * batch < batch ? n_sets - b * batch : batch;
  return {b * batch + r % n, r / n};
}

// XOR swizzle of the 16-byte chunk index inside a row; keeps both the 16-byte tile stores and the
// MFMA fragment reads (16 consecutive rows, four neighbouring chunks) spread over all LDS banks.
template <int D>
__device__ __forceinline__ int swz(int row) {
  if constexpr (D == 64) return (row & 7) ^ ((row >> 3) & 1);
  else return row & 15;
}

template <int D>
struct TileRegs {
  u32x4 v[ScoreCfg<D>::LOADS];
};

// Fetches rows [row0, row0 + ROWS) of a [*, D] bf16 matrix; rows >= row_limit re-read the last
// valid row so that every access stays inside the matrix (the caller masks them).
template <int D>
__device__ __forceinline__ void tile_fetch(TileRegs<D>& r, const uint16_t* base, int row0, int row_limit, int tid) {
  using C = ScoreCfg<D>;
  const char* tb = reinterpret_cast<const char*>(base) + (size_t)row0 * (D * 2);
  if (row0 + C::ROWS <= row_limit) {  // interior tile: uniform base plus a per-thread 32-bit offset
    const uint32_t off = (uint32_t)(tid / C::CPR) * (D * 2) + (uint32_t)(tid % C::CPR) * 16;
#pragma unroll
    for (int i = 0; i < C::LOADS; ++i)
      r.v[i] = *reinterpret_cast<const u32x4*>(tb + off + (uint32_t)i * (256 / C::CPR) * (D * 2));
  } else {
#pragma unroll
    for (int i = 0; i < C::LOADS; ++i) {
      const int id = tid + 256 * i;
      const int row = id / C::CPR, ch = id % C::CPR;
      int grow = row0 + row;
      grow = grow < row_limit ? grow : row_limit - 1;
      r.v[i] = *reinterpret_cast<const u32x4*>(base + (size_t)grow * D + ch * 8);
    }
  }
}

template <int D>
__device__ __forceinline__ void tile_store(const TileRegs<D>& r, u32x4* lds, int tid) {
  using C = ScoreCfg<D>;
#pragma unroll
  for (int i = 0; i < C::LOADS; ++i) {
    const int id = tid + 256 * i;
    const int row = id / C::CPR, ch = id % C::CPR;
    lds[row * C::CPR + (ch ^ swz<D>(row))] = r.v[i];
  }
}

// The same from fp32, rounded to bf16 (to nearest even) when the tile is stored.
template <int D>
struct TileRegsF32 {
  u32x4 v[2 * ScoreCfg<D>::LOADS];
};
__device__ __forceinline__ u32x4 round_bf16(u32x4 lo, u32x4 hi) {
  typedef float f32x8 __attribute__((ext_vector_type(8)));
  const f32x4 a = __builtin_bit_cast(f32x4, lo), b = __builtin_bit_cast(f32x4, hi);
  return __builtin_bit_cast(u32x4, __builtin_convertvector(f32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}, bf16x8));
}
template <int D>
__device__ __forceinline__ void tile_fetch(TileRegsF32<D>& r, const float* base, int row0, int row_limit, int tid) {
  using C = ScoreCfg<D>;
#pragma unroll
  for (int i = 0; i < C::LOADS; ++i) {
    const int id = tid + 256 * i, ch = id % C::CPR, row = row0 + id / C::CPR;
    const float* at = base + (size_t)(row < row_limit ? row : row_limit - 1) * D + ch * 8;
    r.v[2 * i] = *reinterpret_cast<const u32x4*>(at);
    r.v[2 * i + 1] = *reinterpret_cast<const u32x4*>(at + 4);
  }
}
// `copy`, if not null: the rounded tile goes there as well, rows below `copy_rows` (the tile's first row is row 0 of it).
template <int D>
__device__ __forceinline__ void tile_store(const TileRegsF32<D>& r, u32x4* lds, int tid, uint16_t* copy, int copy_rows) {
  using C = ScoreCfg<D>;
#pragma unroll
  for (int i = 0; i < C::LOADS; ++i) {
    const int id = tid + 256 * i, ch = id % C::CPR, row = id / C::CPR;
    const u32x4 v = round_bf16(r.v[2 * i], r.v[2 * i + 1]);
    lds[row * C::CPR + (ch ^ swz<D>(row))] = v;
    if (copy != nullptr && row < copy_rows) *reinterpret_cast<u32x4*>(copy + (size_t)row * D + ch * 8) = v;
  }
}

template <int D>
__device__ __forceinline__ bf16x8 frag_read(const u32x4* lds, int row, int ch) {
  return as_bf16x8(lds[row * ScoreCfg<D>::CPR + (ch ^ swz<D>(row))]);
}

// Products of 32 rows (of an LDS tile) with a tile of W columns (resident), W = 32 with v_mfma_f32_32x32x16_bf16, W = 16 with two
// v_mfma_f32_16x16x32_bf16 per k-step.  A lane owns column lane % W and E of the 32 rows, acc_row(r) + 4 (lane / W).
template <int D, int W>
struct Rows32 {
  static constexpr int RT = 32 / W, KS = W == 32 ? 16 : 32, KK = D / KS, E = W / 2;
  struct Acc {
    std::conditional_t<W == 32, f32x16, f32x4> v[RT];
    __device__ __forceinline__ float get(int r) const { return W == 32 ? v[0][r] : v[r >> 2][r & 3]; }
    __device__ __forceinline__ void set(int r, float x) {
      if constexpr (W == 32) v[0][r] = x;
      else v[r >> 2][r & 3] = x;
    }
  };
  static __device__ __forceinline__ constexpr int acc_row(int r) { return (r >> 2) * (W == 32 ? 8 : 16) + (r & 3); }

  bf16x8 a[RT][KK];
  __device__ __forceinline__ void read(const u32x4* lds, int row0, int lane) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) a[rt][kk] = frag_read<D>(lds, row0 + rt * W + lane % W, kk * (KS / 8) + lane / W);
  }
  // a column tile's resident fragments: this lane's column is row `row` of a [*, D] matrix
  static __device__ __forceinline__ void columns(bf16x8 (&b)[KK], const uint16_t* base, int row, int lane) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) b[kk] = as_bf16x8(*reinterpret_cast<const u32x4*>(base + (size_t)row * D + kk * KS + lane / W * 8));
  }
  static __device__ __forceinline__ void columns(bf16x8 (&b)[KK], const float* base, int row, int lane) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const u32x4* at = reinterpret_cast<const u32x4*>(base + (size_t)row * D + kk * KS + lane / W * 8);
      b[kk] = as_bf16x8(round_bf16(at[0], at[1]));
    }
  }
  static __device__ __forceinline__ void keep_columns(const bf16x8 (&b)[KK], uint16_t* base, int row, int lane) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) *reinterpret_cast<u32x4*>(base + (size_t)row * D + kk * KS + lane / W * 8) = __builtin_bit_cast(u32x4, b[kk]);
  }
  static __device__ __forceinline__ Acc zero() {
    Acc c;
#pragma unroll
    for (int r = 0; r < E; ++r) c.set(r, 0.0f);
    return c;
  }
  __device__ __forceinline__ void step(Acc& c, const bf16x8 (&b)[KK], int rt, int kk) const {
    if constexpr (W == 32) c.v[rt] = mfma_bf16_32x32x16(a[rt][kk], b[kk], c.v[rt]);
    else c.v[rt] = mfma_bf16_16x16x32(a[rt][kk], b[kk], c.v[rt]);
  }
  // init + rows x one column tile
  __device__ __forceinline__ Acc product(const bf16x8 (&b)[KK], const Acc& init) const {
    Acc c = init;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) step(c, b, rt, kk);
    return c;
  }
  // the same with NT column tiles, a tile's products of two k-steps NT instructions or more apart
  template <int NT>
  __device__ __forceinline__ void products(Acc (&c)[NT], const bf16x8 (&b)[NT][KK], const Acc& init) const {
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) c[ct] = init;
    static_for<KK * RT * NT>([&](auto jc) {
      constexpr int j = decltype(jc)::value, kk = j / (RT * NT), rt = (j / NT) % RT, ct = rt ? NT - 1 - j % NT : j % NT;
      step(c[ct], b[ct], rt, kk);
    });
  }
};

// max(seed, the accumulators)
template <class R>
__device__ __forceinline__ float max_of(const typename R::Acc& a, float seed) {
  float m = max3f(a.get(0), a.get(1), a.get(2)), n = max3f(a.get(3), a.get(4), a.get(5));
#pragma unroll
  for (int r = 6; r < R::E; r += 4) {
    m = max3f(m, a.get(r), a.get(r + 1));
    if (r + 3 < R::E) n = max3f(n, a.get(r + 2), a.get(r + 3));
  }
  return max3f(seed, m, n);
}

constexpr float kNegInf = -__builtin_huge_valf();

// One workgroup's share of a query's softmax denominator: sum 2^(c * logit - m) over its keys.
struct LsePart {
  float m, l;
};
constexpr int kMaxLseSplits = 8;
// What pass 1 left of query `row` of [rows], from one word or from `splits` shares; neg_lse() = -log2(sum over all keys of
// 2^(c * logit)) / c.  Read when the query's tile is asked for, put together when the tile goes to LDS.
template <bool SPLIT>
struct LseRegs {
  float v;
  __device__ __forceinline__ void none() { v = kNegInf; }
  __device__ __forceinline__ void read(const float* p, size_t row, size_t, int) { v = p[row]; }
  __device__ __forceinline__ float neg_lse(float) const { return v; }
};
template <>
struct LseRegs<true> {
  LsePart p[kMaxLseSplits];
  __device__ __forceinline__ void none() {  // a sum that is too large for any logit: -inf
#pragma unroll
    for (int s = 0; s < kMaxLseSplits; ++s) p[s] = LsePart{0.0f, s == 0 ? -kNegInf : 0.0f};
  }
  __device__ __forceinline__ void read(const float* parts, size_t row, size_t rows, int splits) {
#pragma unroll
    for (int s = 0; s < kMaxLseSplits; ++s)
      p[s] = s < splits ? reinterpret_cast<const LsePart*>(parts)[(size_t)s * rows + row] : LsePart{-1.0e30f, 0.0f};
  }
  __device__ __forceinline__ float neg_lse(float inv_c) const {
    float m = p[0].m, l = 0.0f;
#pragma unroll
    for (int s = 1; s < kMaxLseSplits; ++s) m = __builtin_fmaxf(m, p[s].m);
#pragma unroll
    for (int s = 0; s < kMaxLseSplits; ++s) l = __builtin_fmaf(p[s].l, __builtin_amdgcn_exp2f(p[s].m - m), l);
    return -(m + __builtin_amdgcn_logf(l)) * inv_c;
  }
};

}  // namespace
}  // namespace pkv
