// KV-cache compaction (paper Sec. 3 and Sec. 4.3: the mask is applied to the target's cache and
// only the kept tokens remain): an ordered row gather, out[r, j, :] = in[r, idx[r, j], :], for K
// and V in one launch so the index read is shared.  Pure data movement in 16-byte pieces, two token rows in flight per thread (measured at
// N = 32 768, keep ratio 0.3: 0.436 ms with one or two, 0.45 ms with four, 0.96 ms with eight; plain instead of
// non-temporal loads 0.48 ms).
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"

namespace pkv {
namespace {

constexpr int kUnroll = 2;
constexpr int64_t kMaxThreads = 0xffffffff;  // per dimension of a launch

// grid (ceil(K / rows_per_block), rows); cpr = 16-byte chunks per token row.
__global__ __launch_bounds__(256) void compact_kernel(const u32x4* __restrict__ k_in, const u32x4* __restrict__ v_in,
                                                       const int32_t* __restrict__ idx, int64_t N, int K, int cpr,
                                                       u32x4* __restrict__ k_out, u32x4* __restrict__ v_out) {
  const int r = blockIdx.y;
  const int tokens_per_step = 256 / cpr;
  const int ch = threadIdx.x % cpr, tsub = threadIdx.x / cpr;
  const int j0 = blockIdx.x * tokens_per_step * kUnroll + tsub;
  const int32_t* ridx = idx + (size_t)r * K;
  const size_t in_base = (size_t)r * N * cpr, out_base = (size_t)r * K * cpr;
  u32x4 kv[kUnroll], vv[kUnroll];
  int jj[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    jj[u] = j0 + u * tokens_per_step;
    if (jj[u] < K && tsub < tokens_per_step) {
      const size_t src = in_base + (size_t)ridx[jj[u]] * cpr + ch;
      kv[u] = __builtin_nontemporal_load(k_in + src);
      vv[u] = __builtin_nontemporal_load(v_in + src);
    }
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    if (jj[u] < K && tsub < tokens_per_step) {
      const size_t dst = out_base + (size_t)jj[u] * cpr + ch;
      __builtin_nontemporal_store(kv[u], k_out + dst);
      __builtin_nontemporal_store(vv[u], v_out + dst);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The same gather with the cache as its own destination (the paper's mask is applied to the target's
// cache where it lies): afterwards tokens 0 .. K-1 of every row r are the kept tokens in order; what
// lies behind them is not touched.  idx is ascending, so token j moves from idx[j] >= j: a destination
// never lies behind its source, and the only hazard is a later token's destination overwriting an
// earlier token's source before it was read.  One workgroup per row walks the kept tokens in chunks
// of 128 in order: the loads of chunk c+1 are issued, a barrier makes sure every thread holds chunk
// c, then chunk c is stored.  Chunk c+1 reads tokens at or behind (c+1)*128, which chunk c's stores
// (tokens below (c+1)*128) cannot touch, so the two overlap safely.  K and V, and the 128-byte parts of a token, are
// independent of each other, so each gets a workgroup of its own: what bounds this kernel is the bytes in flight (tokens of
// 256 bytes, half kept: 32 rows of 12 000 with one workgroup per row 264 us, so 56; 600 rows 814 and 778).
// grid (rows, 2 * slices), 256 threads; cpr = 16-byte chunks per token, cps = those of a slice (<= 32).
// ---------------------------------------------------------------------------------------------
constexpr int kInplaceTokens = 128, kNoToken = 1 << 30;

// With counts != nullptr the rows are ragged (a budget shared by the `heads` rows of a layer): idx holds,
// per layer, heads * K flat indices h * N + n in ascending order, row r = (layer, h) keeps counts[r] of
// them, and its list starts behind those of the layer's earlier heads.
template <int PER>  // 16-byte pieces per thread and chunk
__global__ __launch_bounds__(256) void compact_inplace_kernel(u32x4* __restrict__ k, u32x4* __restrict__ v,
                                                               const int32_t* __restrict__ idx, int64_t N, int K, int cpr, int cps,
                                                               const int32_t* __restrict__ counts, int heads) {
  const int r = blockIdx.x, tid = threadIdx.x;
  const int32_t* ridx = idx + (size_t)r * K;
  int32_t sub = 0;  // what a stored index is ahead of the row's token number
  if (counts != nullptr) {
    const int layer = r / heads, h = r % heads;
    int start = 0;
    for (int hh = 0; hh < h; ++hh) start += counts[layer * heads + hh];
    ridx = idx + (size_t)layer * heads * K + start;
    K = counts[r];
    if (K <= 0) return;
    sub = (int32_t)(h * N);
  }
  u32x4* base = ((blockIdx.y & 1) ? v : k) + (size_t)r * N * cpr + (blockIdx.y >> 1) * cps;
  const int whole = K / kInplaceTokens, tail0 = whole * kInplaceTokens;  // whole chunks; the first token of the cut one behind them
  int tok[PER], ch[PER];  // token within a chunk of tokens, and 16-byte chunk of it, of this thread's pieces
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int piece = tid + 256 * u;
    tok[u] = piece < kInplaceTokens * cps ? piece / cps : kNoToken;
    ch[u] = piece % cps;
  }
  auto load_idx = [&](int c, int last, int32_t (&at)[PER]) {  // (positions behind `last` read that one)
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int left = last - c * kInplaceTokens;
      at[u] = ridx[c * kInplaceTokens + (tok[u] < left ? tok[u] : left)];
    }
  };
  auto store = [&](int c, int n, const u32x4 (&x)[PER]) {
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (tok[u] < n) base[(size_t)(c * kInplaceTokens + tok[u]) * cpr + ch[u]] = x[u];
  };
  // Every thread holds its part of a chunk (and of every chunk before it) before any of that chunk is stored: a barrier alone does
  // not wait for loads under way, so each thread's must have arrived in front of it (no slower: they are stored next).
  auto meet = [&](u32x4 (&x)[PER]) {
#pragma unroll
    for (int u = 0; u < PER; ++u) asm volatile("" : "+v"(x[u]));
    __syncthreads();
  };
  // the cut chunk: nothing that is stored before it lies in its way, so it is asked for first and stored last
  u32x4 xt[PER];
  if (tail0 < K) {
    int32_t at[PER];
    load_idx(whole, K - 1, at);
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (tok[u] < K - tail0) xt[u] = __builtin_nontemporal_load(base + (size_t)(at[u] - sub) * cpr + ch[u]);
  }
  if (whole > 0) {
    // A piece without a token reads the last one of its chunks and stores nothing.  There is no branch around a load, and indices are
    // asked for a chunk ahead of the pieces they lead to: with a branch and its index in front of every piece, a thread has one
    // piece in flight instead of two chunks of them (600 rows of 12 000 tokens of 256 bytes, half kept: 889 us, so 775).
    auto load = [&](const int32_t (&at)[PER], u32x4 (&x)[PER]) {
#pragma unroll
      for (int u = 0; u < PER; ++u) x[u] = __builtin_nontemporal_load(base + (size_t)(at[u] - sub) * cpr + ch[u]);
    };
    // x holds chunk c and a the indices of chunk c + 1; y takes that chunk and b the indices of the one behind it
    auto step = [&](int c, u32x4 (&x)[PER], u32x4 (&y)[PER], int32_t (&a)[PER], int32_t (&b)[PER]) {
      load_idx(c + 2, tail0 - 1, b);
      if (c + 1 < whole) load(a, y);
      meet(x);
      store(c, kInplaceTokens, x);
    };
    int32_t a0[PER], a1[PER];
    u32x4 x0[PER], x1[PER];
    load_idx(0, tail0 - 1, a0);
    load_idx(1, tail0 - 1, a1);
    load(a0, x0);
    for (int c = 0; c < whole; c += 2) {  // (two steps by name: moving x1 to x0 would wait for it)
      step(c, x0, x1, a1, a0);
      if (c + 1 < whole) step(c + 1, x1, x0, a0, a1);
    }
  }
  if (tail0 < K) {
    meet(xt);
    store(whole, K - tail0, xt);
  }
}

// ---------------------------------------------------------------------------------------------
// The same in parts of a row that any number of workgroups move at once.  A workgroup takes kPartPieces pieces of 16 bytes (640 tokens of 256),
// all of them into registers, and stores them when the parts in front of it in the row have been loaded: a token's new place never
// lies behind its old one, so what a part's places still hold belongs to itself or to a part in front.  Parts are dealt by a
// counter per layer and tensor, in order: whoever a workgroup waits for has started before it and waits for earlier ones only, so every wait
// ends, whatever order the workgroups are launched in, as long as no other launch uses the same counters at the same time.  It has no
// bound: a part that stored before the ones in front are loaded would destroy tokens, and a clock goes on while the queue is off the chip.
// What bounds it is memory.  With workgroups of a whole row, two chunks of it in flight, a long row was what the launch waited for.  Half kept,
// D = 128, us: 512 rows of 12 345 tokens 652 -> 548 (3.2 GB: 5.9 TB/s), with budgets that eight heads share 727 -> 567; 256 of 32 000, 0.3
// kept, shared 756 -> 455; 112 of 8000 96 -> 87; 4 of 30 000 97 -> 16.
// Parts of 160 KB, one workgroup on a CU; the first three also in us with 128 KB, two on a CU: 566, 574, 465; 256 KB: 548, 553, 442, but 256 rows
// of 2200 64 instead of 57; 64 KB in eight pieces a thread 579, 641, 569.
// state: per (layer, tensor) the counter, then a word per part, all zero at the start.  grid 2 * layers * (stride - 1).
// ---------------------------------------------------------------------------------------------
constexpr int kPartThreads = 512, kPartPer = 20, kPartPieces = kPartThreads * kPartPer;

__global__ __launch_bounds__(256) void clear_words_kernel(uint32_t* __restrict__ words, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) words[i] = 0u;
}

__device__ __forceinline__ int wave_scan(int v) {  // inclusive
#pragma unroll
  for (int off = 1; off < 64; off *= 2) {
    const int o = __shfl_up(v, off, 64);
    v += ((int)threadIdx.x & 63) >= off ? o : 0;
  }
  return v;
}

__global__ __launch_bounds__(kPartThreads, 3) void compact_parts_kernel(u32x4* __restrict__ k, u32x4* __restrict__ v, const int32_t* __restrict__ idx,
                                                                     int64_t N, int K, int cpr, int part_tokens, const int32_t* __restrict__ counts,
                                                                     int heads, uint32_t* __restrict__ state, int stride) {
  __shared__ int32_t at[kPartPieces];
  __shared__ int s_head, s_part, s_kept, s_start;
  const int tid = threadIdx.x, lane = tid & 63, group = blockIdx.x / (stride - 1), layer = group >> 1;
  uint32_t* mine = state + (size_t)group * stride;
  uint32_t ticket = 0;
  if (tid < 64) {
    if (lane == 0) ticket = atomicAdd(mine, 1u);
    ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)ticket);
    // the head and part that this is, parts counted over the layer's heads
    int part = (int)ticket, start = 0;
    if (lane == 0) s_part = -1;
    if (counts == nullptr) {
      if (lane == 0 && part * (int64_t)part_tokens < K) {
        s_head = 0;
        s_part = part;
        s_kept = K;
        s_start = 0;
      }
    } else {
      for (int h0 = 0; h0 < heads && part >= 0; h0 += 64) {
        const int c = h0 + lane < heads ? counts[(size_t)layer * heads + h0 + lane] : 0;
        const int parts = (c + part_tokens - 1) / part_tokens, upto = wave_scan(parts), kept = wave_scan(c);
        if (part >= upto - parts && part < upto) {
          s_head = h0 + lane;
          s_part = part - (upto - parts);
          s_kept = c;
          s_start = start + kept - c;
        }
        part -= __shfl(upto, 63, 64);
        start += __shfl(kept, 63, 64);
      }
    }
  }
  __syncthreads();
  const int part = s_part, j0 = part * part_tokens;
  if (part < 0) return;
  const int n = s_kept - j0 < part_tokens ? s_kept - j0 : part_tokens;
  const int32_t* list = idx + (size_t)layer * heads * K + s_start + j0;
  const int32_t sub = (int32_t)(s_head * N);  // what a stored index is ahead of the row's token number
  for (int i = tid; i < n; i += kPartThreads) at[i] = list[i] - sub;
  __syncthreads();
  u32x4* base = ((group & 1) ? v : k) + ((size_t)layer * heads + s_head) * N * cpr;
  u32x4 x[kPartPer];
  const int tok_step = kPartThreads / cpr, ch_step = kPartThreads % cpr;
  {
    int tok = tid / cpr, ch = tid % cpr;
#pragma unroll
    for (int u = 0; u < kPartPer; ++u) {  // (a piece without a token loads the last one's)
      x[u] = __builtin_nontemporal_load(base + (size_t)at[tok < n ? tok : n - 1] * cpr + ch);
      tok += tok_step;
      ch += ch_step;
      if (ch >= cpr) {
        ch -= cpr;
        ++tok;
      }
    }
  }
  // every thread's pieces have arrived: the part is loaded
#pragma unroll
  for (int u = 0; u < kPartPer; ++u) asm volatile("" : "+v"(x[u]));
  __syncthreads();
  if (tid < 64) {
    uint32_t* loaded = mine + 1 + ticket;
    if (lane == 0) __hip_atomic_store(loaded, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int p = lane; p < part; p += 64)
      while (__hip_atomic_load(loaded - 1 - p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) __builtin_amdgcn_s_sleep(1);
  }
  __syncthreads();
  int tok = tid / cpr, ch = tid % cpr;
#pragma unroll
  for (int u = 0; u < kPartPer; ++u) {
    if (tok < n) __builtin_nontemporal_store(x[u], base + (size_t)(j0 + tok) * cpr + ch);
    tok += tok_step;
    ch += ch_step;
    if (ch >= cpr) {
      ch -= cpr;
      ++tok;
    }
  }
}

// mask[r, n] = 1 for the kept tokens of row r, 0 elsewhere (uint8).  One workgroup per row clears the row,
// then sets the kept positions: 1024 threads for rows that keep them busy (256 rows of 32 768: 9.2 us with 256, 5.4 us with
// 1024; 512 rows of 3000: 1.9 and 3.1 us).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void mask_kernel(const int32_t* __restrict__ idx, int64_t N, int K,
                                                       uint8_t* __restrict__ mask) {
  const int r = blockIdx.x, tid = threadIdx.x;
  uint8_t* row = mask + (size_t)r * N;
  // 16-byte stores over the aligned middle, bytes at the ragged ends
  const uintptr_t addr = reinterpret_cast<uintptr_t>(row);
  const int64_t head = (int64_t)((16 - (addr & 15)) & 15) < N ? (int64_t)((16 - (addr & 15)) & 15) : N;
  const int64_t n16 = (N - head) / 16;
  for (int64_t i = tid; i < head; i += THREADS) row[i] = 0;
  u32x4* mid = reinterpret_cast<u32x4*>(row + head);
  for (int64_t i = tid; i < n16; i += THREADS) mid[i] = u32x4{0, 0, 0, 0};
  for (int64_t i = head + n16 * 16 + tid; i < N; i += THREADS) row[i] = 0;
  __syncthreads();  // workgroup-scope release/acquire: the zeros are in place before the ones
  const int32_t* ridx = idx + (size_t)r * K;
  for (int j = tid; j < K; j += THREADS) row[ridx[j]] = 1;
}

// counts[layer, h] = number of a layer's kept flat indices (ascending, heads * K of them) that fall into
// [h * N, (h + 1) * N): the difference of two lower bounds.  One wave per (layer, head); every step of a search probes 64
// places at once, so that the two searches are three or four trips to memory instead of 34 (9.9 us with one thread each).
__global__ __launch_bounds__(64) void head_counts_kernel(const int32_t* __restrict__ flat, int64_t pairs, int heads, int64_t N, int K,
                                                         int32_t* __restrict__ counts) {
  for (int64_t t = blockIdx.x; t < pairs; t += gridDim.x) {
    const int h = (int)(t % heads), n = heads * K, lane = threadIdx.x;
    const int32_t* row = flat + (size_t)(t / heads) * n;
    int lo[2] = {0, 0}, hi[2] = {n, n};  // the first position whose index is >= (h + e) * N lies in [lo[e], hi[e]]
    while (lo[0] < hi[0] || lo[1] < hi[1]) {
      bool less[2];
      int step[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        step[e] = (hi[e] - lo[e] + 63) / 64;
        const int64_t at = lo[e] + (int64_t)lane * step[e];
        less[e] = at < hi[e] && (int64_t)row[at] < (int64_t)(h + e) * N;
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int below = __popcll(__builtin_amdgcn_ballot_w64(less[e]));  // the probes are in order: the first `below` are less
        if (below == 0) {
          hi[e] = lo[e];
        } else {
          const int64_t top = lo[e] + (int64_t)below * step[e];
          hi[e] = top < hi[e] ? (int)top : hi[e];
          lo[e] += (below - 1) * step[e] + 1;
        }
      }
    }
    if (lane == 0) counts[t] = lo[1] - lo[0];
  }
}

}  // namespace

hipError_t launch_compact(const void* k_in, const void* v_in, const int32_t* idx, int64_t rows, int64_t N, int64_t K,
                          int64_t row_bytes, void* k_out, void* v_out, hipStream_t stream) {
  if (rows <= 0 || K <= 0) return hipSuccess;
  const int cpr = (int)(row_bytes / 16);
  const int tokens_per_block = (256 / cpr) * kUnroll;
  dim3 grid((unsigned)((K + tokens_per_block - 1) / tokens_per_block), (unsigned)rows);
  compact_kernel<<<grid, 256, 0, stream>>>((const u32x4*)k_in, (const u32x4*)v_in, idx, N, (int)K, cpr,
                                           (u32x4*)k_out, (u32x4*)v_out);
  return hipGetLastError();
}

// Parts that a layer's kept tokens (heads * K) can make, however its heads share them; 0 where a launch has no room for them.
static int64_t layer_parts(int64_t layers, int64_t K, int64_t row_bytes, int heads) {
  const int64_t tokens = kPartPieces / (row_bytes / 16), parts = (heads * K + tokens - 1) / tokens + (heads > 1 ? heads - 1 : 0);
  return 2 * layers * parts * kPartThreads <= kMaxThreads ? parts : 0;
}
// Whether parts are faster than whole rows.  What a row keeps has to fill one and a half of them (three with budgets of their own in fewer
// than 256 rows), and they have to be worth their turns: whole rows take as long as a workgroup's chain, 8 ns a token, and as their bytes
// beside it; parts a launch that clears the state and 10 us for every 256 of them, the last few like a full turn.  In us, fitted over
// 1832 shapes with cold caches: 1 to 512 rows, D = 8 to 256, 1.5 to 50 parts a row, 0.3 and 0.7 kept.  With parts taken by their number
// alone 128 of the shapes were more than 2 % slower than whole rows, up to 1.29 times; so 52, up to 1.19 (80 rows of D = 256, 3.9 parts,
// parts / whole rows 43.6 / 36.6; 112 of D = 128, shared budgets, 1.6 parts 31.1 / 28.3 and 31.8 / 31.6).  Parts / whole rows on either side: D = 256,
// one row that keeps 1440 tokens 12.8 / 10.5, 1984 12.8 / 14.5; 28 rows, 1440 23.7 / 19.0, 2880 35.2 / 37.3; D = 128, four rows with shared
// budgets, 1024 12.3 / 9.9, 1408 12.3 / 12.0 to 13.2; 256 rows, 1024 54 / 57.
static bool parts_pay(int64_t rows, int64_t K, int64_t row_bytes, int heads) {
  const int64_t cpr = row_bytes / 16, tokens = kPartPieces / cpr, least = heads > 1 || rows >= 256 ? 3 : 6;
  if (2 * K < least * tokens) return false;
  const double mb = 2e-6 * (double)rows * (double)K * (double)row_bytes, wide = cpr % 8 == 0 ? 1.0 : (double)cpr / 8.0;
  const double chain = 0.008 * wide * (double)K + 0.25 * mb, bytes = 0.38 * mb;
  const double whole = (chain > bytes ? chain : bytes) * (heads > 1 ? 1.2 : 1.0);  // (of shared budgets the longest row is what is left)
  const double parts = 2.0 * (double)rows * (heads > 1 ? (double)K / (double)tokens + 0.5 : (double)((K + tokens - 1) / tokens));
  const double turns = 4.0 + 10.0 * ceil(parts / 256.0);
  return (turns > 0.36 * mb ? turns : 0.36 * mb) <= whole;
}
size_t compact_inplace_scratch_most(int64_t rows, int64_t K, int64_t row_bytes, int heads) {
  const int64_t layers = rows / heads, parts = rows > 0 ? layer_parts(layers, K, row_bytes, heads) : 0;
  return (size_t)(2 * layers * (parts + 1)) * 4;
}
size_t compact_inplace_scratch_bytes(int64_t rows, int64_t K, int64_t row_bytes, int heads) {
  if (rows <= 0 || layer_parts(rows / heads, K, row_bytes, heads) == 0 || !parts_pay(rows, K, row_bytes, heads)) return 0;
  return compact_inplace_scratch_most(rows, K, row_bytes, heads);
}

hipError_t launch_compact_inplace(void* k, void* v, const int32_t* idx, int64_t rows, int64_t N, int64_t K, int64_t row_bytes,
                                  const int32_t* counts, int heads, void* scratch, size_t scratch_bytes, hipStream_t stream) {
  if (rows <= 0 || K <= 0) return hipSuccess;
  const int cpr = (int)(row_bytes / 16);
  const size_t need = compact_inplace_scratch_bytes(rows, K, row_bytes, heads);
  if (need > 0 && scratch_bytes >= need) {
    const int64_t layers = rows / heads, parts = layer_parts(layers, K, row_bytes, heads), words = (int64_t)(need / 4);
    clear_words_kernel<<<(unsigned)((words + 255) / 256), 256, 0, stream>>>((uint32_t*)scratch, words);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    compact_parts_kernel<<<(unsigned)(2 * layers * parts), kPartThreads, 0, stream>>>((u32x4*)k, (u32x4*)v, idx, N, (int)K, cpr, kPartPieces / cpr,
                                                                                     counts, heads, (uint32_t*)scratch, (int)parts + 1);
    return hipGetLastError();
  }
  // 128-byte parts of a token where it divides into them, and 256-byte ones where K and V of the rows alone give every CU two workgroups
  // (D = 128, 128-byte and 256-byte parts, us: 512 rows of 12 345 tokens, half kept, 697 and 680; 256 of 2000, 0.8 kept, 78 and 76, of
  // 5000 with shared budgets, 0.3 kept, 139 and 128; but 112 of 2000 49 and 51, of 21 718 with shared budgets, 0.145 kept, 144 and 150: a long
  // row is then all that is left at the end; 4 rows of 20 000, 67 and 89).  Rows of equal budgets of up to four chunks are better off with
  // twice as many workgroups (256 rows, kept 150 of 1500 18.3 and 19.3, 280 of 700 23.9 and 24.2, 500 of 5000 36.8 and 37.4; 600 of 1500 level,
  // 512 rows 69.7 and 67.8), those of shared budgets are not (256 rows, 280 a head of 700 35.9 and 35.2, 400 of 1000 44.5 and 43.0).
  const int part = rows >= 256 && (counts != nullptr || K > 4 * kInplaceTokens) && cpr % 16 == 0 ? 16 : 8;
  const int slices = cpr % part == 0 ? cpr / part : 1, cps = cpr / slices;
  const int per = (kInplaceTokens * cps + 255) / 256;                 // 16-byte pieces per thread and chunk
  u32x4 *kp = (u32x4*)k, *vp = (u32x4*)v;
  const dim3 grid((unsigned)rows, (unsigned)(2 * slices));
  auto go = [&](auto p) { compact_inplace_kernel<decltype(p)::value><<<grid, 256, 0, stream>>>(kp, vp, idx, N, (int)K, cpr, cps, counts, heads); };
  if (per <= 1) go(std::integral_constant<int, 1>{});
  else if (per <= 2) go(std::integral_constant<int, 2>{});
  else if (per <= 4) go(std::integral_constant<int, 4>{});
  else if (per <= 8) go(std::integral_constant<int, 8>{});
  else if (per <= 16) go(std::integral_constant<int, 16>{});
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_head_counts(const int32_t* flat, int64_t layers, int64_t heads, int64_t N, int64_t K, int32_t* counts,
                              hipStream_t stream) {
  const int64_t n = layers * heads;
  if (n <= 0) return hipSuccess;
  const int64_t most = kMaxThreads / 64;
  head_counts_kernel<<<(unsigned)(n < most ? n : most), 64, 0, stream>>>(flat, n, (int)heads, N, (int)K, counts);
  return hipGetLastError();
}

hipError_t launch_mask(const int32_t* idx, int64_t rows, int64_t N, int64_t K, uint8_t* mask, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (N >= 8192 && rows <= kMaxThreads / 1024) mask_kernel<1024><<<(unsigned)rows, 1024, 0, stream>>>(idx, N, (int)K, mask);
  else mask_kernel<256><<<(unsigned)rows, 256, 0, stream>>>(idx, N, (int)K, mask);
  return hipGetLastError();
}

}  // namespace pkv
