// Per-row Top-K selection (paper Sec. 3: the mask keeps the Top-K of the mapped scores per target
// layer and head; Sec. 4.3 names a Top-K kernel that materialises it).  Integer work only: scores
// are turned into order-preserving 32-bit keys, the K-th largest key is found by a radix select, and one more ordered
// pass emits the kept indices in ascending order, taking equal keys by lower index.
//
// Every kernel reads a row in chunks of 4096 scores, four consecutive ones per thread: a wave's load is 1 KB in one piece
// (36 consecutive scores per thread, which makes the ordered output a plain prefix sum over the threads, reads 64 lines
// per load instead of 8 and took 44 us for 256 rows of 32 768 against 27 us).  The order of the output is kept
// by counting per (chunk, wave) and ranking inside a wave with ballots, so that stores too lie side by side.
//
// A row of up to 36 864 scores is one workgroup's, its keys stay in registers for all passes.  A longer row is split into
// parts, one workgroup each.  Where there are rows enough, and all parts fit the chip at once, those stay in registers too and the workgroups
// of a row meet after every digit (one launch).  Few rows, and more than fit, take three launches of an 11-bit radix pass on the raw
// keys whose per-part histograms meet in a per-row histogram in device scratch memory (the last workgroup of a row to
// arrive picks the digit), then one launch that writes every part's kept indices behind those of the parts before it.
// Where the scratch memory is too small for 2048-bin histograms the same kernels run four passes of 8 bits.
#include "common.hpp"
#include "kernels.hpp"

namespace pkv {
namespace {

constexpr int kTopkThreads = 1024;
constexpr int kTopkWaves = kTopkThreads / 64;

// Larger key <=> earlier in the selection order.  NaN maps to 0 (below -inf), -0.0 onto +0.0 (-0.0 + 0.0 = +0.0).
__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f + 0.0f);
  const uint32_t k = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
  return f == f ? k : 0u;
}
// The score of a key other than 0: score > that float <=> key above it, and NaN is neither above nor equal.
__device__ __forceinline__ float key_score(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? k ^ 0x80000000u : ~k);
}

// Four scores row[i], ..., row[i + 3] of a row that starts on any 4-byte boundary.  Nothing at or past hi is read: a quad that
// would is the last four below it, so that row[i] is its element quad_shift(i, hi) (the row has at least four scores below
// hi).  There is no branch: with one per quad the compiler waits for a quad before it asks for the next (nine trips to
// memory, one after the other, in a row of 36 864 scores).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ int quad_shift(int i, int hi) { return i > hi - 4 ? i - (hi - 4) : 0; }
__device__ __forceinline__ f32x4 load_quad(const float* row, int i, int hi) {
  const f32x4_any v = *reinterpret_cast<const f32x4_any*>(row + (i - quad_shift(i, hi)));
  return f32x4{v[0], v[1], v[2], v[3]};
}
// the quad with row[i] in element 0 again; the last `shift` elements mean nothing
__device__ __forceinline__ f32x4 shift_quad(f32x4 v, int shift) {
  if (shift & 2) v = f32x4{v[2], v[3], v[3], v[3]};
  if (shift & 1) v = f32x4{v[1], v[2], v[3], v[3]};
  return v;
}
constexpr int kChunk = 4 * kTopkThreads;

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask, uint32_t add) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, add));
}
// inclusive prefix sum over the wave within the vector ALU: four steps inside rows of 16 lanes, then the row totals
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  auto add = [&](auto ctrl, auto rows) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xf, true);
  };
  add(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});  // row_shr 1
  add(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});  // row_shr 2
  add(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});  // row_shr 4
  add(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});  // row_shr 8
  add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});  // row_bcast 15 into rows 1 and 3
  add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});  // row_bcast 31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ uint32_t wave_total(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(v), 63);
}
// Ordered output of a wave's scores: quad q of lane l holds the scores 256 q + 4 l .. +3 of the wave's stretch, whose first has
// index i0.  Kept: scores above the threshold (bit 4 (q % 8) + j of m_gt[q / 8]), and those equal to it (m_eq) of which fewer than
// eq_take equal ones lie in front; gt and eq count the scores above and equal in front of the stretch.  A kept one goes to
// out[kept ones in front of it].  Loops are left rolled: this code runs once per wave, and straight-line code of 25 KB
// spends its time on instruction fetch (112 rows of 170 000 scores: 31 us without any load or store).
// Four quads share a prefix sum, a byte each: a lane has at most 252 scores of a quad in front of it, and what a full quad carries into the
// next byte of lane 63's inclusive sum goes away with the lane's own counts.
// Kept indices go to the wave's place in LDS first and from there to memory side by side: stored from where they are found,
// a wave's stores of four quads are sixteen instructions of a fifth of its lanes each (256 rows of 32 767 scores, nine in ten kept: the whole
// kernel 28.5 -> 23.3 us; 512 of 12 000, half kept, 14.3 -> 12.9 with the shared prefix sum).
constexpr int kStageWords = 1024;  // of a wave: four quads
template <int WORDS>
__device__ __forceinline__ void wave_write(const uint32_t (&m_gt)[WORDS], const uint32_t (&m_eq)[WORDS], int quads, uint32_t gt, uint32_t eq,
                                           uint32_t eq_take, int i0, int lane, int32_t* stage, int32_t* out) {
  int i = i0 + 4 * lane;
  out += (size_t)gt + (eq < eq_take ? eq : eq_take);
#pragma unroll
  for (int w = 0; w < WORDS; ++w) {
    uint32_t wg = m_gt[w], we = m_eq[w];
#pragma unroll 1
    for (int left = quads - 8 * w < 8 ? quads - 8 * w : 8; left > 0; left -= 4, wg >>= 16, we >>= 16, i += 1024) {
      uint32_t n = wg & 0xffffu;  // per nibble its number of bits, to a byte
      const uint64_t any_eq = __builtin_amdgcn_ballot_w64((we & 0xffffu) != 0);
      uint32_t kept = wg;
      if (any_eq != 0) {
        // equal ones join the others here; lanes, and in a lane quads, hold them in another order than the indices': quad by quad
        uint32_t first = eq;
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {
          const uint32_t be = (we >> (4 * q)) & 15u, ne = (uint32_t)__popc(be), inc = wave_inclusive_scan(ne);
          uint32_t e = first + inc - ne, take = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t is = (be >> j) & 1u;
            take |= (e < eq_take ? is : 0u) << j;
            e += is;
          }
          kept |= take << (4 * q);
          first += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
        eq = first;
        n = kept & 0xffffu;
      }
      if (left <= 2) {  // short rows and parts, and the end of others: stored from where they are found, the way through LDS is longer
#pragma unroll 1
        for (int q = 0; q < left; ++q, kept >>= 4) {
          const uint32_t bits = kept & 15u, own = (uint32_t)__popc(bits), inc = wave_inclusive_scan(own);
          int32_t* at = out + (inc - own);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t bit = (bits >> j) & 1u;
            if (bit) *at = i + q * 256 + j;
            at += bit;
          }
          out += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
        continue;
      }
      n = (n | n << 8) & 0x00ff00ffu;
      n = (n | n << 4) & 0x0f0f0f0fu;
      n -= (n >> 1) & 0x05050505u;
      n = (n & 0x03030303u) + ((n >> 2) & 0x03030303u);
      const uint32_t front = wave_inclusive_scan(n) - n;
      const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)front, 63), own = (uint32_t)__builtin_amdgcn_readlane((int)n, 63);
      uint32_t total = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q < left) {
          int32_t* at = stage + total + ((front >> (8 * q)) & 255u);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t bit = (kept >> (4 * q + j)) & 1u;
            if (bit) *at = i + q * 256 + j;
            at += bit;
          }
          total += ((last >> (8 * q)) & 255u) + ((own >> (8 * q)) & 255u);
        }
      }
      // (a wave's LDS operations are carried out in order: the compiler is all that has to keep it)
      asm volatile("" ::: "memory");
      for (uint32_t k = 4 * lane; k < total; k += 256) {
        const i32x4 v = *reinterpret_cast<const i32x4*>(stage + k);
        if (k + 4 <= total) {
          *reinterpret_cast<i32x4_any*>(out + k) = i32x4_any{v[0], v[1], v[2], v[3]};
        } else {
#pragma unroll
          for (int j = 0; j < 3; ++j)
            if (k + j < total) out[k + j] = v[j];
        }
      }
      asm volatile("" ::: "memory");
      out += total;
    }
  }
}
// bits of a quad's scores above and equal to the threshold: t = key_score(T), or any number with nan_t where T is the key
// of NaN (then every number lies above it and NaNs are equal to it).  `valid`: scores of the quad that exist.
__device__ __forceinline__ void quad_bits(const f32x4& v, int valid, float t, bool nan_t, uint32_t& bg, uint32_t& be) {
  bg = 0;
  be = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bg |= (uint32_t)(nan_t ? v[j] == v[j] : v[j] > t) << j;
    be |= (uint32_t)(nan_t ? v[j] != v[j] : v[j] == t) << j;
  }
  const uint32_t m = valid >= 4 ? 15u : (valid > 0 ? (1u << valid) - 1u : 0u);
  bg &= m;
  be &= m;
}

// sum over the workgroup of one value per thread; `part`: kTopkWaves words of LDS, free again after the call
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* part, int tid) {
  v = wave_total(v);
  if ((tid & 63) == 0) part[tid >> 6] = v;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int w = 0; w < kTopkWaves; ++w) t += part[w];
  __syncthreads();
  return t;
}

// exclusive prefix sum of one value per thread over the workgroup; `part` as in block_sum, but in use until the caller's
// next barrier
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* part, int wave, int lane) {
  const uint32_t inc = wave_inclusive_scan(v);
  if (lane == 63) part[wave] = inc;
  __syncthreads();
  uint32_t before = inc - v;
#pragma unroll
  for (int w = 0; w < kTopkWaves; ++w) before += w < wave ? part[w] : 0u;
  return before;
}

// The digit that holds the krem-th largest key, from the counts of kDigits bins, thread t holding the kPer bins
// kDigits - 1 - t * kPer, ... in descending order (cnt zero for threads without bins): calls found(digit, krem left, the digit's
// count) in one thread.
template <int kDigits, int kPer, class F>
__device__ __forceinline__ void pick_digit(const uint32_t (&cnt)[kPer], uint32_t krem, uint32_t* part, int tid, F&& found) {
  uint32_t own = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) own += cnt[i];
  uint32_t above = block_exclusive_scan(own, part, tid >> 6, tid & 63);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (above < krem && krem <= above + cnt[i]) found((uint32_t)(kDigits - 1 - (tid * kPer + i)), krem - above, cnt[i]);
    above += cnt[i];
  }
}

// ---------------------------------------------------------------------------------------------
// Rows whose keys stay in registers, so that the row is read from memory once and every radix digit runs on registers: 11, 11 and 10 bits
// of the raw key.  The first digit holds the sign, the exponent and two bits of mantissa, so scores of a row hit a few dozen of its 2048
// bins; eight copies of every bin side by side, one per lane modulo eight, keep the lanes of a wave off each other's words.  (8-bit
// digits of the key's distance from the row's smallest, a histogram per wave: 28 us of the kernel's 44 in the passes where scores change
// sign, since the positive ones then share two or three bins.)  Wave w owns the scores [w * seg, (w + 1) * seg),
// seg = 256 * ceil(length / 4096): a short row is one quad per thread in all waves, not 36 scores per thread in a few.
// What bounds it is the vector ALU (1 us per instruction and 150 000 keys of a CU), the loads, and the first digit's adds, which go with the making of
// the keys.  A wave waits for all of its loads before the first of them: there is a branch around each, so that the compiler cannot count
// them.  Later digits look at a quad's four keys with one comparison.
//
// TEAM = false: a workgroup per row of up to kTopkRegMax scores (QUADS = 9 per thread).
// (Its wait for the loads stands in front of the first barrier.)
//
// TEAM: longer rows, QUADS = 21, in parts, where all parts fit the chip at once, one workgroup per CU.  After counting a digit the workgroups
// of a row meet: each leaves its histogram in scratch memory, waits until all have, and adds them up by itself.  112 rows of
// 170 000 scores: 66.7 us as five launches that read the scores three times, 50.7 so (20 until the first digit is counted, 19 for the
// digits and their meetings, 10 for the write); 64 of 300 000 68.8 -> 51.7, 256 of 85 001 73.8 -> 51.5.
// The wait ends whatever else the device runs: a workgroup whose others have not come within `patience` ticks of the constant clock
// (another stream may hold their places) selects from the whole row by itself, every digit counted over the row as it
// lies in memory, and goes on leaving what the others wait for.  The workgroups of a row follow each other eight apart in the launch, which
// puts them on one XCD where workgroups go round the XCDs; nothing but the time depends on it.
// Scratch memory: 16 words per row (arrivals per digit at [0], [1], [2]), cleared by a launch in front, then three histograms of 2048
// words per part: one each, since a workgroup that goes on alone waits for nobody to have read the one before.
// ---------------------------------------------------------------------------------------------
constexpr int kTopkChunks = 9;                     // quads per thread
constexpr int kTopkRegMax = kTopkChunks * kChunk;
static_assert(kTopkRegMax == kTopkSingleMax, "kernels.hpp states the longest single-workgroup row");
// Rows of up to two and five quads per thread have kernels of their own: 47 and 62 registers instead of 75 let two workgroups share a CU,
// and a short row's has less code to fetch.  512 rows of 5000 / 20 000 scores 20.3 -> 17.4 and 31.6 -> 25.1 us, 256 of 2000 10.1 -> 9.6.
constexpr int kShortChunks = 2, kMidChunks = 5;
constexpr int kRegCopies = 8;

constexpr int kTeamQuads = 21, kTeamPartMax = kTeamQuads * kChunk;
// Workgroups in all, one per CU (what is left over would start when the first are done), and of a row; scores of a part and rows for which
// it pays: every workgroup reads the others' histograms, so fewer and longer parts meet faster, and with few rows most of the chip
// would wait either way.  Teams / five launches, us: 28 rows of 40 000 24.3 / 24.9, of 56 000 25.4 (28.1 in parts of 8192) / 25.7, 32 of 160 000
// 31.3 / 35.1, 64 of 100 000 31.1 / 35.7; 16 of 60 000 25.1 / 24.2, 24 of 60 000 25.5 / 24.8, 4 of 120 000 27.7 / 23.9.
constexpr int kTeamPlaces = 256, kTeamMost = 8, kTeamPartLeast = 16384, kTeamLeastRows = 28;
constexpr int kTeamGroup = 8;                        // rows whose workgroups alternate
constexpr int kTeamStateWords = 16, kTeamPartWords = 3 * 2048;

struct TeamArgs {
  int rows, parts, part_len;
  uint32_t* scratch;
  unsigned long long patience;
};

__global__ __launch_bounds__(256) void team_init_kernel(uint32_t* __restrict__ scratch, int words) {
  const int i = (int)blockIdx.x * 256 + threadIdx.x;
  if (i < words) scratch[i] = 0u;
}

// bits = 2 bits + (a > b), and with a == b
__device__ __forceinline__ void shift_in_above(uint32_t& bits, uint32_t a, uint32_t b) {
  asm("v_cmp_gt_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(a), "v"(b) : "vcc");
}
__device__ __forceinline__ void shift_in_equal(uint32_t& bits, uint32_t a, uint32_t b) {
  asm("v_cmp_eq_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(a), "v"(b) : "vcc");
}

// the thread's two bins, 2047 - 2 t and 2046 - 2 t, over the copies; clears them for the next digit, whose adds lie a barrier ahead
__device__ __forceinline__ void take_bins(uint32_t* hist, int tid, uint32_t (&cnt)[2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    u32x4* h = reinterpret_cast<u32x4*>(hist + (2047 - (tid * 2 + i)) * kRegCopies);
    const u32x4 a = h[0], b = h[1];
    h[0] = u32x4{0, 0, 0, 0};
    h[1] = u32x4{0, 0, 0, 0};
    cnt[i] = ((a[0] + a[1]) + (a[2] + a[3])) + ((b[0] + b[1]) + (b[2] + b[3]));
  }
}

// Ordered gather of the token rows a workgroup has just selected (the mask applied to the target's cache, Sec. 4.3):
// dst[j, :] = src[list[j], :] for j in [j_lo, j_hi), K and V together.  `list` was written by this workgroup before
// the barrier that precedes the call.  cpr = 16-byte chunks per token row.
struct GatherArgs {
  const u32x4* k_in;
  const u32x4* v_in;
  u32x4* k_out;
  u32x4* v_out;
  int cpr;
};
__device__ __forceinline__ void gather_rows(const GatherArgs& ga, size_t in_base, size_t out_base, const int32_t* list,
                                            int j_lo, int j_hi, int tid) {
  const int cpr = ga.cpr, tokens_per_step = kTopkThreads / cpr;
  const int ch = tid % cpr, tsub = tid / cpr;
  if (tsub >= tokens_per_step) return;
  constexpr int kU = 2;
  for (int j0 = j_lo + tsub; j0 < j_hi; j0 += kU * tokens_per_step) {
    u32x4 kv[kU], vv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int j = j0 + u * tokens_per_step;
      if (j < j_hi) {
        const size_t src = in_base + (size_t)list[j] * cpr + ch;
        kv[u] = __builtin_nontemporal_load(ga.k_in + src);
        vv[u] = __builtin_nontemporal_load(ga.v_in + src);
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int j = j0 + u * tokens_per_step;
      if (j < j_hi) {
        const size_t dst = out_base + (size_t)j * cpr + ch;
        __builtin_nontemporal_store(kv[u], ga.k_out + dst);
        __builtin_nontemporal_store(vv[u], ga.v_out + dst);
      }
    }
  }
}

template <int QUADS, bool TEAM, bool GATHER>
__global__ __launch_bounds__(kTopkThreads) void topk_reg_kernel(const float* __restrict__ scores, int N, int K, int32_t* __restrict__ idx_out,
                                                                GatherArgs ga, TeamArgs ta) {
  const int b = blockIdx.x, parts = TEAM ? ta.parts : 1;
  const int r = TEAM ? b / (kTeamGroup * parts) * kTeamGroup + b % kTeamGroup : b, part = TEAM ? b / kTeamGroup % parts : 0;
  if (TEAM && r >= ta.rows) return;
  const float* row = scores + (size_t)r * N;
  int32_t* out = idx_out + (size_t)r * K;
  uint32_t* state = TEAM ? ta.scratch + (size_t)r * kTeamStateWords : nullptr;
  uint32_t* team = TEAM ? ta.scratch + (size_t)ta.rows * kTeamStateWords + (size_t)r * parts * kTeamPartWords : nullptr;
  __shared__ __attribute__((aligned(16))) uint32_t hist[2048 * kRegCopies];
  __shared__ uint32_t wave_part[kTopkWaves], wave_eq[kTopkWaves];
  __shared__ uint32_t s_prefix, s_krem, s_came;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lo = TEAM ? part * ta.part_len : 0, len = TEAM && N - lo > ta.part_len ? ta.part_len : N - lo;
  const int seg = (len + kChunk - 1) / kChunk * 256, s0 = wave * seg;
  const int left = len - s0 < seg ? len - s0 : seg, quads = left > 0 ? (left + 255) / 256 : 0;  // the wave's scores, and quads per lane
  const int i0 = s0 + 4 * lane;  // index in the part of the thread's first quad; the next ones follow 256 apart

  // keys of this thread's scores; those at and past the end hold a key that no score has (the largest, +inf's, is 0xff800000)
  constexpr uint32_t kNoKey = 0xffffffffu;
  // (Of 21 quads per thread 16 are meant for registers and five go to LDS; all 21 in registers, 48 of the 128 were spilled.  So it is 40 still: one quad, and
  // what only the wait needs, lie in 20 bytes of scratch memory per lane, written once and read again for each later digit and the write.  112 rows of
  // 170 000 scores write 32.2 MB, of which indices and histograms are 28.4.)
  constexpr int kRegQuads = QUADS < 16 ? QUADS : 16;
  __shared__ u32x4 stash[QUADS > kRegQuads ? (QUADS - kRegQuads) * kTopkThreads : 1];
  uint32_t reg_key[kRegQuads][4];
  auto set_quad = [&](int c, const u32x4& k) __attribute__((always_inline)) {
    if (c < kRegQuads) {
#pragma unroll
      for (int j = 0; j < 4; ++j) reg_key[c][j] = k[j];
    } else {
      stash[(c - kRegQuads) * kTopkThreads + tid] = k;
    }
  };
  auto quad = [&](int c) __attribute__((always_inline)) {
    return c < kRegQuads ? u32x4{reg_key[c][0], reg_key[c][1], reg_key[c][2], reg_key[c][3]} : stash[(c - kRegQuads) * kTopkThreads + tid];
  };
  f32x4 v[QUADS];
  if (!TEAM && N < 4) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[0][j] = row[j < N ? j : 0];
  } else {
#pragma unroll
    for (int c = 0; c < QUADS; ++c)
      if (c < quads) v[c] = load_quad(row + lo, i0 + c * 256, len);
  }
#pragma unroll
  for (int i = 0; i < 2048 * kRegCopies / 4 / kTopkThreads; ++i) reinterpret_cast<u32x4*>(hist)[tid + i * kTopkThreads] = u32x4{0, 0, 0, 0};
  // (a barrier that need not wait for the scores; in the team's kernel alone it does not)
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

  uint32_t* mine = hist + (lane & (kRegCopies - 1));
  // the first digit's adds go with the keys
#pragma unroll
  for (int c = 0; c < QUADS; ++c)
    if (c < quads) {
      u32x4 k;
      if (left >= (c + 1) * 256) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          k[j] = order_key(v[c][j]);
          atomicAdd(&mine[(k[j] >> 21) * kRegCopies], 1u);
        }
      } else {
        if (TEAM || N >= 4) v[c] = shift_quad(v[c], quad_shift(i0 + c * 256, len));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool is = i0 + c * 256 + j < len;
          k[j] = is ? order_key(v[c][j]) : kNoKey;
          if (is) atomicAdd(&mine[(k[j] >> 21) * kRegCopies], 1u);
        }
      }
      set_quad(c, k);
    }

  uint32_t prefix = 0, krem = (uint32_t)K;
  uint32_t g = 0, e = 0;  // of the parts in front: keys above T, and equal to it (summed over threads)
  bool alone = false;
  uint32_t alone_T = 0, alone_take = 0;
#pragma unroll 1
  for (int digit = 0; digit < 3; ++digit) {  // rolled, like everything that runs once per wave
    const int shift = digit == 0 ? 21 : (digit == 1 ? 10 : 0), bits = digit == 2 ? 10 : 11;
    if (digit > 0) {
      const uint32_t from = prefix << (shift + bits), span = 1u << (shift + bits);
#pragma unroll
      for (int c = 0; c < QUADS; ++c)
        if (c < quads) {
          const u32x4 t = quad(c) - from;
          const uint32_t a = t[0] < t[1] ? t[0] : t[1], z = t[2] < t[3] ? t[2] : t[3];
          if ((a < z ? a : z) < span) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (t[j] < span) atomicAdd(&mine[(t[j] >> shift) * kRegCopies], 1u);
          }
        }
    }
    __syncthreads();
    uint32_t cnt[2], front[2] = {0, 0};
    take_bins(hist, tid, cnt);
    if constexpr (TEAM) {
      uint64_t* own = reinterpret_cast<uint64_t*>(team + (size_t)part * kTeamPartWords + digit * 2048);
      __hip_atomic_store(own + tid, (uint64_t)cnt[1] << 32 | cnt[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // every wave's words are where all meet before the arrival counts (see mw_pass_kernel)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) {
        atomicAdd(&state[digit], 1u);
        uint32_t came = 1;
        if (!alone) {
          const unsigned long long start = __builtin_amdgcn_s_memrealtime();
          while (__hip_atomic_load(&state[digit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)parts) {
            if (__builtin_amdgcn_s_memrealtime() - start >= ta.patience) {
              came = 0;
              break;
            }
            __builtin_amdgcn_s_sleep(1);
          }
        }
        s_came = came;
      }
      __syncthreads();
      if (!alone && !s_came) {
        alone = true;
        alone_take = (uint32_t)K;
        g = e = 0;  // what the digits before gave is counted again below
#pragma unroll 1
        for (int d = 0; d < 3; ++d) {
          const int sh = d == 0 ? 21 : (d == 1 ? 10 : 0), n = d == 2 ? 10 : 11;
          for (int i = tid; i < N; i += kTopkThreads) {
            const uint32_t k = order_key(row[i]);
            if (d == 0 || k >> ((sh + n) & 31) == alone_T) atomicAdd(&mine[((k >> sh) & ((1u << n) - 1u)) * kRegCopies], 1u);
          }
          __syncthreads();
          uint32_t all[2];
          take_bins(hist, tid, all);
          pick_digit<2048, 2>(all, alone_take, wave_part, tid, [&](uint32_t found, uint32_t rest, uint32_t) {
            s_prefix = alone_T << n | found;
            s_krem = rest;
          });
          __syncthreads();
          alone_T = s_prefix;
          alone_take = s_krem;
          __syncthreads();
        }
      }
      if (alone) {
        prefix = alone_T >> shift;
        krem = alone_take;
        continue;
      }
      for (int q = 0; q < parts; ++q) {
        if (q == part) continue;
        const uint64_t* theirs = reinterpret_cast<const uint64_t*>(team + (size_t)q * kTeamPartWords + digit * 2048);
        const uint64_t two = __hip_atomic_load(theirs + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        cnt[0] += (uint32_t)two;
        cnt[1] += (uint32_t)(two >> 32);
        front[0] += q < part ? (uint32_t)two : 0u;
        front[1] += q < part ? (uint32_t)(two >> 32) : 0u;
      }
    }
    pick_digit<2048, 2>(cnt, krem, wave_part, tid, [&](uint32_t d, uint32_t rest, uint32_t) {
      s_prefix = prefix << bits | d;
      s_krem = rest;
    });
    __syncthreads();
    prefix = s_prefix;
    krem = s_krem;
    if constexpr (TEAM) {
      const int d = (int)(prefix & ((1u << bits) - 1u));
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int bin = 2047 - (tid * 2 + i);
        g += bin > d ? front[i] : 0u;
        if (digit == 2) e += bin == d ? front[i] : 0u;
      }
    }
  }
  const uint32_t T = prefix, eq_take = krem;

  // kept: keys above T, and the eq_take lowest-index keys equal to T; eight quads' bits to a word, the first key's lowest
  constexpr int kWords = (QUADS + 7) / 8;
  uint32_t m_gt[kWords], m_eq[kWords], n_gt = 0, n_eq = 0;
#pragma unroll
  for (int w = 0; w < kWords; ++w) {
    m_gt[w] = m_eq[w] = 0;
#pragma unroll
    for (int c = 8 * w; c < 8 * w + 8; ++c) {
      uint32_t above = 0, equal = 0;
      if (c < QUADS && c < quads) {
        const u32x4 k = quad(c);
#pragma unroll
        for (int j = 3; j >= 0; --j) {
          shift_in_above(above, k[j], T);
          shift_in_equal(equal, k[j], T);
        }
        if (left < (c + 1) * 256) {
          const int n = len - (i0 + c * 256);
          above &= n >= 4 ? 15u : (n > 0 ? (1u << n) - 1u : 0u);
        }
      }
      m_gt[w] |= above << (4 * (c % 8));
      m_eq[w] |= equal << (4 * (c % 8));
    }
    n_gt += (uint32_t)__popc(m_gt[w]);
    n_eq += (uint32_t)__popc(m_eq[w]);
  }
  n_gt = wave_total(n_gt);
  n_eq = wave_total(n_eq);
  uint32_t gt = 0, eq = 0;  // in front of the wave's scores
  if constexpr (TEAM) {
    if (alone) {
      for (int i = tid; i < lo; i += kTopkThreads) {
        const uint32_t k = order_key(row[i]);
        g += k > T;
        e += k == T;
      }
    }
    __syncthreads();
    gt = block_sum(g, wave_part, tid);
    eq = block_sum(e, wave_part, tid);
  }
  if (lane == 0) {
    wave_part[wave] = n_gt;
    wave_eq[wave] = n_eq;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kTopkWaves; ++w) {
    gt += w < wave ? wave_part[w] : 0u;
    eq += w < wave ? wave_eq[w] : 0u;
  }
  static_assert(2048 * kRegCopies >= kTopkWaves * kStageWords, "the histogram's place");
  wave_write(m_gt, m_eq, quads, gt, eq, eq_take, lo + s0, lane, reinterpret_cast<int32_t*>(hist) + wave * kStageWords, out);
  if constexpr (GATHER) {
    __syncthreads();  // the row's list is complete and visible to the whole workgroup
    gather_rows(ga, (size_t)r * N * ga.cpr, (size_t)r * K * ga.cpr, out, 0, K, tid);
  }
}

// ---------------------------------------------------------------------------------------------
// Rows longer than kTopkRegMax are cut into parts of at most kMwPartMax = 45 056 scores, one workgroup each.
// Scratch memory per row (32-bit words), B = 2^BITS bins, P passes:
//   [0, 16)                          state: prefix, krem, the keys under the last pass's prefix, then one arrival counter per pass at
//                                    [4 + pass]
//   [16, 16 + P * B)                 the row's histogram of every pass
//   [16 + P * B, ... )               per part, for every digit of the last pass and one past them: its number of keys under
//                                    the prefix with at least that digit plus its keys above the prefix
// and behind all rows, where there is room, two 64-bit masks per thread of every part: its scores above the prefix and under it.
// mw_init_kernel clears the first 16 + P * B words of every row; the per-part words are all written by the last pass.
// A pass takes the next BITS bits of the keys whose higher bits equal the prefix found so far; the workgroup that arrives
// last at the row's counter has every part's contribution in the row's histogram and picks the bin that holds the krem-th
// largest key.
// Eleven bits: three passes instead of four, and the first digit (sign, exponent, two bits of mantissa) spreads scores
// that share an exponent over four bins.  112 rows of 170 000 scores: 67 us in all, with 8 bits and scores read by thread 222 us.
// ---------------------------------------------------------------------------------------------
constexpr int kMwQuads = 11, kMwPartMax = kMwQuads * 256 * kTopkWaves;  // quads per lane and scores per part
constexpr int kMwStateWords = 16;

template <int BITS>
struct Mw {
  static constexpr int kBins = 1 << BITS;
  static constexpr int kPasses = (32 + BITS - 1) / BITS;
  static constexpr int kLastBits = 32 - (kPasses - 1) * BITS;
  static constexpr int kFixedWords = kMwStateWords + kPasses * kBins;
  static constexpr int kPartWords = (1 << kLastBits) + 1;
  // Copies of the LDS histogram, one per lane modulo kCopies and side by side, so that lanes that hit one bin (scores of
  // a row share sign and exponent) hit different words and banks.
  static constexpr int kCopies = BITS == 8 ? 16 : 8;
};

// bits = 2 bits + (f > t), and with f >= t: false for NaN
__device__ __forceinline__ void shift_in_gt(uint32_t& bits, float f, float t) {
  asm("v_cmp_gt_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(f), "v"(t) : "vcc");
}
__device__ __forceinline__ void shift_in_ge(uint32_t& bits, float f, float t) {
  asm("v_cmp_ge_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(f), "v"(t) : "vcc");
}

// Wave w owns the scores [s0, s1) of its part of `len`, at most kMwQuads quads per lane.
struct WaveSpan {
  int s0, s1, quads;
};
__device__ __forceinline__ WaveSpan wave_span(int len, int wave) {
  const int seg = ((len + kTopkWaves - 1) / kTopkWaves + 255) & ~255;
  const int s0 = wave * seg < len ? wave * seg : len, s1 = s0 + seg < len ? s0 + seg : len;
  return {s0, s1, (s1 - s0 + 255) / 256};
}

// Whether the last pass leaves two bits per score for mw_write_kernel: where there is room for them, where few keys of the row lie
// under its prefix (each is looked up on its own, and rows with many scores nearly the same have many), and where that bin is an
// interval of numbers: not with infinities or NaN in it, or the key of -0.0 at its end, which no score has.
constexpr uint32_t kFewKeys = 1024;
template <int BITS>
__device__ __forceinline__ bool by_bits(const u32x4* masks, uint32_t n_keys, uint32_t prefix) {
  const uint32_t k_lo = prefix << Mw<BITS>::kLastBits, k_hi = k_lo | ((1u << Mw<BITS>::kLastBits) - 1u);
  return masks != nullptr && n_keys <= kFewKeys && k_lo >= 0x00800000u && k_hi < 0xff800000u && k_hi != 0x7fffffffu;
}

template <int BITS>
__global__ void mw_init_kernel(uint32_t* __restrict__ scratch, int rows, int row_words, int K) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)rows * Mw<BITS>::kFixedWords) return;
  const int r = (int)(gid / Mw<BITS>::kFixedWords), w = (int)(gid % Mw<BITS>::kFixedWords);
  scratch[(size_t)r * row_words + w] = (w == 1) ? (uint32_t)K : 0u;  // word 0: prefix, word 1: krem
}

// grid (parts, rows)
template <int BITS, int PASS>
__global__ __launch_bounds__(kTopkThreads) void mw_pass_kernel(const float* __restrict__ scores, int N, int part_len,
                                                               uint32_t* __restrict__ scratch, int row_words, u32x4* __restrict__ masks) {
  using C = Mw<BITS>;
  constexpr int kHi = 32 - BITS * PASS, kShift = kHi > BITS ? kHi - BITS : 0, kDigitBins = 1 << (kHi - kShift);
  constexpr bool kLast = PASS == C::kPasses - 1;
  const int part = blockIdx.x, parts = gridDim.x, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const float* row = scores + (size_t)blockIdx.y * N;
  uint32_t* rs = scratch + (size_t)blockIdx.y * row_words;
  uint32_t* row_hist = rs + kMwStateWords + PASS * C::kBins;
  __shared__ __attribute__((aligned(16))) uint32_t hist[C::kBins * C::kCopies];
  __shared__ uint32_t wave_part[kTopkWaves];
  __shared__ uint32_t s_last;
  const int lo = part * part_len, len = N - lo < part_len ? N - lo : part_len;
  row += lo;
  const uint32_t prefix = rs[0];  // the bits above kHi of the K-th largest key (written by the previous launch)
  for (int i = tid; i < C::kBins * C::kCopies / 4; i += kTopkThreads) reinterpret_cast<u32x4*>(hist)[i] = u32x4{0, 0, 0, 0};
  __syncthreads();
  uint32_t n_hi = 0;  // last pass: keys above the prefix
  uint32_t* mine = hist + (lane & (C::kCopies - 1));
  if (kLast && by_bits<BITS>(masks, rs[2], prefix)) {
    // Two comparisons per score and a bit each, in the order of mw_write_kernel, which takes them from `masks`; the few keys under the
    // prefix are counted afterwards.  (With keys and the histogram's adds in the loop this pass is bound by the vector ALU: 112 rows
    // of 170 000 scores 24 us, so 20.5.)
    const WaveSpan w = wave_span(len, wave);
    uint64_t m_hi = 0, m_in = 0;  // keys above the prefix, and under it
    const float f_lo = key_score(prefix << kHi), f_hi = key_score(prefix << kHi | ((1u << kHi) - 1u));
    constexpr int kFly = 6;  // quads in flight
#pragma unroll 1
    for (int q0 = 0; q0 < w.quads; q0 += kFly) {
      f32x4 v[kFly];
#pragma unroll
      for (int u = 0; u < kFly; ++u) v[u] = load_quad(row, w.s0 + (q0 + u) * 256 + 4 * lane, w.s1);
      uint32_t above = 0, from = 0, valid = ~0u;  // four bits a quad, the first score's the highest
      if (w.s0 + (q0 + kFly) * 256 > w.s1) {
        valid = 0;
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
          const int i = w.s0 + (q0 + u) * 256 + 4 * lane, n = w.s1 - i;
          v[u] = shift_quad(v[u], quad_shift(i, w.s1));
          valid |= (n >= 4 ? 15u : (n > 0 ? (1u << n) - 1u : 0u)) << (4 * u);
        }
      }
#pragma unroll
      for (int u = 0; u < kFly; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          shift_in_gt(above, v[u][j], f_hi);
          shift_in_ge(from, v[u][j], f_lo);
        }
      above = __brev(above) >> (32 - 4 * kFly);
      from = __brev(from) >> (32 - 4 * kFly);
      m_hi |= (uint64_t)(above & valid) << (4 * q0);
      m_in |= (uint64_t)(from & ~above & valid) << (4 * q0);
    }
    n_hi = (uint32_t)__popcll(m_hi);
    masks[((size_t)blockIdx.y * parts + part) * kTopkThreads + tid] =
        u32x4{(uint32_t)m_hi, (uint32_t)(m_hi >> 32), (uint32_t)m_in, (uint32_t)(m_in >> 32)};
    for (; __builtin_amdgcn_ballot_w64(m_in != 0); m_in &= m_in - 1)
      if (m_in != 0) {
        const int bit = __ffsll((unsigned long long)m_in) - 1;
        const uint32_t key = order_key(row[w.s0 + (bit >> 2) * 256 + 4 * lane + (bit & 3)]);
        atomicAdd(&mine[((key >> kShift) & (kDigitBins - 1)) * C::kCopies], 1u);
      }
  } else {
    for (int c0 = 0; c0 < len; c0 += 4 * kChunk) {  // four chunks in flight
      f32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = load_quad(row, c0 + u * kChunk + 4 * tid, len);
      auto count = [&](bool valid, float f) {
        const uint32_t key = order_key(f);
        if constexpr (PASS == 0) {
          if (valid) atomicAdd(&mine[(key >> kShift) * C::kCopies], 1u);
        } else {
          const uint32_t top = key >> (kHi & 31);
          if (valid && top == prefix) atomicAdd(&mine[((key >> kShift) & (kDigitBins - 1)) * C::kCopies], 1u);
          if (kLast) n_hi += valid && top > prefix;
        }
      };
      if (c0 + 4 * kChunk <= len) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j) count(true, v[u][j]);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j) count(j >= quad_shift(c0 + u * kChunk + 4 * tid, len), v[u][j]);
      }
    }
  }
  __syncthreads();
  // thread t holds bins kDigitBins - 1 - t, ... (descending)
  uint32_t n_hi_all = 0;
  if (kLast) n_hi_all = block_sum(n_hi, wave_part, tid);
  uint32_t last_sum = 0;
  for (int t = tid; t < kDigitBins; t += kTopkThreads) {
    const int b = kDigitBins - 1 - t;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < C::kCopies; i += 4) {
      const u32x4 h = *reinterpret_cast<const u32x4*>(hist + b * C::kCopies + i);
      sum += (h[0] + h[1]) + (h[2] + h[3]);
    }
    if (sum) atomicAdd(&row_hist[b], sum);
    last_sum = sum;  // the last pass has at most one bin per thread
  }
  if constexpr (kLast) {
    static_assert(kDigitBins <= kTopkThreads, "one bin per thread");
    const uint32_t at_or_above = n_hi_all + last_sum + block_exclusive_scan(last_sum, wave_part, wave, lane);
    uint32_t* part_words = rs + C::kFixedWords + (size_t)part * C::kPartWords;
    if (tid < kDigitBins) part_words[kDigitBins - 1 - tid] = at_or_above;
    if (tid == 0) part_words[kDigitBins] = n_hi_all;
  }
  // This part's bins must be in the row's histogram before its ticket is taken.  The adds are device-scope atomics, carried out
  // where all workgroups meet, but nothing orders them before the ticket, which is an add to another address: a barrier does
  // not wait for memory operations under way.  So every wave waits until its own adds have been acknowledged, then the
  // workgroup meets.  (A device-wide fence instead writes back the whole L2 per workgroup: 200 us per launch at 560 groups.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) s_last = (atomicAdd(&rs[4 + PASS], 1u) == (uint32_t)(parts - 1));
  __syncthreads();
  if (!s_last) return;
  // the bins in descending order, kPer per thread, read where the adds met
  constexpr int kPer = kDigitBins > kTopkThreads ? kDigitBins / kTopkThreads : 1;
  uint32_t cnt[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    cnt[i] = tid * kPer < kDigitBins ? atomicAdd(&row_hist[kDigitBins - 1 - (tid * kPer + i)], 0u) : 0u;
  const uint32_t krem = rs[1];
  // (pick_digit's barriers lie between this read and the write)
  pick_digit<kDigitBins, kPer>(cnt, krem, wave_part, tid, [&](uint32_t d, uint32_t left, uint32_t n) {
    rs[0] = (PASS == 0 ? 0u : prefix << (kHi - kShift)) | d;
    rs[1] = left;
    if (PASS == C::kPasses - 2) rs[2] = n;
  });
}

// grid (parts, rows): rs[0] is the K-th largest key T, rs[1] the number of keys equal to T that are kept (lowest
// index first).  A part's first output slot follows from two words of every part before it.
template <int BITS, bool GATHER>
__global__ __launch_bounds__(kTopkThreads, 8) void mw_write_kernel(const float* __restrict__ scores, int N, int K, int part_len,
                                                                const uint32_t* __restrict__ scratch, int row_words,
                                                                const u32x4* __restrict__ masks, int32_t* __restrict__ idx_out,
                                                                GatherArgs ga) {
  using C = Mw<BITS>;
  constexpr int kDigitBins = 1 << C::kLastBits;
  const int part = blockIdx.x, tid = threadIdx.x;
  const float* row = scores + (size_t)blockIdx.y * N;
  const uint32_t* rs = scratch + (size_t)blockIdx.y * row_words;
  int32_t* out = idx_out + (size_t)blockIdx.y * K;
  __shared__ uint32_t wave_part[kTopkWaves], wave_eq[kTopkWaves];
  __shared__ __attribute__((aligned(16))) int32_t stage[kTopkWaves * kStageWords];
  const int lo = part * part_len, len = N - lo < part_len ? N - lo : part_len;
  row += lo;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const WaveSpan w = wave_span(len, wave);
  const int s0 = w.s0, s1 = w.s1, quads = w.quads;
  const uint32_t T = rs[0], eq_take = rs[1], t_last = T & (kDigitBins - 1);
  // keys above T and keys equal to T in the parts before this one
  uint32_t g = 0, e = 0;
  for (int q = tid; q < part; q += kTopkThreads) {
    const uint32_t* pw = rs + C::kFixedWords + (size_t)q * C::kPartWords + t_last;
    g += pw[1];
    e += pw[0] - pw[1];
  }
  const uint32_t gt_before = block_sum(g, wave_part, tid), eq_before = block_sum(e, wave_part, tid);
  const float t = key_score(T);
  const bool nan_t = T == 0;
  uint64_t m_gt = 0, m_eq = 0;
  if (by_bits<BITS>(masks, rs[2], T >> C::kLastBits)) {
    const u32x4 m = masks[((size_t)blockIdx.y * gridDim.x + part) * kTopkThreads + tid];
    m_gt = (uint64_t)m[1] << 32 | m[0];
    // keys that agree with T in all but the last digit
    for (uint64_t m_in = (uint64_t)m[3] << 32 | m[2]; __builtin_amdgcn_ballot_w64(m_in != 0); m_in &= m_in - 1)
      if (m_in != 0) {
        const int bit = __ffsll((unsigned long long)m_in) - 1;
        const float f = row[s0 + (bit >> 2) * 256 + 4 * lane + (bit & 3)];
        m_gt |= (uint64_t)(f > t) << bit;
        m_eq |= (uint64_t)(f == t) << bit;
      }
  } else {
#pragma unroll 1
    for (int q0 = 0; q0 < quads; q0 += 4) {
      f32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = load_quad(row, s0 + (q0 + u) * 256 + 4 * lane, s1);
      const bool cut = s0 + (q0 + 4) * 256 > s1;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (cut) v[u] = shift_quad(v[u], quad_shift(s0 + (q0 + u) * 256 + 4 * lane, s1));
        uint32_t bg, be;
        quad_bits(v[u], s1 - (s0 + (q0 + u) * 256 + 4 * lane), t, nan_t, bg, be);
        m_gt |= (uint64_t)bg << (4 * (q0 + u));
        m_eq |= (uint64_t)be << (4 * (q0 + u));
      }
    }
  }
  const uint32_t n_gt = wave_total((uint32_t)__popcll(m_gt)), n_eq = wave_total((uint32_t)__popcll(m_eq));
  if (lane == 0) {
    wave_part[wave] = n_gt;
    wave_eq[wave] = n_eq;
  }
  __syncthreads();
  uint32_t gt = gt_before, eq = eq_before, gt_end = gt_before, eq_end = eq_before;
#pragma unroll
  for (int w = 0; w < kTopkWaves; ++w) {
    const uint32_t a = wave_part[w], b = wave_eq[w];
    gt += w < wave ? a : 0u;
    eq += w < wave ? b : 0u;
    gt_end += a;
    eq_end += b;
  }
  const uint32_t w_gt[2] = {(uint32_t)m_gt, (uint32_t)(m_gt >> 32)}, w_eq[2] = {(uint32_t)m_eq, (uint32_t)(m_eq >> 32)};
  wave_write(w_gt, w_eq, quads, gt, eq, eq_take, lo + s0, lane, stage + wave * kStageWords, out);
  if constexpr (GATHER) {
    __syncthreads();  // this part's stretch of the list is complete and visible to the whole workgroup
    gather_rows(ga, (size_t)blockIdx.y * N * ga.cpr, (size_t)blockIdx.y * K * ga.cpr, out,
                (int)(gt_before + (eq_before < eq_take ? eq_before : eq_take)),
                (int)(gt_end + (eq_end < eq_take ? eq_end : eq_take)), tid);
  }
}

// Parts of a row for the register kernel's teams: as many as the chip has places for, none longer than its registers take; 0 where there are not
// places enough.
static int team_parts(int64_t rows, int64_t N) {
  const int64_t least = (N + kTeamPartMax - 1) / kTeamPartMax;
  if (rows < kTeamLeastRows || rows * least > kTeamPlaces || least > kTeamMost) return 0;
  int64_t parts = kTeamPlaces / rows;
  const int64_t most = (N + kTeamPartLeast - 1) / kTeamPartLeast;
  if (parts > most) parts = most;
  if (parts > kTeamMost) parts = kTeamMost;
  return (int)(parts > least ? parts : least);
}
static size_t team_scratch(int64_t rows, int parts) { return (size_t)rows * (kTeamStateWords + (size_t)parts * kTeamPartWords) * 4; }

}  // namespace

// Parts of a row that is too long for one register-resident workgroup.  With 8 bits as few as there can be (the caller's
// scratch memory is short); with 11 as many as give 512 workgroups, two per CU, of at least 8192 scores.
template <int BITS>
static int topk_parts(int64_t rows, int64_t N) {
  const int64_t least = (N + kMwPartMax - 1) / kMwPartMax;
  if (BITS == 8) return (int)least;
  const int64_t most = (N + 8191) / 8192, want = 512 / rows < most ? 512 / rows : most;
  return (int)(want > least ? want : least);
}
template <int BITS>
static size_t topk_scratch(int64_t rows, int64_t N) {
  if (N <= kTopkRegMax || rows <= 0) return 0;
  return (size_t)rows * (size_t)(Mw<BITS>::kFixedWords + (size_t)topk_parts<BITS>(rows, N) * Mw<BITS>::kPartWords) * 4;
}
constexpr size_t kMaskBytes = kTopkThreads * 16;  // of a part: four words per thread
// (the parts of up to `rows` rows of up to N scores: 512, or as few as each row can have; the masks start on a 16-byte boundary)
static size_t topk_most_parts(int64_t rows, int64_t N) {
  const size_t least = (size_t)rows * (size_t)((N + kMwPartMax - 1) / kMwPartMax);
  return least > 512 ? least : 512;
}
size_t topk_scratch_bytes_no_masks(int64_t rows, int64_t N) {
  if (N <= kTopkRegMax || rows <= 0) return 0;
  return ((size_t)rows * Mw<11>::kFixedWords + topk_most_parts(rows, N) * Mw<11>::kPartWords) * 4;
}
size_t topk_scratch_bytes(int64_t rows, int64_t N) {
  if (N <= kTopkRegMax || rows <= 0) return 0;
  return topk_scratch_bytes_no_masks(rows, N) + 16 + topk_most_parts(rows, N) * kMaskBytes;
}
size_t topk_scratch_bytes_least(int64_t rows, int64_t N) { return topk_scratch<8>(rows, N); }

template <int BITS>
static hipError_t launch_topk_split(const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out, void* scratch,
                                    size_t scratch_bytes, const GatherArgs* gather, hipStream_t stream) {
  using C = Mw<BITS>;
  const GatherArgs none = {nullptr, nullptr, nullptr, nullptr, 0};
  // parts of equal length, a multiple of four scores (16-byte loads when the row itself is aligned), none of them empty
  const int most_parts = topk_parts<BITS>(rows, N);
  const int part_len = (int)((((N + most_parts - 1) / most_parts) + 3) & ~(int64_t)3);
  const int parts = (int)((N + part_len - 1) / part_len);
  const int row_words = C::kFixedWords + parts * C::kPartWords;
  uint32_t* sc = (uint32_t*)scratch;
  // What the last pass finds about every score, two bits each, saves the kernel behind it from reading the scores (112 rows of
  // 170 000: that one 28 -> 16 us, the last pass 17 -> 20.5, all 78 -> 67; 4 rows of 262 144, in 64 parts each, 26.4 -> 25.3); where the
  // scratch memory does not hold it, the scores are read a fourth time.
  const size_t mask_at = ((size_t)rows * row_words * 4 + 15) & ~(size_t)15;
  u32x4* masks = BITS == 11 && mask_at + (size_t)(rows * parts) * kMaskBytes <= scratch_bytes ? (u32x4*)((uint8_t*)scratch + mask_at) : nullptr;
  const int64_t init_words = rows * C::kFixedWords;
  mw_init_kernel<BITS><<<(unsigned)((init_words + 255) / 256), 256, 0, stream>>>(sc, (int)rows, row_words, (int)K);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)parts, (unsigned)rows);
  mw_pass_kernel<BITS, 0><<<grid, kTopkThreads, 0, stream>>>(scores, (int)N, part_len, sc, row_words, masks);
  mw_pass_kernel<BITS, 1><<<grid, kTopkThreads, 0, stream>>>(scores, (int)N, part_len, sc, row_words, masks);
  mw_pass_kernel<BITS, 2><<<grid, kTopkThreads, 0, stream>>>(scores, (int)N, part_len, sc, row_words, masks);
  if constexpr (C::kPasses > 3) mw_pass_kernel<BITS, 3><<<grid, kTopkThreads, 0, stream>>>(scores, (int)N, part_len, sc, row_words, masks);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (gather) mw_write_kernel<BITS, true><<<grid, kTopkThreads, 0, stream>>>(scores, (int)N, (int)K, part_len, sc, row_words, masks, idx_out, *gather);
  else mw_write_kernel<BITS, false><<<grid, kTopkThreads, 0, stream>>>(scores, (int)N, (int)K, part_len, sc, row_words, masks, idx_out, none);
  return hipGetLastError();
}

static hipError_t launch_topk_team(const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out, void* scratch, int most_parts,
                                   unsigned long long patience, hipStream_t stream) {
  const int part_len = (int)((((N + most_parts - 1) / most_parts) + 3) & ~(int64_t)3);
  const int parts = (int)((N + part_len - 1) / part_len);
  const int words = (int)rows * kTeamStateWords;
  team_init_kernel<<<(unsigned)((words + 255) / 256), 256, 0, stream>>>((uint32_t*)scratch, words);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const GatherArgs none = {nullptr, nullptr, nullptr, nullptr, 0};
  const TeamArgs ta = {(int)rows, parts, part_len, (uint32_t*)scratch, patience};
  topk_reg_kernel<kTeamQuads, true, false><<<(unsigned)((rows + kTeamGroup - 1) / kTeamGroup * kTeamGroup * parts), kTopkThreads, 0, stream>>>(
      scores, (int)N, (int)K, idx_out, none, ta);
  return hipGetLastError();
}

// gather != nullptr: every workgroup also gathers the token rows it selected (k/v in [rows, N, row_bytes], out [rows, K, row_bytes])
static hipError_t launch_topk_impl(const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out, void* scratch,
                                   size_t scratch_bytes, const GatherArgs* gather, unsigned long long patience, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (N <= kTopkRegMax) {
    const GatherArgs none = {nullptr, nullptr, nullptr, nullptr, 0};
    const TeamArgs no_team = {0, 1, 0, nullptr, 0};
    if (gather) topk_reg_kernel<kTopkChunks, false, true><<<dim3((unsigned)rows), kTopkThreads, 0, stream>>>(scores, (int)N, (int)K, idx_out, *gather, no_team);
    else if (N <= kShortChunks * kChunk) topk_reg_kernel<kShortChunks, false, false><<<dim3((unsigned)rows), kTopkThreads, 0, stream>>>(scores, (int)N, (int)K, idx_out, none, no_team);
    else if (N <= kMidChunks * kChunk) topk_reg_kernel<kMidChunks, false, false><<<dim3((unsigned)rows), kTopkThreads, 0, stream>>>(scores, (int)N, (int)K, idx_out, none, no_team);
    else topk_reg_kernel<kTopkChunks, false, false><<<dim3((unsigned)rows), kTopkThreads, 0, stream>>>(scores, (int)N, (int)K, idx_out, none, no_team);
    return hipGetLastError();
  }
  if (scratch == nullptr || rows > 65535) return hipErrorInvalidValue;
  if (!gather) {
    const int want = team_parts(rows, N);
    if (want > 0 && scratch_bytes >= team_scratch(rows, want)) return launch_topk_team(scores, rows, N, K, idx_out, scratch, want, patience, stream);
  }
  if (scratch_bytes >= topk_scratch<11>(rows, N)) return launch_topk_split<11>(scores, rows, N, K, idx_out, scratch, scratch_bytes, gather, stream);
  if (scratch_bytes >= topk_scratch<8>(rows, N)) return launch_topk_split<8>(scores, rows, N, K, idx_out, scratch, scratch_bytes, gather, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_topk(const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out, void* scratch,
                       size_t scratch_bytes, hipStream_t stream, unsigned long long patience) {
  return launch_topk_impl(scores, rows, N, K, idx_out, scratch, scratch_bytes, nullptr, patience, stream);
}

hipError_t launch_topk_gather(const float* scores, int64_t rows, int64_t N, int64_t K, int32_t* idx_out, void* scratch,
                              size_t scratch_bytes, const void* k_in, const void* v_in, int64_t row_bytes, void* k_out, void* v_out,
                              hipStream_t stream) {
  const GatherArgs ga = {(const u32x4*)k_in, (const u32x4*)v_in, (u32x4*)k_out, (u32x4*)v_out, (int)(row_bytes / 16)};
  if (ga.cpr < 1 || ga.cpr > kTopkThreads || kTopkThreads % ga.cpr != 0) return hipErrorInvalidValue;
  return launch_topk_impl(scores, rows, N, K, idx_out, scratch, scratch_bytes, &ga, kTopkPatience, stream);
}

}  // namespace pkv
