// The encoder of the large-tile mapper, everything but the attention: out-projection, residual, LayerNorm, both FFN products, residual,
// LayerNorm and the next layer's q, k and v in one launch per layer.  (The first launch has only q, k and v, the last no q, k and v.)
//
// A workgroup takes a block of 128 rows through all of it.  As separate products (256 x 256 and 128 x 512 tiles, normalised rows
// and hidden rows through memory) a layer moved 28 times the 1 KB of an fp16 row, as here with the attention 12 times; and those kernels
// stood in waits of one workgroup per CU 28 to 42 % of the time: 126 976 rows took 1117 us per layer beside the attention.
//
// Four waves, one per SIMD, each with all 512 registers of a lane.  The block's operand (attention output, then normalised rows) lies
// in LDS, 128 KB, in the order in which MFMA fragments are read.  Every wave owns a quarter of each product's features, so it needs
// weights that no other wave of the workgroup reads: they come from L2 straight into registers, in the order of their use, eight
// fragments ahead, and never through LDS (16 columns of arithmetic per byte read from either: 128 rows x 128 features per wave).
// The weights are the products' left operand, so a lane holds a token's column and what it has accumulated are, eight
// at a time, exactly what it has to supply of the next product's right operand: the hidden rows go to the other waves through
// LDS as they are, 64 features at a time, the product with them starting from the residual row in the accumulators.
// K is taken in that order everywhere: element j of half-wave h's eight is feature 4 h + j % 4 + 8 (j / 4) of the sixteen.
// Biases are products as well: three bf16 terms, which add up to the fp32 bias exactly, times ones.
#include "common.hpp"
#include "context.hpp"
#include "kernels.hpp"
#include "mapper.hpp"

namespace pkv {
namespace {

constexpr int kBlkWaves = 4;

// LDS in 16-byte units: the token tile, then two stages of 64 hidden features
constexpr int kXtU4 = kBlk * kDT / 8, kHidU4 = kBlk * 64 / 8;
constexpr int kBlkLds = (kXtU4 + 2 * kHidU4) * 16;

struct BlockArgs {
  const u32x4* w;      // packed weights, this launch's stream of wave 0; wave w's starts w_wave fragments later
  const u32x4* bias;   // packed biases, likewise
  int w_wave, bias_wave;
  const float *ln1_g, *ln1_b, *ln2_g, *ln2_b;
  const u32x4* ao;     // attention output
  f32x4* x;            // residual stream
  u32x4* qkv;
  int T, Tp, blocks;   // valid rows of a layer, rows between layers, blocks of a layer
  int chunks;          // d_ffn / 256
};

// The hidden features' accumulators lie in vector registers (the other 256 of a lane's accumulators fill the accumulation registers), which
// the compiler does not choose by itself.  It does not know these instructions' hazards either: no operand of theirs is
// written by a vector instruction less than two issues before, and s_nop 24 stands between the last of them and the first reader.
__device__ __forceinline__ void mfma_v(f32x16& d, f16x8 a, f16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void bias_v(f32x16& d, bf16x8 a, bf16x8 b) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void bias_a(f32x16& d, bf16x8 a, bf16x8 b) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&a"(d) : "v"(a), "v"(b));
}

template <bool FIRST, bool LAST>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void encoder_block_kernel(BlockArgs a) {
  extern __shared__ u32x4 lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = (unsigned)lane >> 5, l32 = lane & 31;
  const int layer = blockIdx.x / a.blocks, b = blockIdx.x % a.blocks;
  const size_t blk = (size_t)layer * (a.Tp / kBlk) + b;
  u32x4* xt = lds + lane;
  u32x4* hid = lds + kXtU4 + lane;
  f32x4* xu = a.x + (blk * 4 + wave) * (4 * 4 * 4 * 64);  // the wave's part of the residual stream
  const unsigned ul = (unsigned)lane;

  const u32x4* wp = a.w + (size_t)wave * a.w_wave * 64;
  const u32x4* bp = a.bias + (size_t)wave * a.bias_wave * 64;
  u32x4 rg[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) rg[i] = (wp + i * 64)[ul];

  const bf16x8 ones = as_bf16x8(u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
  f32x16 acc[4][4];  // [32 tokens][32 features]

  auto store_half = [&](const f32x16& v, int which) {
    f32x8 t;
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = v[which * 8 + e];
    return __builtin_bit_cast(u32x4, __builtin_convertvector(t, f16x8));
  };

  if constexpr (FIRST) {
    const int rows = a.T - b * kBlk;  // valid rows of the block
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      const bool in = tt * 32 + l32 < rows;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        f32x16 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 t = (xu + ((tt * 4 + mt) * 4 + q) * 64)[ul];
          if (!in) t = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          if (rows < kBlk) (xu + ((tt * 4 + mt) * 4 + q) * 64)[ul] = t;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[q * 4 + e] = t[e];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) xt[(tt * 32 + wave * 8 + mt * 2 + s) * 64] = store_half(v, s);
      }
    }
    __syncthreads();
  } else {
    // the block's attention output, as it lies
    const u32x4* ag = a.ao + blk * kXtU4 + wave * 64;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
#pragma unroll
    for (int i = 0; i < kXtU4 / 256; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)((ag + i * 256) + ul), (lptr_t)(lds + i * 256 + wave * 64), 16, 0, 0);
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 t = (xu + ((tt * 4 + mt) * 4 + q) * 64)[ul];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[tt][mt][q * 4 + e] = t[e];
        }
    bf16x8 bf[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) bf[mt] = as_bf16x8((bp + mt * 64)[ul]);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) acc[tt][mt] = mfma_32x32x16(bf[mt], ones, acc[tt][mt]);
    bp += 4 * 64;

    // K = 512 over the token tile, four feature tiles
    auto gemm_x4 = [&](auto swap) {
      f16x8 xf[2][4];
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) xf[0][tt] = as_f16x8(xt[tt * 32 * 64]);
      const u32x4* xp = xt;
      for (int g = 0; g < 16; ++g) {
        static_for<2>([&](auto kc) {
          constexpr int kk = decltype(kc)::value, cur = kk, nxt = cur ^ 1;
          static_for<16>([&](auto jc) {
            constexpr int j = decltype(jc)::value, mt = j >> 2, tt = j & 3;
            if constexpr (decltype(swap)::value) acc[tt][mt] = mfma_f16_32x32x16(xf[cur][tt], as_f16x8(rg[kk * 4 + mt]), acc[tt][mt]);
            else acc[tt][mt] = mfma_f16_32x32x16(as_f16x8(rg[kk * 4 + mt]), xf[cur][tt], acc[tt][mt]);
            if constexpr (j < 4) xf[nxt][j] = as_f16x8(xp[(j * 32 + kk + 1) * 64]);
            if constexpr (tt == 3) rg[kk * 4 + mt] = (wp + (kk * 4 + mt + 8) * 64)[ul];
            __builtin_amdgcn_sched_barrier(0);
          });
        });
        xp += 2 * 64;
        wp += 8 * 64;
      }
    };
    gemm_x4(std::false_type{});

    struct Pair {
      float s1, s2;
    };
    Pair* red = reinterpret_cast<Pair*>(lds + kXtU4);  // [4 waves][128 tokens]
    auto layer_norm = [&](const float* g, const float* be) {
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            s1 += acc[tt][mt][i];
            s2 = __builtin_fmaf(acc[tt][mt][i], acc[tt][mt][i], s2);
          }
        s1 = halves_sum(s1);
        s2 = halves_sum(s2);
        if (half == 0) red[wave * kBlk + tt * 32 + l32] = Pair{s1, s2};
      }
      __syncthreads();
      const f32x4 *gw = reinterpret_cast<const f32x4*>(g + wave * 128), *bw = reinterpret_cast<const f32x4*>(be + wave * 128);
      float mu[4], rs[4];
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const Pair p = red[w * kBlk + tt * 32 + l32];
          s1 += p.s1;
          s2 += p.s2;
        }
        mu[tt] = s1 * (1.0f / kDT);
        const float var = __builtin_fmaxf(__builtin_fmaf(-mu[tt], mu[tt], s2 * (1.0f / kDT)), 0.0f);
        rs[tt] = 1.0f / sqrtf(var + 1e-5f);
      }
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 g4 = (gw + mt * 8 + q * 2)[half], b4 = (bw + mt * 8 + q * 2)[half];
#pragma unroll
          for (int tt = 0; tt < 4; ++tt)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[tt][mt][q * 4 + e] = (acc[tt][mt][q * 4 + e] - mu[tt]) * rs[tt] * g4[e] + b4[e];
        }
      }
    };
    auto put_x = [&]() {
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int s = 0; s < 2; ++s) xt[(tt * 32 + wave * 8 + mt * 2 + s) * 64] = store_half(acc[tt][mt], s);
    };
    layer_norm(a.ln1_g, a.ln1_b);
    put_x();
    // second FFN product's bias
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) bf[mt] = as_bf16x8((bp + mt * 64)[ul]);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) acc[tt][mt] = mfma_32x32x16(bf[mt], ones, acc[tt][mt]);
    bp += 4 * 64;
    bf16x8 b1[2] = {as_bf16x8(bp[ul]), as_bf16x8((bp + 64)[ul])};
    __syncthreads();

    for (int c = 0; c < a.chunks; ++c) {
      u32x4 ph[4][4];  // [token tile][quarter]
      {
        f32x16 h[4][2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) bias_v(h[tt][mt], b1[mt], ones);
        f16x8 xf[2][4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) xf[0][tt] = as_f16x8(xt[tt * 32 * 64]);
        const u32x4* xp = xt;
        for (int g = 0; g < 8; ++g) {
          static_for<4>([&](auto kc) {
            constexpr int kk = decltype(kc)::value, cur = kk & 1, nxt = cur ^ 1;
            static_for<8>([&](auto jc) {
              constexpr int j = decltype(jc)::value, mt = j >> 2, tt = j & 3;
              mfma_v(h[tt][mt], as_f16x8(rg[kk * 2 + mt]), xf[cur][tt]);
              if constexpr (j < 4) xf[nxt][j] = as_f16x8(xp[(j * 32 + kk + 1) * 64]);
              if constexpr (tt == 3) rg[kk * 2 + mt] = (wp + (kk * 2 + mt + 8) * 64)[ul];
              __builtin_amdgcn_sched_barrier(0);
            });
          });
          xp += 4 * 64;
          wp += 8 * 64;
        }
        asm volatile("s_nop 15\n\ts_nop 7" : "+v"(h[0][0]), "+v"(h[0][1]), "+v"(h[1][0]), "+v"(h[1][1]), "+v"(h[2][0]), "+v"(h[2][1]), "+v"(h[3][0]), "+v"(h[3][1]));
        bp += 2 * 64;
        b1[0] = as_bf16x8(bp[ul]);
        b1[1] = as_bf16x8((bp + 64)[ul]);
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x8 t;
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = __builtin_fmaxf(h[tt][q >> 1][(q & 1) * 8 + e], 0.0f);
            ph[tt][q] = __builtin_bit_cast(u32x4, __builtin_convertvector(t, f16x8));
          }
      }
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) hid[(tt * 4 + wave) * 64] = ph[tt][0];
      static_for<4>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        __syncthreads();
        if constexpr (q < 3) {
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) hid[((q + 1) & 1) * kHidU4 + (tt * 4 + wave) * 64] = ph[tt][q + 1];
        }
        const u32x4* hp = hid + (q & 1) * kHidU4;
        f16x8 hf[2][4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) hf[0][tt] = as_f16x8(hp[tt * 4 * 64]);
        static_for<4>([&](auto kc) {
          constexpr int kk = decltype(kc)::value, cur = kk & 1, nxt = cur ^ 1;
          static_for<16>([&](auto jc) {
            constexpr int j = decltype(jc)::value, mt = j >> 2, tt = j & 3;
            acc[tt][mt] = mfma_f16_32x32x16(as_f16x8(rg[cur * 4 + mt]), hf[cur][tt], acc[tt][mt]);
            if constexpr (j < 4 && kk < 3) hf[nxt][j] = as_f16x8(hp[(j * 4 + kk + 1) * 64]);
            if constexpr (tt == 3) rg[cur * 4 + mt] = (wp + (cur * 4 + mt + 8) * 64)[ul];
            __builtin_amdgcn_sched_barrier(0);
          });
          if constexpr (cur == 1) wp += 8 * 64;
        });
      });
    }
    layer_norm(a.ln2_g, a.ln2_b);
    asm volatile("" : "+s"(xu));
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          (xu + ((tt * 4 + mt) * 4 + q) * 64)[ul] = f32x4{acc[tt][mt][q * 4], acc[tt][mt][q * 4 + 1], acc[tt][mt][q * 4 + 2], acc[tt][mt][q * 4 + 3]};
    if constexpr (!LAST) {
      put_x();
      __syncthreads();
    }
  }
  if constexpr (!LAST) {
    static_for<3>([&](auto rc) {
      constexpr int r = decltype(rc)::value;
      bf16x8 bf[4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) bf[mt] = as_bf16x8((bp + (r * 4 + mt) * 64)[ul]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
          if constexpr (r < 2) bias_a(acc[tt][mt], bf[mt], ones);
          else bias_a(acc[tt][mt], ones, bf[mt]);
        }
      f16x8 xf[2][4];
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) xf[0][tt] = as_f16x8(xt[tt * 32 * 64]);
      const u32x4* xp = xt;
      for (int g = 0; g < 16; ++g) {
        static_for<2>([&](auto kc) {
          constexpr int kk = decltype(kc)::value, cur = kk, nxt = cur ^ 1;
          static_for<16>([&](auto jc) {
            constexpr int j = decltype(jc)::value, mt = j >> 2, tt = j & 3;
            if constexpr (r == 2) acc[tt][mt] = mfma_f16_32x32x16(xf[cur][tt], as_f16x8(rg[kk * 4 + mt]), acc[tt][mt]);
            else acc[tt][mt] = mfma_f16_32x32x16(as_f16x8(rg[kk * 4 + mt]), xf[cur][tt], acc[tt][mt]);
            if constexpr (j < 4) xf[nxt][j] = as_f16x8(xp[(j * 32 + kk + 1) * 64]);
            if constexpr (tt == 3) rg[kk * 4 + mt] = (wp + (kk * 4 + mt + 8) * 64)[ul];
            __builtin_amdgcn_sched_barrier(0);
          });
        });
        xp += 2 * 64;
        wp += 8 * 64;
      }
      u32x4* og = a.qkv + blk * (kBlk * 3 * kDT / 8) + (size_t)wave * (2 * 3 * 1024);
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const int head = mt >> 1;
            const int at = r < 2 ? tt * 4 + (mt & 1) * 2 + s : (tt * 2 + s) * 2 + (mt & 1);
            (og + (head * 3 + r) * 1024 + at * 64)[ul] = store_half(acc[tt][mt], s);
          }
    });
  }
}
// ------------------------------------------------------------------------------------------
// Packing: fragment f of wave w of launch li.  grid (fragments of a wave), 256 threads, a wave each.
// ------------------------------------------------------------------------------------------
struct PackArgs {
  const uint16_t *out_w, *ffn1_w, *ffn2_w, *in_w;  // null: not in this launch
  const float *out_b, *ffn1_b, *ffn2_b, *in_b;
  int d_ffn;
  u32x4 *w, *bias;
};

__global__ __launch_bounds__(256) void pack_weights_kernel(PackArgs a) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  int f = blockIdx.x;
  const uint16_t* src;
  const int layer_frags = 128 + a.d_ffn / 2;
  if (a.out_w && f < layer_frags) {
    if (f < 128) {
      src = a.out_w + (size_t)(wave * 128 + (f & 3) * 32 + l32) * kDT + (f >> 2) * 16;
    } else {
      const int c = (f - 128) >> 7, g = (f - 128) & 127;
      if (g < 64) {
        src = a.ffn1_w + (size_t)(c * 256 + wave * 64 + (g & 1) * 32 + l32) * kDT + (g >> 1) * 16;
      } else {
        const int q = (g - 64) >> 4, k = ((g - 64) >> 2) & 3;
        src = a.ffn2_w + (size_t)(wave * 128 + (g & 3) * 32 + l32) * a.d_ffn + c * 256 + k * 64 + q * 16;
      }
    }
  } else {
    if (a.out_w) f -= layer_frags;
    src = a.in_w + (size_t)((f >> 7) * kDT + wave * 128 + (f & 3) * 32 + l32) * kDT + ((f & 127) >> 2) * 16;
  }
  const u32x2 lo = *reinterpret_cast<const u32x2*>(src + half * 4), hi = *reinterpret_cast<const u32x2*>(src + half * 4 + 8);
  a.w[((size_t)wave * gridDim.x + blockIdx.x) * 64 + lane] = u32x4{lo[0], lo[1], hi[0], hi[1]};
}

__global__ __launch_bounds__(256) void pack_bias_kernel(PackArgs a) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l32 = lane & 31;
  int f = blockIdx.x;
  float b;
  const int layer_frags = 8 + a.d_ffn / 128;
  if (a.out_b && f < layer_frags) {
    if (f < 4) b = a.out_b[wave * 128 + f * 32 + l32];
    else if (f < 8) b = a.ffn2_b[wave * 128 + (f - 4) * 32 + l32];
    else b = a.ffn1_b[((f - 8) >> 1) * 256 + wave * 64 + (f & 1) * 32 + l32];
  } else {
    if (a.out_b) f -= layer_frags;
    b = a.in_b[(f >> 2) * kDT + wave * 128 + (f & 3) * 32 + l32];
  }
  const float hi = bf16_bits_to_f32(f32_to_bf16_bits(b));
  float mid = bf16_bits_to_f32(f32_to_bf16_bits(b - hi)), lo = (b - hi) - mid;
  if (!(__builtin_fabsf(hi) < __builtin_huge_valf())) mid = lo = 0.0f;
  u32x4 v = {pack_bf16x2(hi, mid), pack_bf16x2(lo, 0.0f), 0u, 0u};
  if (lane >= 32) v = u32x4{0u, 0u, 0u, 0u};
  a.bias[((size_t)wave * gridDim.x + blockIdx.x) * 64 + lane] = v;
}

template <bool FIRST, bool LAST>
hipError_t launch(const BlockArgs& a, int blocks, hipStream_t stream) {
  static bool attr_set = false;  // per instantiation; setting it again is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&encoder_block_kernel<FIRST, LAST>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kBlkLds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  encoder_block_kernel<FIRST, LAST><<<blocks, 256, kBlkLds, stream>>>(a);
  return hipGetLastError();
}
}  // namespace

hipError_t pack_encoder_blocks(const proxykv_config& c, const MapperWeights& w, void* blk_w, void* blk_b, hipStream_t stream) {
  u32x4 *pw = (u32x4*)blk_w, *pb = (u32x4*)blk_b;
  for (int li = 0; li <= c.n_enc_layers; ++li) {
    PackArgs a = {};
    if (li > 0) {
      const EncoderLayerWeights& e = w.enc[li - 1];
      a.out_w = e.out_w;
      a.ffn1_w = e.ffn1_w;
      a.ffn2_w = e.ffn2_w;
      a.out_b = e.out_b;
      a.ffn1_b = e.ffn1_b;
      a.ffn2_b = e.ffn2_b;
    }
    if (li < c.n_enc_layers) {
      a.in_w = w.enc[li].in_w;
      a.in_b = w.enc[li].in_b;
    }
    a.d_ffn = c.d_ffn;
    a.w = pw;
    a.bias = pb;
    pack_weights_kernel<<<(unsigned)block_frags(c, li), 256, 0, stream>>>(a);
    PKV_TRY(hipGetLastError());
    pack_bias_kernel<<<(unsigned)block_bias_frags(c, li), 256, 0, stream>>>(a);
    PKV_TRY(hipGetLastError());
    pw += 4 * block_frags(c, li) * 64;
    pb += 4 * block_bias_frags(c, li) * 64;
  }
  return hipSuccess;
}

hipError_t launch_encoder_block(const proxykv_ctx* ctx, const MapPlan& p, int n_layers, int li, float* x, const uint16_t* ao, uint16_t* qkv,
                                hipStream_t stream) {
  const proxykv_config& c = ctx->cfg;
  BlockArgs a = {};
  size_t w_off = 0, b_off = 0;
  for (int i = 0; i < li; ++i) {
    w_off += 4 * block_frags(c, i);
    b_off += 4 * block_bias_frags(c, i);
  }
  a.w = (const u32x4*)ctx->w.blk_w + w_off * 64;
  a.bias = (const u32x4*)ctx->w.blk_b + b_off * 64;
  a.w_wave = (int)block_frags(c, li);
  a.bias_wave = (int)block_bias_frags(c, li);
  if (li > 0) {
    const EncoderLayerWeights& e = ctx->w.enc[li - 1];
    a.ln1_g = e.ln1_g;
    a.ln1_b = e.ln1_b;
    a.ln2_g = e.ln2_g;
    a.ln2_b = e.ln2_b;
  }
  a.ao = (const u32x4*)ao;
  a.x = (f32x4*)x;
  a.qkv = (u32x4*)qkv;
  a.T = (int)p.T;
  a.Tp = (int)p.Tp;
  a.blocks = (int)((p.T + kBlk - 1) / kBlk);
  a.chunks = c.d_ffn / 256;
  const int blocks = n_layers * a.blocks;
  if (li == 0) return launch<true, false>(a, blocks, stream);
  if (li == c.n_enc_layers) return launch<false, true>(a, blocks, stream);
  return launch<false, false>(a, blocks, stream);
}

}  // namespace pkv
