// The encoder of the large-tile mapper, everything but the attention: out-projection, residual, LayerNorm, both FFN products, residual,
// LayerNorm and the next layer's q, k and v in one launch per layer.  (The first launch has only q, k and v, the last no q, k and v.)
//
// A workgroup takes a block of 128 rows, or half of one, through all of it.  As separate products (256 x 256 and 128 x 512 tiles, normalised rows
// and hidden rows through memory) a layer moved 28 times the 1 KB of an fp16 row, as here with the attention 12 times; and those kernels
// stood in waits of one workgroup per CU 28 to 42 % of the time: 126 976 rows took 1117 us per layer beside the attention.
//
// Four waves, one per SIMD, each with all 512 registers of a lane.  The block's operand (attention output, then normalised rows) lies
// in LDS, 128 KB, in the order in which MFMA fragments are read.  Every wave owns a quarter of each product's features, so it needs
// weights that no other wave of the workgroup reads: they come from L2 straight into registers, in the order of their use, eight
// fragments ahead (sixteen for half a block), and never through LDS.
// The weights are the products' left operand, so a lane holds a token's column and what it has accumulated are, eight
// at a time, exactly what it has to supply of the next product's right operand: the hidden rows go to the other waves through
// LDS as they are, 64 features at a time, the product with them starting from the residual row in the accumulators.
// K is taken in that order everywhere: element j of lane quarter g's eight is feature 4 g + j % 4 + 16 (j / 4) of the thirty-two.
// Biases are products as well: three bf16 terms, which add up to the fp32 bias exactly, times ones.
#include "common.hpp"
#include "context.hpp"
#include "kernels.hpp"
#include "mapper.hpp"

namespace pkv {
namespace {

// LDS in 16-byte units: the token tile, then two stages of 64 hidden features
template <int NT>
struct BlockLds {
  static constexpr int kX = NT * 16 * 64, kHid = NT * 2 * 64, kBytes = (kX + 2 * kHid) * 16;
};

struct BlockArgs {
  const u32x4* w;      // packed weights, this launch's stream of wave 0; wave w's starts w_wave fragments later
  const u32x4* bias;   // packed biases, likewise
  int w_wave, bias_wave;
  const float *ln1_g, *ln1_b, *ln2_g, *ln2_b;
  const u32x4* ao;     // attention output
  f32x4* x;            // residual stream
  u32x4* qkv;
  int T, Tp, parts;    // valid rows of a layer, rows between layers, workgroups of a layer
  int chunks;          // d_ffn / 256
};

// The hidden features' accumulators lie in vector registers (the other 256 of a lane's accumulators fill the accumulation registers), which
// the compiler does not choose by itself.  It does not know these instructions' hazards either: no operand of theirs is
// written by a vector instruction less than two issues before, and s_nop 24 stands between the last of them and the first reader.
__device__ __forceinline__ void mfma_v(f32x4& d, u32x4 a, u32x4 b) {
  asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
// d = bias: the first product of a sum, which needs no cleared accumulators
__device__ __forceinline__ void bias_v(f32x4& d, u32x4 a, u32x4 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void bias_a(f32x4& d, u32x4 a, u32x4 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&a"(d) : "v"(a), "v"(b));
}

// Memory through buffer resources: a uniform base and offset in scalar registers, the lane's 16 bytes the same vector register everywhere.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t resource(const void* base, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 load16(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, int at) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_bytes, at, 0);
}
__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, int at, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)lane_bytes, at, 0);
}

__device__ __forceinline__ u32x4 pack8(const f32x4& lo, const f32x4& hi) {
  const f32x8 t = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(u32x4, __builtin_convertvector(t, f16x8));
}

// NT token tiles of 16: a whole block of 128 rows, or half of one (kHalfBlocks).  The sums are the same, in the same order.
template <int NT, bool FIRST, bool LAST>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void encoder_block_kernel(BlockArgs a) {
  // the token tile, [NT tiles of 16 tokens][16 K steps of 32], then two stages of hidden rows, [2][NT][2]
  extern __shared__ u32x4 lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const unsigned ul = (unsigned)lane;
  constexpr int kXtU4 = BlockLds<NT>::kX, kHidU4 = BlockLds<NT>::kHid, P = 8 / NT, R = NT == 8 ? 8 : 16;  // R: fragments asked for ahead
  const int layer = blockIdx.x / a.parts, part = blockIdx.x % a.parts, b = part / P, t0 = part % P * NT;
  const size_t blk = (size_t)layer * (a.Tp / kBlk) + b;
  const unsigned l16b = ul * 16;
  const __amdgpu_buffer_rsrc_t xr = resource(a.x + ((blk * 4 + wave) * 8 + t0) * (8 * 64), NT * 8 * 1024);  // the wave's part of the residual stream
  const __amdgpu_buffer_rsrc_t wr = resource(a.w + (size_t)wave * a.w_wave * 64, (a.w_wave + R) * kBlkFragBytes);
  const __amdgpu_buffer_rsrc_t br = resource(a.bias + (size_t)wave * a.bias_wave * 64, (a.bias_wave + 4) * kBlkFragBytes);
  int wp = 0, bp = 0;  // positions in the weights and the biases, bytes
  u32x4 rg[R];
#pragma unroll
  for (int i = 0; i < R; ++i) rg[i] = load16(wr, l16b, i * 1024);

  u32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};  // bf16
  asm volatile("" : "+v"(ones));  // made once, and not in front of an instruction that reads it
  f32x4 acc[NT][8];  // [16 tokens][16 features]
  u32x4 f[2][NT];    // token fragments of this K step and the next

  // The lane, as a value that the compiler does not know: addresses made from it are made anew and not kept (and spilled) between
  // phases.  A reload behind the stores of the residual rows would wait for all of them.
  auto fresh = [&]() __attribute__((always_inline)) {
    unsigned v = ul;
    asm volatile("" : "+v"(v));
    return v;
  };
  auto read_x = [&]() __attribute__((always_inline)) {
    const u32x4* src = lds + fresh();
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) f[0][tt] = src[tt * 16 * 64];
  };
  // acc (+)= product with the token tile, K = 512.  Of two MFMAs in a row one operand is the same, also where the feature tile changes:
  // what the matrix cores draw, and with it the clock, depends on how much of their input changes.
  auto gemm_x = [&](auto swap) __attribute__((always_inline)) {
    const u32x4* xp = lds + fresh();
    for (int g = 0; g < 8; ++g) {
      static_for<2>([&](auto kc) {
        constexpr int kk = decltype(kc)::value;
        static_for<8 * NT>([&](auto jc) {
          constexpr int j = decltype(jc)::value, mt = j / NT, tt = (mt & 1) ? NT - 1 - j % NT : j % NT, slot = (kk * 8 + mt) % R;
          const f16x8 fw = as_f16x8(rg[slot]), fx = as_f16x8(f[kk][tt]);
          acc[tt][mt] = decltype(swap)::value ? mfma_f16_16x16x32(fx, fw, acc[tt][mt]) : mfma_f16_16x16x32(fw, fx, acc[tt][mt]);
          if constexpr (j % 4 == 0 && j < 4 * NT) f[kk ^ 1][j / 4] = xp[(j / 4 * 16 + kk + 1) * 64];
          if constexpr (j % NT == NT - 1) rg[slot] = load16(wr, l16b, wp + (kk * 8 + mt + R) * 1024);
          __builtin_amdgcn_sched_barrier(0);
        });
      });
      wp += 16 * 1024;
      xp += 2 * 64;
    }
  };
  auto put_x = [&]() __attribute__((always_inline)) {
    u32x4* dst = lds + wave * 4 * 64 + fresh();
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int s = 0; s < 4; ++s) dst[(tt * 16 + s) * 64] = pack8(acc[tt][2 * s], acc[tt][2 * s + 1]);
  };

  u32x4 bf[8];      // bias fragments
  auto load_bf = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < 8; ++mt) bf[mt] = load16(br, l16b, bp + mt * 1024);
    bp += 8 * 1024;
  };

  if constexpr (!FIRST) {
    // the block's attention output, as it lies
    const u32x4* ag = a.ao + (blk * 8 + t0) * (16 * 64) + wave * 64;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
#pragma unroll
    for (int i = 0; i < kXtU4 / 256; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)((ag + i * 256) + ul), (lptr_t)(lds + i * 256 + wave * 64), 16, 0, 0);
  }
#pragma unroll
  for (int tt = 0; tt < NT; ++tt)
#pragma unroll
    for (int mt = 0; mt < 8; ++mt) acc[tt][mt] = __builtin_bit_cast(f32x4, load16(xr, l16b, (tt * 8 + mt) * 1024));

  if constexpr (FIRST) {
    // rows past the layer's last one become zeros, so that everything computed from them is finite
    const int rows = a.T - b * kBlk - t0 * 16;
    if (rows < NT * 16) {
#pragma unroll
      for (int tt = 0; tt < NT; ++tt)
        if (tt * 16 + (lane & 15) >= rows) {
#pragma unroll
          for (int mt = 0; mt < 8; ++mt) {
            acc[tt][mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            store16(xr, l16b, (tt * 8 + mt) * 1024, u32x4{0u, 0u, 0u, 0u});
          }
        }
    }
    load_bf();
    put_x();
    __syncthreads();
    read_x();
  } else {
    // acc = residual + bias + out-projection
    load_bf();
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the tile has landed
    __syncthreads();
    read_x();
    auto add_bias = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int mt = 0; mt < 8; ++mt)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
          acc[tt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(bf[mt]), as_bf16x8(ones), acc[tt][mt], 0, 0, 0);
    };
    add_bias();
    gemm_x(std::false_type{});

    // LayerNorm of the rows: a token's features lie in four lanes of each of four waves
    struct Pair {
      float s1, s2;
    };
    Pair* red = reinterpret_cast<Pair*>(lds + kXtU4);  // [4 waves][16 NT tokens], in place of the hidden rows
    auto layer_norm = [&](const float* g, const float* be) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t gr = resource(g + wave * 128, 512), er = resource(be + wave * 128, 512);
      const unsigned l = fresh(), q = l >> 4, col = l & 15;
      f32x4 g4[8], b4[8];
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) {
        g4[mt] = __builtin_bit_cast(f32x4, load16(gr, q * 16, mt * 64));
        b4[mt] = __builtin_bit_cast(f32x4, load16(er, q * 16, mt * 64));
      }
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int mt = 0; mt < 8; ++mt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s1 += acc[tt][mt][i];
            s2 = __builtin_fmaf(acc[tt][mt][i], acc[tt][mt][i], s2);
          }
        s1 = quads_sum(s1);
        s2 = quads_sum(s2);
        if (q == 0) red[wave * NT * 16 + tt * 16 + col] = Pair{s1, s2};
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const Pair p = red[w * NT * 16 + tt * 16 + col];
          s1 += p.s1;
          s2 += p.s2;
        }
        const float mu = s1 * (1.0f / kDT);
        const float var = __builtin_fmaxf(__builtin_fmaf(-mu, mu, s2 * (1.0f / kDT)), 0.0f);
        const float rs = 1.0f / sqrtf(var + 1e-5f), shift = -mu * rs;
#pragma unroll
        for (int mt = 0; mt < 8; ++mt)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[tt][mt][e] = __builtin_fmaf(__builtin_fmaf(acc[tt][mt][e], rs, shift), g4[mt][e], b4[mt][e]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    layer_norm(a.ln1_g, a.ln1_b);
    put_x();
    load_bf();
    u32x4 b1[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) b1[mt] = load16(br, l16b, bp + mt * 1024);
    add_bias();  // the second FFN product's
    __syncthreads();
    read_x();

    for (int c = 0; c < a.chunks; ++c) {
      // 64 hidden features per wave
      f32x4 h[NT][4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) bias_v(h[tt][mt], b1[mt], ones);
      const u32x4* xp = lds + fresh();
      u32x2 ph[NT][4];
      // ReLU and rounding of a finished tile; half of them are at once what another wave reads
      auto finish = [&](auto tc, auto mc) __attribute__((always_inline)) {
        constexpr int tt = decltype(tc)::value, mt = decltype(mc)::value;
        const f16x4 z = {0, 0, 0, 0};
        ph[tt][mt] = __builtin_bit_cast(u32x2, __builtin_elementwise_max(__builtin_convertvector(h[tt][mt], f16x4), z));
      };
      constexpr int kLag = 8 / NT;  // rows of tiles between a tile's last MFMA and its rounding: eight MFMAs
      auto step = [&](auto kc, auto last) __attribute__((always_inline)) {
        constexpr int kk = decltype(kc)::value, cur = kk & 1;
        static_for<4 * NT>([&](auto jc) {
          constexpr int j = decltype(jc)::value, mt = j / NT, tt = (mt & 1) ? NT - 1 - j % NT : j % NT, slot = (kk * 4 + mt) % R;
          mfma_v(h[tt][mt], rg[slot], f[cur][tt]);
          if constexpr (!decltype(last)::value && j % 3 == 0 && j < 3 * NT) f[cur ^ 1][j / 3] = xp[(j / 3 * 16 + kk + 1) * 64];
          if constexpr (j % NT == NT - 1) rg[slot] = load16(wr, l16b, wp + (kk * 4 + mt + R) * 1024);
          if constexpr (decltype(last)::value && mt >= kLag)
            finish(std::integral_constant<int, kLag % 2 ? NT - 1 - tt : tt>{}, std::integral_constant<int, mt - kLag>{});
          __builtin_amdgcn_sched_barrier(0);
        });
      };
      constexpr int kSteps = R / 4;
#pragma unroll 1
      for (int g = 0; g < 16 / kSteps - 1; ++g) {
        static_for<kSteps>([&](auto kc) { step(kc, std::false_type{}); });
        xp += kSteps * 64;
        wp += R * 1024;
      }
      static_for<kSteps>([&](auto kc) { step(kc, std::integral_constant<bool, decltype(kc)::value == kSteps - 1>{}); });
      wp += R * 1024;
      if constexpr (NT == 8)
        asm volatile("s_nop 15\n\ts_nop 7" : "+v"(h[0][3]), "+v"(h[1][3]), "+v"(h[2][3]), "+v"(h[3][3]), "+v"(h[4][3]), "+v"(h[5][3]), "+v"(h[6][3]), "+v"(h[7][3]));
      else
        asm volatile("s_nop 15\n\ts_nop 7" : "+v"(h[0][2]), "+v"(h[1][2]), "+v"(h[2][2]), "+v"(h[3][2]), "+v"(h[0][3]), "+v"(h[1][3]), "+v"(h[2][3]), "+v"(h[3][3]));
      static_for<NT * kLag>([&](auto tc) {
        constexpr int i = decltype(tc)::value;
        finish(std::integral_constant<int, i % NT>{}, std::integral_constant<int, 4 - kLag + i / NT>{});
      });
      bp += 4 * 1024;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) b1[mt] = load16(br, l16b, bp + mt * 1024);
      // Stage q holds feature tile q of every wave: two K steps, each half of one wave's and half of the next's.
      auto put_h = [&](int q) __attribute__((always_inline)) {
        u32x2* dst = reinterpret_cast<u32x2*>(lds + kXtU4 + (q & 1) * kHidU4 + (wave >> 1) * 64 + fresh()) + (wave & 1);
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) dst[tt * 2 * 64 * 2] = ph[tt][q];
      };
      put_h(0);
      put_h(1);
      __syncthreads();
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) f[0][tt] = lds[kXtU4 + tt * 2 * 64 + ul];
      static_for<4>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const u32x4* hp = lds + kXtU4 + (q & 1) * kHidU4 + ul;
        const u32x4* hn = lds + kXtU4 + ((q + 1) & 1) * kHidU4 + ul;
        static_for<2>([&](auto kc) {
          constexpr int kk = decltype(kc)::value;
          if constexpr (kk == 1) {
            // Every wave has read all of stage q: stage q + 2 takes its place, and stage q + 1, written a step ago, is complete.
            __syncthreads();
            if constexpr (q < 2) put_h(q + 2);
          }
          static_for<8 * NT>([&](auto jc) {
            constexpr int j = decltype(jc)::value, mt = j / NT, tt = (mt & 1) ? NT - 1 - j % NT : j % NT, slot = (kk * 8 + mt) % R;
            acc[tt][mt] = mfma_f16_16x16x32(as_f16x8(rg[slot]), as_f16x8(f[kk][tt]), acc[tt][mt]);
            if constexpr (j % 4 == 0 && j < 4 * NT) {
              if constexpr (kk == 0) f[1][j / 4] = hp[(j / 4 * 2 + 1) * 64];
              else if constexpr (q < 3) f[0][j / 4] = hn[j / 4 * 2 * 64];
              else f[0][j / 4] = lds[j / 4 * 16 * 64 + ul];
            }
            if constexpr (j % NT == NT - 1) rg[slot] = load16(wr, l16b, wp + (kk * 8 + mt + R) * 1024);
            __builtin_amdgcn_sched_barrier(0);
          });
        });
        wp += 16 * 1024;
      });
    }
    layer_norm(a.ln2_g, a.ln2_b);
    if constexpr (!LAST) load_bf();  // in front of the stores: loads are counted in order with them
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) store16(xr, l16b, (tt * 8 + mt) * 1024, __builtin_bit_cast(u32x4, acc[tt][mt]));
    if constexpr (!LAST) {
      put_x();
      __syncthreads();
      read_x();
    }
  }
  if constexpr (!LAST) {
    // q, k (a lane holds a token's column) and v (a lane holds a feature's column of tokens, as the attention's second product wants it)
    const __amdgpu_buffer_rsrc_t qr = resource(a.qkv + (blk * 4 + wave) * (kBlk * 3 * kDT / 8 / 4), kBlk * 3 * kDT * 2 / 4);
    static_for<3>([&](auto rc) {
      constexpr int r = decltype(rc)::value;
#pragma unroll
      for (int mt = 0; mt < 8; ++mt)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
          if constexpr (r < 2) bias_a(acc[tt][mt], bf[mt], ones);
          else bias_a(acc[tt][mt], ones, bf[mt]);
        }
      if constexpr (r > 0) read_x();
      gemm_x(std::integral_constant<bool, r == 2>{});
      if constexpr (r < 2) load_bf();
      static_for<2 * NT>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        static_for<2>([&](auto hc) {
          constexpr int head = decltype(hc)::value;
          const int at = ((head * 3 + r) * 16 + t0 * 2 + u) * 1024;
          if constexpr (r < 2) store16(qr, l16b, at, pack8(acc[u >> 1][head * 4 + 2 * (u & 1)], acc[u >> 1][head * 4 + 2 * (u & 1) + 1]));
          else store16(qr, l16b, at, pack8(acc[2 * (u >> 2)][head * 4 + (u & 3)], acc[2 * (u >> 2) + 1][head * 4 + (u & 3)]));
        });
      });
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
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, quad = lane >> 4, l16 = lane & 15;
  int f = blockIdx.x, second = 16;  // second: elements from the first four of a lane's eight to the others
  const uint16_t* src;
  const int layer_frags = 128 + a.d_ffn / 2;
  if (a.out_w && f < layer_frags) {
    if (f < 128) {
      src = a.out_w + (size_t)(wave * 128 + (f & 7) * 16 + l16) * kDT + (f >> 3) * 32;
    } else {
      const int c = (f - 128) >> 7, g = (f - 128) & 127;
      if (g < 64) {
        src = a.ffn1_w + (size_t)(c * 256 + wave * 64 + (g & 3) * 16 + l16) * kDT + (g >> 2) * 32;
      } else {
        const int q = (g - 64) >> 4, k = ((g - 64) >> 3) & 1;
        src = a.ffn2_w + (size_t)(wave * 128 + (g & 7) * 16 + l16) * a.d_ffn + c * 256 + k * 128 + q * 16;
        second = 64;
      }
    }
  } else {
    if (a.out_w) f -= layer_frags;
    src = a.in_w + (size_t)((f >> 7) * kDT + wave * 128 + (f & 7) * 16 + l16) * kDT + ((f & 127) >> 3) * 32;
  }
  const u32x2 lo = *reinterpret_cast<const u32x2*>(src + quad * 4), hi = *reinterpret_cast<const u32x2*>(src + quad * 4 + second);
  a.w[((size_t)wave * gridDim.x + blockIdx.x) * 64 + lane] = u32x4{lo[0], lo[1], hi[0], hi[1]};
}

__global__ __launch_bounds__(256) void pack_bias_kernel(PackArgs a) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15;
  int f = blockIdx.x;
  float b;
  const int layer_frags = 16 + a.d_ffn / 64;
  if (a.out_b && f < layer_frags) {
    if (f < 8) b = a.out_b[wave * 128 + f * 16 + l16];
    else if (f < 16) b = a.ffn2_b[wave * 128 + (f - 8) * 16 + l16];
    else b = a.ffn1_b[((f - 16) >> 2) * 256 + wave * 64 + (f & 3) * 16 + l16];
  } else {
    if (a.out_b) f -= layer_frags;
    b = a.in_b[(f >> 3) * kDT + wave * 128 + (f & 7) * 16 + l16];
  }
  const float hi = bf16_bits_to_f32(f32_to_bf16_bits(b));
  float mid = bf16_bits_to_f32(f32_to_bf16_bits(b - hi)), lo = (b - hi) - mid;
  if (!(__builtin_fabsf(hi) < __builtin_huge_valf())) mid = lo = 0.0f;
  u32x4 v = {pack_bf16x2(hi, mid), pack_bf16x2(lo, 0.0f), 0u, 0u};
  if (lane >= 16) v = u32x4{0u, 0u, 0u, 0u};
  a.bias[((size_t)wave * gridDim.x + blockIdx.x) * 64 + lane] = v;
}

template <int NT, bool FIRST, bool LAST>
hipError_t launch(const BlockArgs& a, int n_layers, hipStream_t stream) {
  static bool attr_set = false;  // per instantiation; setting it again is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&encoder_block_kernel<NT, FIRST, LAST>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, BlockLds<NT>::kBytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  encoder_block_kernel<NT, FIRST, LAST><<<n_layers * a.parts, 256, BlockLds<NT>::kBytes, stream>>>(a);
  return hipGetLastError();
}
template <int NT>
hipError_t launch_parts(BlockArgs a, int n_layers, int li, int n_enc, hipStream_t stream) {
  a.parts = (a.T + NT * 16 - 1) / (NT * 16);
  if (li == 0) return launch<NT, true, false>(a, n_layers, stream);
  if (li == n_enc) return launch<NT, false, true>(a, n_layers, stream);
  return launch<NT, false, false>(a, n_layers, stream);
}
// Up to this many blocks in flight (half the CUs) each is given to two workgroups.  A whole block's time is its matrix work (131 us a middle launch
// alone on the chip), a half's its weights' way from L2 (6.3 MB for each workgroup and layer, 42 us at 64 bytes a clock and CU) and its products (42 us)
// in turn, with one wave per SIMD to do both: 88 us.  A quarter would read as many weights for half of the products.
// us, halves / wholes: one layer of 5548 rows 821 / 1139, of 16 k 1132 / 1323, 16 of 500 665 / 978; with 129 .. 256 blocks some
// CUs do two halves in turn, one layer of 26 k 1945 / 1738.
// Two lanes' blocks are not in step: while one lane's launch ends or its attention runs, the other's halves have the chip, so up to three quarters
// of the CUs' number pay there (half of them in either launch).  16 layers of 1100 rows (144 blocks of both lanes) 1193 / 1306, of 1500 (192)
// 1514 / 1644, 24 of 900 (192) 1305 / 1369, 28 of 700 (168) 1101 / 1190; beyond that the shapes differ: 16 of 1700 (224) 1786 / 1811, 28 of 1000
// (224) 1547 / 1476, 16 of 2000 (256) 2331 / 2202.
constexpr int64_t kHalfBlocks = 128, kHalfBlocksLanes = 192;
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
  a.chunks = c.d_ffn / 256;
  const int64_t blocks = (p.T + kBlk - 1) / kBlk * n_layers * p.lanes;  // of all lanes together
  return blocks <= (p.lanes > 1 ? kHalfBlocksLanes : kHalfBlocks) ? launch_parts<4>(a, n_layers, li, c.n_enc_layers, stream) : launch_parts<8>(a, n_layers, li, c.n_enc_layers, stream);
}

}  // namespace pkv
