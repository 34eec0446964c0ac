// Instruction-mix ceiling of scoring pass 1 (row log-sum-exp, paper Sec. 3) on gfx950, with no memory traffic at all.
//
// Per 32-key sub-tile and wave, pass 1 issues 8 v_mfma_f32_32x32x16_bf16 (two query sub-tiles, d = 64) and, on the
// 2 x 16 logits per lane that they produce, 32 x (v_fma_f32, v_exp_f32, v_add_f32).  This program runs exactly that
// mix out of registers, at the kernel's occupancy (256-thread workgroups, WPE waves per SIMD), in three forms:
//   mfma    the 8 MFMAs only
//   vector  the 96 vector instructions only
//   both    the MFMAs, then the vector work on their results (the kernel's shape)
// and prints, for each, the elapsed time and the fraction of the matrix pipe's peak it corresponds to
// (8 MFMAs x 32 cycles per sub-tile and wave against the elapsed cycles at 2.4 GHz).  If the two kinds of work ran
// side by side, "both" would take as long as the longer of the two; in that order of instructions it takes nearly their sum.
//
// Then the same work in two orders, on zeros, which draw little power, and on random numbers, with which the chip's power sets its
// clock:
//   program  a sub-tile's MFMAs, then the vector work on their results, as the compiler arranges it
//   first    units of one column tile (score_lse_piped.hip): 16 fma, 16 exponentials at a higher wave priority with the next unit's
//            MFMAs between them, 16 adds
// printed as time per logit of a lane, all waves of a SIMD taken together: what pass 1 can be measured against in that order.
//
// Build and run (one MI355X):
//   hipcc --offload-arch=gfx950 -O3 -std=c++17 -Xclang -target-feature -Xclang -packed-fp32-ops \
//         -o paper_2605_16360_amd/microbench/score_mix paper_2605_16360_amd/microbench/score_mix.hip
//   ./paper_2605_16360_amd/microbench/score_mix
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#define CHECK(x)                                                            \
  do {                                                                      \
    hipError_t e_ = (x);                                                    \
    if (e_ != hipSuccess) {                                                 \
      printf("HIP error %s at line %d\n", hipGetErrorString(e_), __LINE__); \
      exit(1);                                                              \
    }                                                                       \
  } while (0)

__device__ __forceinline__ f32x16 mm(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() { return f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}; }

enum Form { kMfma, kVector, kBoth };

// LDSKB keeps further workgroups off the CU, so that WPE is the occupancy that runs
template <int FORM, int WPE, int LDSKB>
__global__ __launch_bounds__(256, WPE) void mix_kernel(float* out, int iters, float seed) {
  __shared__ float pad[LDSKB * 256];
  pad[threadIdx.x] = seed;
  __syncthreads();
  const float sd = pad[threadIdx.x & 63];
  bf16x8 a[4], b[2][4];
  for (int kk = 0; kk < 4; ++kk)
    for (int i = 0; i < 8; ++i) {
      a[kk][i] = (__bf16)(sd * 0.01f * (i + kk));
      b[0][kk][i] = (__bf16)(sd * 0.02f * (i - kk));
      b[1][kk][i] = (__bf16)(sd * 0.03f * (i + 2 * kk));
    }
  const float c = 0.18f * sd, nref = -1.0f * sd;
  float l0 = 0, l1 = 0, l2 = 0, l3 = 0;
  auto vec16 = [&](const f32x16& acc) {
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
      l0 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 0], c, nref));
      l1 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 1], c, nref));
      l2 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 2], c, nref));
      l3 += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[r + 3], c, nref));
    }
  };
  if constexpr (FORM == kMfma) {
    f32x16 acc[2] = {zero16(), zero16()};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int cs = 0; cs < 2; ++cs)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) acc[cs] = mm(a[kk], b[cs][kk], acc[cs]);
    }
    l0 = acc[0][0] + acc[1][1];
  } else if constexpr (FORM == kVector) {
    f32x16 acc[2];
    for (int i = 0; i < 16; ++i) {
      acc[0][i] = sd * i;
      acc[1][i] = sd * (i + 16);
    }
    for (int it = 0; it < iters; ++it) {
      vec16(acc[0]);
      vec16(acc[1]);
      acc[0][it & 15] += l0 * 1e-30f;  // keeps the iterations distinct
    }
  } else {
    for (int it = 0; it < iters; ++it) {
      f32x16 acc[2];
#pragma unroll
      for (int cs = 0; cs < 2; ++cs) {
        acc[cs] = zero16();
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) acc[cs] = mm(a[kk], b[cs][kk], acc[cs]);
      }
      vec16(acc[0]);
      vec16(acc[1]);
      a[0][0] += (__bf16)l0;  // keeps the iterations distinct
    }
  }
  out[blockIdx.x * 256 + threadIdx.x] = (l0 + l1) + (l2 + l3);
}

// FIRST: the units' order; otherwise the compiler's.  The keys' fragments change places from sub-tile to sub-tile, so that
// operands change as they do in the kernel.
template <bool FIRST, int WPE, int LDSKB>
__global__ __launch_bounds__(256, WPE) void order_kernel(float* out, int iters, float scale, float c) {
  __shared__ float pad[LDSKB * 256];
  pad[threadIdx.x] = scale;
  __syncthreads();
  const float sc = pad[threadIdx.x & 63];
  uint32_t h = (blockIdx.x * 256 + threadIdx.x) * 2654435761u + 1u;
  auto random = [&]() {  // the sum of four uniform numbers, mean 0, variance 1
    float s = -2.0f;
    for (int i = 0; i < 4; ++i) {
      h = h * 1664525u + 1013904223u;
      s += (float)(h >> 8) * (1.0f / 16777216.0f);
    }
    return (__bf16)(sc * 1.7320508f * s);
  };
  bf16x8 a[4], b[2][4];
  for (int kk = 0; kk < 4; ++kk)
    for (int i = 0; i < 8; ++i) {
      a[kk][i] = random();
      b[0][kk][i] = random();
      b[1][kk][i] = random();
    }
  float nref[2] = {-3.0f * sc, -4.0f * sc}, sum[2] = {0.0f, 0.0f};
  f32x16 acc[2] = {zero16(), zero16()};
  for (int it = 0; it < iters; ++it) {
    for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(a[kk]));
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if constexpr (FIRST) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float e[16];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int r = 0; r < 16; ++r) e[r] = __builtin_fmaf(acc[u][r], c, nref[u]);
          __builtin_amdgcn_sched_barrier(0);
          __builtin_amdgcn_s_setprio(2);
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const int f = (kk + s + u) & 3;  // the next unit's sub-tile: s, or behind its second unit s + 1
            acc[u ^ 1] = mm(a[f], b[u ^ 1][kk], kk == 0 ? zero16() : acc[u ^ 1]);
#pragma unroll
            for (int r = kk * 4; r < kk * 4 + 4; ++r) e[r] = __builtin_amdgcn_exp2f(e[r]);
            __builtin_amdgcn_sched_barrier(0);
          }
          __builtin_amdgcn_s_setprio(0);
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = e[r];
#pragma unroll
          for (int r = 4; r < 16; ++r) v[r & 3] += e[r];
          sum[u] += (v[0] + v[1]) + (v[2] + v[3]);
        }
      } else {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          acc[u] = zero16();
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) acc[u] = mm(a[(kk + s) & 3], b[u][kk], acc[u]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[u][r], c, nref[u]));
#pragma unroll
          for (int r = 4; r < 16; ++r) v[r & 3] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[u][r], c, nref[u]));
          sum[u] += (v[0] + v[1]) + (v[2] + v[3]);
        }
      }
    }
  }
  out[blockIdx.x * 256 + threadIdx.x] = sum[0] + sum[1] + acc[0][0] + acc[1][0];
}

template <bool FIRST, int WPE, int LDSKB>
void run_order(float* out, int iters, float scale) {
  hipEvent_t e0, e1;
  CHECK(hipEventCreate(&e0));
  CHECK(hipEventCreate(&e1));
  const int blocks = 256 * WPE, reps = 4;
  auto go = [&]() {
    order_kernel<FIRST, WPE, LDSKB><<<blocks, 256>>>(out, iters, scale, 0.1803369f);
    CHECK(hipGetLastError());
  };
  for (int i = 0; i < reps; ++i) go();  // until the clock has settled
  CHECK(hipEventRecord(e0));
  for (int i = 0; i < reps; ++i) go();
  CHECK(hipEventRecord(e1));
  CHECK(hipEventSynchronize(e1));
  float ms;
  CHECK(hipEventElapsedTime(&ms, e0, e1));
  const double logits = (double)iters * 4 * 32 * WPE;  // of a lane, all waves of a SIMD
  printf("%-8s %-8s %d waves/SIMD  %8.3f ms   %.2f ns per logit\n", FIRST ? "first" : "program", scale == 0.0f ? "zeros" : "random", WPE, ms / reps, ms / reps * 1e6 / logits);
  fflush(stdout);
  CHECK(hipEventDestroy(e0));
  CHECK(hipEventDestroy(e1));
}

template <int FORM, int WPE, int LDSKB>
double run(const char* name, float* out, int iters) {
  hipEvent_t e0, e1;
  CHECK(hipEventCreate(&e0));
  CHECK(hipEventCreate(&e1));
  const int blocks = 256 * WPE;  // one per CU and occupancy slot
  mix_kernel<FORM, WPE, LDSKB><<<blocks, 256>>>(out, 10, 1.0f);
  CHECK(hipGetLastError());
  CHECK(hipDeviceSynchronize());
  CHECK(hipEventRecord(e0));
  mix_kernel<FORM, WPE, LDSKB><<<blocks, 256>>>(out, iters, 1.0f);
  CHECK(hipGetLastError());
  CHECK(hipEventRecord(e1));
  CHECK(hipEventSynchronize(e1));
  float ms;
  CHECK(hipEventElapsedTime(&ms, e0, e1));
  const double mfma_cycles = (double)WPE * iters * 8 * 32;  // matrix-pipe cycles per SIMD
  if (FORM == kVector) printf("%-8s %d waves/SIMD  %8.3f ms\n", name, WPE, ms);
  else printf("%-8s %d waves/SIMD  %8.3f ms   fraction of the MFMA peak at 2.4 GHz: %.3f\n", name, WPE, ms, mfma_cycles / (ms * 1e-3 * 2.4e9));
  fflush(stdout);
  CHECK(hipEventDestroy(e0));
  CHECK(hipEventDestroy(e1));
  return ms;
}

int main() {
  float* out;
  CHECK(hipMalloc(&out, (size_t)256 * 4 * 256 * sizeof(float)));
  const int iters = 40000;
  const double m3 = run<kMfma, 3, 40>("mfma", out, iters);
  const double v3 = run<kVector, 3, 40>("vector", out, iters);
  const double b3 = run<kBoth, 3, 40>("both", out, iters);
  printf("3 waves/SIMD: both / (mfma + vector) = %.3f, both / max(mfma, vector) = %.3f\n", b3 / (m3 + v3), b3 / (m3 > v3 ? m3 : v3));
  const double m4 = run<kMfma, 4, 30>("mfma", out, iters);
  const double v4 = run<kVector, 4, 30>("vector", out, iters);
  const double b4 = run<kBoth, 4, 30>("both", out, iters);
  printf("4 waves/SIMD: both / (mfma + vector) = %.3f, both / max(mfma, vector) = %.3f\n", b4 / (m4 + v4), b4 / (m4 > v4 ? m4 : v4));
  for (float scale : {0.0f, 1.0f}) {
    run_order<false, 2, 60>(out, iters / 4, scale);
    run_order<true, 2, 60>(out, iters / 4, scale);
    run_order<false, 3, 40>(out, iters / 4, scale);
    run_order<true, 3, 40>(out, iters / 4, scale);
  }
  CHECK(hipFree(out));
  return 0;
}
