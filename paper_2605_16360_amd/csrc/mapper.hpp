// Device-side pieces that the mapper's two sets of kernels share: the large-tile kernels of mapper.hip and the
// small-tile kernels of mapper_small.hip, which run short inputs.
#pragma once
#include "common.hpp"
#include "context.hpp"

namespace pkv {
namespace {

typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

constexpr float kNegInf = -__builtin_huge_valf();
constexpr int kDT = 512;    // d_time
constexpr int kBlk = 128;   // rows of a block of the large-tile encoder kernels
constexpr int kWin = 2048;  // window length
constexpr int kStride = 1024;
constexpr int kHeads = 8;   // encoder heads, 64 wide
constexpr int kRangeWords = 16;  // partial maxima of |score| per layer of a batch

// The distinct proxy layers that one batch of launches handles, and the target layers lo .. hi-1 that each serves.
struct LayerBatch {
  int n;
  int ls[kMaxBatch], lo[kMaxBatch], hi[kMaxBatch];
};

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

__device__ __forceinline__ uint16_t to_h(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }

// 8 chunks of 16 bytes per 128-byte LDS row, XOR-swizzled so that 16-byte tile stores and MFMA fragment reads
// (32 consecutive rows, same chunk) both spread over all LDS banks
__device__ __forceinline__ int swz8(int row) { return (row & 7) ^ ((row >> 3) & 1); }

constexpr int kXcds = 8;

// Where four columns n .. n+3 (n % 4 == 0) of row `row` of the residual stream lie, in units of 16 bytes.  A block of 128 rows is
// kept as the accumulators of encoder_block_kernel hold it, so that its loads and stores are whole kilobytes: by the wave that owns
// 128 columns, by 16 rows, by 16 columns; then a unit per lane.
__device__ __forceinline__ size_t block_x4(int64_t row, int n) {
  const int r = (int)(row & (kBlk - 1));
  return ((((size_t)(row / kBlk) * 4 + (n >> 7)) * 8 + (r >> 4)) * 8 + ((n >> 4) & 7)) * 64 + ((n >> 2) & 3) * 16 + (r & 15);
}

// ------------------------------------------------------------------------------------------
// Range of the first convolution's output.  The scores of Sec. 3 in their sum form are not bounded by one (an
// attention sink collects up to G * N_q), so GELU(BN(conv1(x))) can exceed what IEEE half holds.  The operand of the
// second convolution is therefore stored as half(h1 * 2^-s) with one exponent s per proxy layer, taken from the
// largest score of the layer, and the second convolution's per-channel scale is multiplied by 2^s: exact, since only
// the exponent moves.  s = 0 (nothing changes) whenever the bound below stays under 2^15.
// |h1| <= |scale_c| * sum |w_c| * max|x| + |shift_c| <= cw * max|x| + cs  (|GELU(y)| <= |y|)
// words: the bits of |x|'s partial maxima over one layer, written by absmax_kernel
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int stem_exponent(const uint32_t* words, float cw, float cs) {
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < kRangeWords; ++i) m = words[i] > m ? words[i] : m;
  const float bound = __builtin_fmaf(cw, __uint_as_float(m), cs);
  const int e = (int)((__float_as_uint(bound) >> 23) & 255u) - 127;  // floor(log2(bound)); 128 for inf or NaN
  return e >= 15 ? e - 14 : 0;                                        // bound * 2^-s < 2^15
}
__device__ __forceinline__ float exp2_int(int s) { return __uint_as_float((uint32_t)(127 + s) << 23); }

constexpr float kAttnLazy = 8.0f;

// max over the 32 elements of two accumulator tiles (v_max3 tree)
__device__ __forceinline__ float max16_8(const f32x16& a, const f32x16& b) {
  float m = max3f(a[0], a[1], a[2]);
#pragma unroll
  for (int r = 3; r < 15; r += 2) m = max3f(m, a[r], a[r + 1]);
  m = max3f(m, a[15], b[0]);
#pragma unroll
  for (int r = 1; r < 15; r += 2) m = max3f(m, b[r], b[r + 1]);
  return __builtin_fmaxf(m, b[15]);
}

// rows of every layer of a batch on a GEMM's M axis: `valid` of them, `stride` apart (a multiple of 256)
struct RowSpace {
  int layers, valid, stride;
  int64_t a_layer;  // elements between the A rows of two layers
};

// Where a lane's buffers lie for a plan: all layers of a batch one behind the other in each.  h1, qk and the two behind it, hid and zg
// share `work`: each is read for the last time before the next one of them is written.
struct LanePointers {
  uint16_t* h1;     // fp16 [(N+2), c_mid]  stem conv1 output with one zero row at each end
  float* x;
  uint16_t *xb, *qk;  // qk: fp16 [Tp, 2*d_time]  q and k of the current layer
  uint16_t* vt;     // fp16 [heads, 64, Tp]  v transposed per head (small tiles)
  uint16_t* ao;     // fp16 [Tp, d_time]    attention output of the small tiles; of the large ones, whose q, k and v lie in blocks at qk, in xb
  uint16_t* hid;    // fp16 [Tp, d_ffn]
  uint16_t* zg;     // fp16 [Np, d_time]    overlap-averaged encoder output
  float *s3, *pre;
  uint32_t* range;
};
inline LanePointers lane_pointers(const proxykv_config& c, const MapPlan& p, const MapperWorkspace& m) {
  uint16_t* work = (uint16_t*)m.work.ptr;
  const size_t n = (size_t)p.batch, d = (size_t)c.d_time;
  uint16_t* vt = work + n * p.Tp * 2 * d;
  uint16_t* ao = vt + n * p.Tp * d;
  return {work, (float*)m.x.ptr, (uint16_t*)m.xb.ptr, work, vt, ao, work, work, (float*)m.s3.ptr, (float*)m.pre.ptr, (uint32_t*)m.range.ptr};
}

#define PKV_TRY(call)                  \
  do {                                 \
    hipError_t e_ = (call);            \
    if (e_ != hipSuccess) return e_;   \
  } while (0)

}  // namespace

// Launch `li` of the large-tile encoder (mapper_block.hip): all of layer li - 1 behind its attention, then q, k and v of layer li; the
// first has only the latter, the last (li = n_enc_layers) only the former.
hipError_t launch_encoder_block(const proxykv_ctx* ctx, const MapPlan& p, int n_layers, int li, float* x, const uint16_t* ao, uint16_t* qkv,
                                hipStream_t stream);

// Second stem convolution, encoder and stage-3 inner products of one batch with the kernels for few rows
// (mapper_small.hip): from h1 to s3.
hipError_t mapper_small_body(proxykv_ctx* ctx, const MapperWorkspace& ws, const MapPlan& p, int n_layers, int64_t N, hipStream_t stream);

}  // namespace pkv
