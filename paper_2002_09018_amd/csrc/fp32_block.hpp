// 32 x 32 output blocks that the bf16 matrix cores should not form, one wave
// each, operands read from global memory straight into fragments.
//
// The products of split_mfma.hpp are 2.7 times as fast as the fp32
// instruction's.  What they cannot do as well:
// - Contractions of at most kShortK (fp64_product).  The bf16 instruction cuts
//   the products of a group of eight k at 2^-23 of the group's largest, and the
//   split drops products of up to 2^-24; a long sum gains far more than that,
//   a short one need not.  Root mean square error of a Gram matrix in units of
//   2^-24, fp32 instruction against split: Gaussian rows 0.42 / 0.44 at K = 1;
//   one column 30 times the others 0.42 / 0.57 at K = 2, 0.57 / 0.83 at 12, 1.5
//   / 0.75 at 16; entries x exp(3 x), its diagonal 1.14 / 1.25 at 16, 1.30 /
//   1.32 at 24, 1.53 / 1.33 at 32.  Such a product is bound by its output, so
//   it is formed in fp64 (exact products, one rounding; 0.42 to 0.43
//   everywhere) and costs no more (20 statistics of 1 x 4096 608 us, split 624,
//   fp32 instruction 869; 40 of 16 x 4096 1287, 1209, 1477).  Up to K = 32 it
//   would (60 of 32 x 2048 737, 506, 656).
// - Outputs that the split leaves non-finite (an infinity or a NaN among the
//   operands, a value that rounds up to infinity in bf16, an overflow): they
//   are recomputed with v_mfma_f32_32x32x2_f32, so that they are what an fp32
//   sum gives (fp32_repair).
#pragma once

#include "tile_mfma.hpp"

namespace shp {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// 16-byte and 4-byte vectors at element alignment (global loads only)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32u __attribute__((aligned(2)));

// Global loads at element alignment (the typedefs' alignment would be lost
// on a template argument).
__device__ __forceinline__ f32x4u gload_f4(const float* p) {
  return *(const __attribute__((address_space(1))) f32x4u*)(p);
}
__device__ __forceinline__ u32x4u gload_h8(const uint16_t* p) {
  return *(const __attribute__((address_space(1))) u32x4u*)(p);
}
__device__ __forceinline__ uint32_t gload_h2(const uint16_t* p) {
  return *(const __attribute__((address_space(1))) u32u*)(p);
}

typedef Mfma<float>::acc_t block_acc;

// Fragment source of one wave: rows (kLayoutRow) or columns (kLayoutK) i0 +
// (lane & 31) of an operand, the lane's 8 of 16 k; past the operand's end its
// last row or column is read (those outputs are not stored), past K zeros.
template <typename S, int LAYOUT>
struct DirectFrag {
  const S* p;
  int64_t step;  // elements between consecutive k
  int k;         // the lane's first k of the step
  S v[8];
  __device__ __forceinline__ void init(const Operand<S>& op, int i0, int lane) {
    const int i = i0 + (lane & 31);
    k = (lane >> 5) * 8;
    if (LAYOUT == kLayoutRow) {
      p = op.ptr + (int64_t)min(i, op.rows - 1) * op.ld;
      step = 1;
    } else {
      p = op.ptr + min(i, op.cols - 1);
      step = op.ld;
    }
  }
  __device__ __forceinline__ void load(int k0, int K) {
    if (k0 + 16 <= K) {
      const S* q = p + (k0 + k) * step;
      if constexpr (LAYOUT == kLayoutRow && sizeof(S) == 4) {
        const f32x4u a = gload_f4(q), b = gload_f4(q + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = a[e];
          v[4 + e] = b[e];
        }
      } else if constexpr (LAYOUT == kLayoutRow) {
        const u32x4u a = gload_h8(q);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[2 * e] = (S)(a[e] & 0xffffu);
          v[2 * e + 1] = (S)(a[e] >> 16);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = gload<S>(q + e * step);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = k0 + k + e < K ? gload<S>(p + (k0 + k + e) * step) : (S)0;
    }
  }
};

// Element (tile row or column i, k) of an operand, in fp32.
template <typename S, int LAYOUT>
__device__ __forceinline__ float operand_at(const Operand<S>& op, int i, int k) {
  const int64_t at = LAYOUT == kLayoutK ? (int64_t)k * op.ld + min(i, op.cols - 1)
                                        : (int64_t)min(i, op.rows - 1) * op.ld + k;
  return cvt<float, S>(gload<S>(op.ptr + at));
}

__device__ __forceinline__ bool finite_f32(float x) { return fabsf(x) <= 3.402823466e38f; }


// The non-finite values of x, recomputed: block (m0, n0) of the product.  A
// NaN stays one whatever follows, so the pass ends once every such value is
// one; an infinity can still turn into a NaN and takes the whole contraction.
//
// What bounds it: 8 MFMAs of 64 cycles a step, one after the other, against
// the latency of 4 KB of operands; a pass over all of a product runs at about
// 65 TFLOP/s.  64 blocks of 1024 x 1024, statistics and two-sided update, in
// ms, against a loop over k in one lane per output (and, for the finite
// gradient, the same): 1.3 and 2.4 finite, 1.4 and 3.4 (13 and 83) with one
// NaN in each gradient, 1.6 and 4.9 (13 and 83) with one infinity, 1.3 and 2.2
// (138 and 138) all NaN, 3.2 and 6.0 (138 and 141) all infinite.  Two by two
// blocks a pass share their fragments but leave no registers for two steps in
// flight: 2.0 and 5.1 with one infinity.
template <typename SA, int LA, typename SB, int LB>
__device__ __forceinline__ void fp32_repair(block_acc& x, const Operand<SA>& A, const Operand<SB>& B, int m0, int n0,
                                            int K) {
  bool bad = false;
#pragma unroll
  for (int v = 0; v < 16; ++v) bad |= !finite_f32(x[v]);
  if (__builtin_expect(!__any(bad), 1)) return;
  const int lane = threadIdx.x & 63;
  DirectFrag<SA, LA> a0, a1;
  DirectFrag<SB, LB> b0, b1;
  a0.init(A, m0, lane);
  b0.init(B, n0, lane);
  a1 = a0;
  b1 = b0;
  block_acc c;
#pragma unroll
  for (int v = 0; v < 16; ++v) c[v] = 0.f;
  auto step = [&](const DirectFrag<SA, LA>& a, const DirectFrag<SB, LB>& b) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(cvt<float, SA>(a.v[e]), cvt<float, SB>(b.v[e]), c, 0, 0, 0);
  };
  // two steps of operands in flight (past K they are zeros)
  a0.load(0, K);
  b0.load(0, K);
#pragma unroll 1
  for (int k = 0; k < K; k += 32) {
    a1.load(k + 16, K);
    b1.load(k + 16, K);
    step(a0, b0);
    a0.load(k + 32, K);
    b0.load(k + 32, K);
    step(a1, b1);
    bool open = false;
#pragma unroll
    for (int v = 0; v < 16; ++v) open |= !finite_f32(x[v]) && c[v] == c[v];
    if (!__any(open)) break;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) x[v] = finite_f32(x[v]) ? x[v] : c[v];
}

constexpr int kShortK = 16;

// Block (m0, n0) of a product of 1 <= K <= kShortK.
template <typename SA, int LA, typename SB, int LB>
__device__ __forceinline__ block_acc fp64_product(const Operand<SA>& A, const Operand<SB>& B, int m0, int n0, int K) {
  typedef Mfma<double> D;
  const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
  D::acc_t c[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) c[i][j][v] = 0.0;
  // every operand first, then the products (a step at a time waited for its
  // loads)
  constexpr int kSteps = kShortK / D::kK;
  float a[kSteps][2], b[kSteps][2];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int k = s * D::kK + g, at = min(k, K - 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[s][i] = operand_at<SA, LA>(A, m0 + 16 * i + i16, at);
      b[s][i] = operand_at<SB, LB>(B, n0 + 16 * i + i16, at);
      if (k >= K) a[s][i] = b[s][i] = 0.f;
    }
  }
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    if (s * D::kK >= K) break;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) c[i][j] = D::mma((double)a[s][i], (double)b[s][j], c[i][j]);
  }
  // to the layout of a 32 x 32 block: value v of a lane is row 8 (v / 4) + 4
  // half + v % 4 of its column
  block_acc x;
  const int right = (lane >> 4) & 1, half = lane >> 5;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int src = ((v & 3) * 16 + i16) * 4, i = v >> 3, w = ((v >> 2) & 1) * 2;
    float y[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        y[j][h] = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int((float)c[i][j][w + h])));
    const float lo = half ? y[0][1] : y[0][0], hi = half ? y[1][1] : y[1][0];
    x[v] = right ? hi : lo;
  }
  return x;
}

}  // namespace shp
