// Products of launches with few 128 x 128 tiles: one wave per 32 x 32 output
// block, operands read from global memory straight into MFMA fragments.
//
// What bounds such launches: a tile of split_mfma.hpp walks its contraction
// in 16-deep stages, and with one workgroup on a compute unit a stage takes
// about 1 us (its loads, split, LDS writes, barrier and MFMAs follow each
// other); a single 128 x 128 x 128 product took 20 us on one compute unit
// with 255 idle.  Here the 16 blocks of a tile go to 16 waves on different
// compute units, without LDS or barriers, and a step is 6 MFMAs and the
// splitting of 16 values per lane.  Each block repeats that splitting, so the
// form only pays while most of the chip would be idle (kDirectBlocks).
//
// The arithmetic of every output is that of split_mfma.hpp, operation for
// operation (same MFMA, same order of products, same runs), so results do
// not depend on which form a launch takes.
#pragma once

#include "split_mfma.hpp"

namespace shp {

// The planes of a step's fragment.
template <bool SC, typename S, int LAYOUT>
__device__ __forceinline__ void frag_planes(const DirectFrag<S, LAYOUT>& x, bf16x8 (&f)[Planes<S>::n]) {
  u32x4 a, b, c;
  if constexpr (Planes<S>::n == 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = (uint32_t)x.v[2 * e] | ((uint32_t)x.v[2 * e + 1] << 16);
    f[0] = __builtin_bit_cast(bf16x8, a);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t t0, t1, t2;
      split_pair<SC>(x.v[2 * e], x.v[2 * e + 1], t0, t1, t2);
      a[e] = t0;
      b[e] = t1;
      c[e] = t2;
    }
    f[0] = __builtin_bit_cast(bf16x8, a);
    f[1] = __builtin_bit_cast(bf16x8, b);
    f[2] = __builtin_bit_cast(bf16x8, c);
  }
}

template <bool FIRST, int NPA, int NPB>
__device__ __forceinline__ void direct_step(const bf16x8 (&fa)[NPA], const bf16x8 (&fb)[NPB], block_acc& c,
                                            block_acc& t) {
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int pa = 0; pa < NPA; ++pa) {
      const int pb = s - pa;
      if (pb < 0 || pb >= NPB) continue;
      block_acc& d = FIRST && s > 0 ? t : c;
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[pa], fb[pb], d, 0, 0, 0);
    }
}

// The 32 x 32 block at (m0, n0), in the accumulator layout (FIX: non-finite
// outputs are recomputed in fp32).
template <bool FIX, typename SA, int LA, typename SB, int LB>
__device__ __forceinline__ block_acc direct_mma(const Operand<SA>& A, const Operand<SB>& B, int m0, int n0, int K) {
  constexpr int NPA = Planes<SA>::n, NPB = Planes<SB>::n;
  constexpr bool kRuns = NPA + NPB > 2;
  const int lane = threadIdx.x & 63;
  block_acc c, t;
#pragma unroll
  for (int v = 0; v < 16; ++v) c[v] = t[v] = 0.f;
  // two steps of operands in flight
  DirectFrag<SA, LA> a0, a1;
  DirectFrag<SB, LB> b0, b1;
  a0.init(A, m0, lane);
  b0.init(B, n0, lane);
  a1 = a0;
  b1 = b0;
  a0.load(0, K);
  b0.load(0, K);
  if (K > 16) {
    a1.load(16, K);
    b1.load(16, K);
  }
  auto steps = [&](int k0, int k1, auto first) {
#pragma unroll 1
    for (int k = k0; k < k1; k += 32) {
      bf16x8 fa[NPA], fb[NPB];
      frag_planes<FIX>(a0, fa);
      frag_planes<FIX>(b0, fb);
      if (k + 32 < K) {
        a0.load(k + 32, K);
        b0.load(k + 32, K);
      }
      direct_step<decltype(first)::value, NPA, NPB>(fa, fb, c, t);
      if (k + 16 >= k1) break;
      frag_planes<FIX>(a1, fa);
      frag_planes<FIX>(b1, fb);
      if (k + 48 < K) {
        a1.load(k + 48, K);
        b1.load(k + 48, K);
      }
      direct_step<decltype(first)::value, NPA, NPB>(fa, fb, c, t);
    }
  };
  if constexpr (!kRuns) {
    steps(0, K, std::false_type{});
  } else {
    steps(0, min(K, kRun), std::true_type{});
#pragma unroll 1
    for (int k = kRun; k < K; k += kRun) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        t[v] += c[v];
        c[v] = 0.f;
      }
      steps(k, min(K, k + kRun), std::false_type{});
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = (c[v] + t[v]) * (FIX ? split_down(NPA, NPB) : 1.f);
    if constexpr (FIX) fp32_repair<SA, LA, SB, LB>(c, A, B, m0, n0, K);
  }
  return c;
}

// Sub-block b of a 128 x 128 tile (16 of them; those strictly below the
// diagonal of a symmetric output's diagonal tile are not computed).
__device__ __forceinline__ void sub_block(int b, int& i, int& j) {
  i = (b >> 2) * 32;
  j = (b & 3) * 32;
}

}  // namespace shp
