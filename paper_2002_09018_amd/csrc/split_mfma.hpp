// fp32 products on the bf16 matrix cores (gfx950): one workgroup computes a
// 128 x 128 output tile C = opA(A) opB(B) with fp32 results.
//
// An fp32 operand is split exactly into three bf16 planes while it is staged,
//   x = p0 + p1 + p2,  p0 = bf16(x), p1 = bf16(x - p0), p2 = x - p0 - p1
// (24 significant bits are three times 8; every difference is exact), and
//   x y = p0 q0 + (p0 q1 + p1 q0) + (p1 q1 + p0 q2 + p2 q0) + the rest,
// at most 2^-24 |x y| (typically 2^-28): six v_mfma_f32_32x32x16_bf16.  Their
// products are exact; the instruction adds k 0..7 and k 8..15 to the
// accumulator one after the other, each sum rounded to nearest, but cuts the
// products of such a group at 2^-23 of the largest.  bf16 operands are one
// plane (one product for bf16 x bf16, three for bf16 x fp32, both without any
// dropped term).
//
// Why: v_mfma_f32_32x32x2_f32 gives 256 flops per cycle and compute unit, the
// bf16 instruction 4096 / 6 useful ones.  Two sets of accumulators keep
// the sums short: over the first kRun k-values the leading products go to one
// and the five others to the other; then each further run of kRun k-values
// collects its six products in the first, which is added to the second at the
// run's end.  A sum so rounds at the magnitude of a short run of terms, where
// the fp32 instruction rounds every term at the magnitude of the whole sum.
// Measured against 64 bits (32 x 32 outputs, Gaussian rows): relative error
// 6.0e-8 / 1.7e-7 / 2.0e-7 at K = 128 / 1024 / 4096, the fp32 instruction
// 2.1e-7 / 5.6e-7 / 1.1e-6.  One accumulator without runs loses 2.1e-6 on the
// diagonal of a K = 4096 Gram matrix (fp32: 8.7e-7); leading and other
// products apart without runs lose more than fp32 on the diagonal of M M for
// M = I + E with rows |E| = 1e-3 (6.1e-7 against 5.8e-7 at K = 2048; with
// runs 1.3e-7), and so gave roots of 2048 x 2048 matrices 6.2e-7 from 64 bits
// (fp32: 4.5e-7; with runs 1.6e-7).
//
// The planes of x below 2^-110 are bf16 subnormals and would lose bits (P of
// gradients around 2^-115 was 1e-6 from 64 bits, around 2^-126 2e-3), so fp32
// operands are split as 2^16 x, exact for every fp32 value, and the sums
// multiplied by 2^-16 or 2^-32 at the end.  The multiplication costs 1 to 2.5%
// of the call (two-sided updates of 1024 x 1024 9.1 -> 9.2 ms); it is left out
// where every operand is near 1 (kSplit).  Sums at or above 2^96 (2^112 with
// one fp32 operand) and elements at or above 2^112 overflow so and are
// recomputed as the next paragraph tells.
//
// Infinities and values that round up to infinity in p0 turn into NaN in the
// other planes; fix_nonfinite recomputes every non-finite output with the fp32
// instruction (fp32_block.hpp), so such inputs give what an fp32 sum gives.
//
// Tile: 4 wave64s, 2 x 2, each 64 x 64 (2 x 2 blocks of 32 x 32, 64 + 64
// accumulator registers; a bf16 x bf16 product, one per step, has no second
// set).  A stage is KS x 16 k-values of both operands,
// double-buffered; LDS holds it as the MFMA fragments themselves,
//   [16-deep step][plane][32-row block][k half][row][8 bf16],
// so a lane's fragment is one 16-byte read and a wave's is 1 KB in a row.
// While stage s is multiplied, the registers loaded during stage s - 1 are
// split and written to the other buffer, and the loads of stage s + 2 are
// issued: one barrier per stage, and a load has a whole stage to arrive.
#pragma once

#include <type_traits>

#include "fp32_block.hpp"

namespace shp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kStepB = 4096;  // bytes of one plane of a 16-deep step: 128 rows x 16 k
constexpr int kBlockB = 1024; // one 32-row block
constexpr int kHalfB = 512;   // its first or last 8 k

template <typename S>
struct Planes {
  static constexpr int n = 3;
};
template <>
struct Planes<uint16_t> {
  static constexpr int n = 1;
};
// 16-deep steps per stage, and the waves per SIMD asked of the register
// allocator.  bf16 x bf16 has one product per step and bf16 x fp32 three, so
// their stages are two steps deep (fewer barriers per product: the mixed
// update's G Rr, 444 GFLOP, 2.05 -> 1.6 ms).  Four steps for bf16 x bf16 leave
// two workgroups to a compute unit and were slower (mixed bf16 statistics 1.56
// against 1.29 ms): with one product per step the loads bound it, and more
// workgroups hide them better.
template <typename SA, typename SB>
struct SplitSteps {
  static constexpr int np = Planes<SA>::n + Planes<SB>::n;
  static constexpr int value = np == 6 ? 1 : 2;
  static constexpr int waves = np == 2 ? 4 : kMinWaves;
};

__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
  const f32x2 v = {x, y};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// Two values into their three planes (pairs of bf16, x in the low half); SC:
// of 2^16 times the values.
constexpr float kSplitScale = 65536.f;

template <bool SC>
__device__ __forceinline__ void split_pair(float x, float y, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  if constexpr (SC) {
    x *= kSplitScale;
    y *= kSplitScale;
  }
  p0 = pack_bf16(x, y);
  x -= __uint_as_float(p0 << 16);
  y -= __uint_as_float(p0 & 0xffff0000u);
  p1 = pack_bf16(x, y);
  x -= __uint_as_float(p1 << 16);
  y -= __uint_as_float(p1 & 0xffff0000u);
  p2 = pack_bf16(x, y);
}

// Staging of one operand: its 128 tile rows (the storage rows i0.. of a
// kLayoutRow operand, the storage columns of a kLayoutK one).  Tile rows past
// the operand's end are clamped to its last one (they only feed outputs that
// are not stored); k-values at or past K are staged as zeros.
template <typename S, int LAYOUT, int KS, bool SC>
struct SplitLoader;

// fp32, k contiguous: a thread takes 4 consecutive k of 2 KS rows.  Eight
// consecutive lanes hold the two k quarters of a half for four rows, so the
// 8-byte LDS writes of a wave are conflict-free.
template <int KS, bool SC>
struct SplitLoader<float, kLayoutRow, KS, SC> {
  static constexpr int PER = 2 * KS;
  static constexpr int BK = 16 * KS;
  const float* p[PER];
  float v[PER][4];
  // unit i of a thread: tile row and 4-wide k quarter of the stage
  static __device__ __forceinline__ void unit(int tid, int i, int& row, int& q) {
    const int s = (tid + i * kThreads) & 511, step = (tid + i * kThreads) >> 9;
    row = ((s >> 1) & 15) | ((s >> 6) << 4);
    q = (s & 1) | ((s >> 4) & 2) | (step << 2);
  }
  __device__ __forceinline__ void init(const Operand<float>& op, int i0, int tid) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      int row, q;
      unit(tid, i, row, q);
      p[i] = op.ptr + (int64_t)min(i0 + row, op.rows - 1) * op.ld + q * 4;
    }
  }
  __device__ __forceinline__ void load(const Operand<float>&, int k0, int K, int tid) {
    if (k0 + BK <= K) {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const f32x4u x = gload_f4(p[i] + k0);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = x[e];
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        int row, q;
        unit(tid, i, row, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = k0 + q * 4 + e < K ? gload<float>(p[i] + k0 + e) : 0.f;
      }
    }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      int row, q;
      unit(tid, i, row, q);
      char* d = lds + (q >> 2) * 3 * kStepB + (row >> 5) * kBlockB + ((q >> 1) & 1) * kHalfB + (row & 31) * 16 +
                (q & 1) * 8;
      u32x2 a, b, c;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        uint32_t t0, t1, t2;
        split_pair<SC>(v[i][2 * e], v[i][2 * e + 1], t0, t1, t2);
        a[e] = t0;
        b[e] = t1;
        c[e] = t2;
      }
      *reinterpret_cast<u32x2*>(d) = a;
      *reinterpret_cast<u32x2*>(d + kStepB) = b;
      *reinterpret_cast<u32x2*>(d + 2 * kStepB) = c;
    }
  }
};

// fp32, k the storage row: a thread takes one column and 8 consecutive k per
// step, loaded as 8 row segments shared by the wave; the transposition is
// the packing of its own registers.
template <int KS, bool SC>
struct SplitLoader<float, kLayoutK, KS, SC> {
  static constexpr int BK = 16 * KS;
  const float* p;
  float v[KS][8];
  __device__ __forceinline__ void init(const Operand<float>& op, int i0, int tid) {
    const int h = __builtin_amdgcn_readfirstlane(tid >> 7);
    p = op.ptr + (int64_t)h * 8 * op.ld + min(i0 + (tid & 127), op.cols - 1);
  }
  __device__ __forceinline__ void load(const Operand<float>& op, int k0, int K, int tid) {
    const int h = tid >> 7;
    if (k0 + BK <= K) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[s][e] = gload<float>(p + (int64_t)(k0 + 16 * s + e) * op.ld);
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[s][e] = k0 + 16 * s + h * 8 + e < K ? gload<float>(p + (int64_t)(k0 + 16 * s + e) * op.ld) : 0.f;
    }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
    const int c = tid & 127, h = tid >> 7;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      char* d = lds + s * 3 * kStepB + (c >> 5) * kBlockB + h * kHalfB + (c & 31) * 16;
      u32x4 a, b, w;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t t0, t1, t2;
        split_pair<SC>(v[s][2 * e], v[s][2 * e + 1], t0, t1, t2);
        a[e] = t0;
        b[e] = t1;
        w[e] = t2;
      }
      *reinterpret_cast<u32x4*>(d) = a;
      *reinterpret_cast<u32x4*>(d + kStepB) = b;
      *reinterpret_cast<u32x4*>(d + 2 * kStepB) = w;
    }
  }
};

// bf16, k contiguous: a thread takes 8 consecutive k of KS rows.
template <int KS, bool SC>
struct SplitLoader<uint16_t, kLayoutRow, KS, SC> {
  static constexpr int BK = 16 * KS;
  const uint16_t* p[KS];
  u32x4 v[KS];
  // eight consecutive lanes take eight rows at one k (128 bytes of LDS)
  static __device__ __forceinline__ void unit(int tid, int i, int& row, int& q) {
    constexpr int QB = KS == 2 ? 2 : 1;  // bits of the 8-wide k index
    const int s = tid + i * kThreads;
    row = (s & 7) | ((s >> (3 + QB)) << 3);
    q = (s >> 3) & ((1 << QB) - 1);
  }
  __device__ __forceinline__ void init(const Operand<uint16_t>& op, int i0, int tid) {
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      int row, q;
      unit(tid, i, row, q);
      p[i] = op.ptr + (int64_t)min(i0 + row, op.rows - 1) * op.ld + q * 8;
    }
  }
  __device__ __forceinline__ void load(const Operand<uint16_t>&, int k0, int K, int tid) {
    if (k0 + BK <= K) {
#pragma unroll
      for (int i = 0; i < KS; ++i) v[i] = gload_h8(p[i] + k0);
    } else {
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        int row, q;
        unit(tid, i, row, q);
        const int k = k0 + q * 8;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t x0 = k + 2 * e < K ? gload<uint16_t>(p[i] + k0 + 2 * e) : 0;
          const uint32_t x1 = k + 2 * e + 1 < K ? gload<uint16_t>(p[i] + k0 + 2 * e + 1) : 0;
          v[i][e] = x0 | (x1 << 16);
        }
      }
    }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      int row, q;
      unit(tid, i, row, q);
      *reinterpret_cast<u32x4*>(lds + (q >> 1) * kStepB + (row >> 5) * kBlockB + (q & 1) * kHalfB + (row & 31) * 16) =
          v[i];
    }
  }
};

// bf16, k the storage row: a thread takes two neighbouring columns and 4
// consecutive k per 16-deep step (4-byte loads of row segments).
template <int KS, bool SC>
struct SplitLoader<uint16_t, kLayoutK, KS, SC> {
  static constexpr int BK = 16 * KS;
  const uint16_t* p;
  bool pair, one;  // both columns inside the operand / at least the first
  uint32_t v[KS][4];
  __device__ __forceinline__ void init(const Operand<uint16_t>& op, int i0, int tid) {
    const int q = __builtin_amdgcn_readfirstlane(tid >> 6), c = i0 + 2 * (tid & 63);
    pair = c + 1 < op.cols;
    one = c < op.cols;
    p = op.ptr + (int64_t)q * 4 * op.ld + min(c, op.cols - 1);
  }
  __device__ __forceinline__ void load(const Operand<uint16_t>& op, int k0, int K, int tid) {
    const int q = tid >> 6;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint16_t* a = p + (int64_t)(k0 + 16 * s + e) * op.ld;
        uint32_t x = 0;
        if (k0 + BK <= K || k0 + 16 * s + q * 4 + e < K) {
          if (pair) x = gload_h2(a);
          else if (one) x = gload<uint16_t>(a);
        }
        v[s][e] = x;
      }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
    const int q = tid >> 6, c = 2 * (tid & 63);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      char* d = lds + s * kStepB + (c >> 5) * kBlockB + (q >> 1) * kHalfB + (c & 31) * 16 + (q & 1) * 8;
      const u32x2 lo = {(v[s][0] & 0xffffu) | (v[s][1] << 16), (v[s][2] & 0xffffu) | (v[s][3] << 16)};
      const u32x2 hi = {(v[s][0] >> 16) | (v[s][1] & 0xffff0000u), (v[s][2] >> 16) | (v[s][3] & 0xffff0000u)};
      *reinterpret_cast<u32x2*>(d) = lo;
      *reinterpret_cast<u32x2*>(d + 16) = hi;
    }
  }
};

// What a product of scaled operands is multiplied by (bf16 ones are not scaled).
constexpr float split_down(int npa, int npb) {
  return (npa > 1 ? 1.f / kSplitScale : 1.f) * (npb > 1 ? 1.f / kSplitScale : 1.f);
}

constexpr int kRun = 256;  // k-values of one accumulation run

// Accumulators of one wave (64 x 64): c the run in progress, t the first
// run's smaller products and the runs before; fold leaves the sum in c.
template <int NPA, int NPB>
struct SplitAcc {
  static constexpr int NB = 2;
  static constexpr bool kRuns = NPA + NPB > 2;
  typedef typename Mfma<float>::acc_t acc_t;
  acc_t c[NB][NB], t[NB][NB];

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) c[i][j][v] = t[i][j][v] = 0.f;
  }
  __device__ __forceinline__ void flush() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          t[i][j][v] += c[i][j][v];
          c[i][j][v] = 0.f;
        }
  }
  template <bool SC>
  __device__ __forceinline__ void fold() {
    if (!kRuns) return;
    constexpr float down = SC ? split_down(NPA, NPB) : 1.f;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) c[i][j][v] = (c[i][j][v] + t[i][j][v]) * down;
  }
  // One 16-deep step over the blocks of MODE; a, b: the step's planes at the
  // wave's first row block.  FIRST: a step of the first run.
  template <int MODE, bool FIRST>
  __device__ __forceinline__ void step(const char* a, const char* b, int lane) {
    bf16x8 fa[NPA][NB], fb[NPB][NB];
    const int lo = lane * 16;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      if (q < NPA)
#pragma unroll
        for (int i = 0; i < NB; ++i)
          if (block_used<MODE, NB>(i, NB - 1))
            fa[q][i] = *reinterpret_cast<const bf16x8*>(a + q * kStepB + i * kBlockB + lo);
      if (q < NPB)
#pragma unroll
        for (int j = 0; j < NB; ++j) fb[q][j] = *reinterpret_cast<const bf16x8*>(b + q * kStepB + j * kBlockB + lo);
    }
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int pa = 0; pa < NPA; ++pa) {
        const int pb = s - pa;
        if (pb < 0 || pb >= NPB) continue;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if (!block_used<MODE, NB>(i, j)) continue;
            acc_t& d = FIRST && s > 0 ? t[i][j] : c[i][j];
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[pa][i], fb[pb][j], d, 0, 0, 0);
          }
      }
  }
};

template <typename SA, typename SB>
struct SplitShm {
  static constexpr int KS = SplitSteps<SA, SB>::value;
  static constexpr int a = KS * Planes<SA>::n * kStepB, b = KS * Planes<SB>::n * kStepB;
  static constexpr int stage = a + b;
  // two stages; at least the epilogue's four 32 x 64 fp32 slices
  static constexpr int bytes = 2 * stage < 32768 ? 32768 : 2 * stage;
};

template <int MODE, bool SC, typename SA, int LA, typename SB, int LB>
__device__ __forceinline__ void split_loop(SplitAcc<Planes<SA>::n, Planes<SB>::n>& acc, const Operand<SA>& A,
                                           const Operand<SB>& B, int m0, int n0, int K, char* smem, int wm0,
                                           int wn0) {
  typedef SplitShm<SA, SB> Shm;
  constexpr int KS = Shm::KS, BK = 16 * KS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int nst = (K + BK - 1) / BK;
  if (nst <= 0) return;
  SplitLoader<SA, LA, KS, SC> la;
  SplitLoader<SB, LB, KS, SC> lb;
  la.init(A, m0, tid);
  lb.init(B, n0, tid);
  la.load(A, 0, K, tid);
  lb.load(B, 0, K, tid);
  la.store(smem, tid);
  lb.store(smem + Shm::a, tid);
  if (nst > 1) {
    la.load(A, BK, K, tid);
    lb.load(B, BK, K, tid);
  }
  __syncthreads();
  auto stage = [&](int st, auto first) {
    char* cur = smem + (st & 1) * Shm::stage;
    char* nxt = smem + ((st & 1) ^ 1) * Shm::stage;
    if (st + 1 < nst) {
      la.store(nxt, tid);
      lb.store(nxt + Shm::a, tid);
    }
    if (st + 2 < nst) {
      la.load(A, (st + 2) * BK, K, tid);
      lb.load(B, (st + 2) * BK, K, tid);
    }
    const char* a = cur + (wm0 >> 5) * kBlockB;
    const char* b = cur + Shm::a + (wn0 >> 5) * kBlockB;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      acc.template step<MODE, decltype(first)::value>(a + s * Planes<SA>::n * kStepB, b + s * Planes<SB>::n * kStepB,
                                                      lane);
    __syncthreads();
  };
  typedef SplitAcc<Planes<SA>::n, Planes<SB>::n> Acc;
  if constexpr (!Acc::kRuns) {
    for (int st = 0; st < nst; ++st) stage(st, std::false_type{});
  } else {
    constexpr int kStages = kRun / BK;
    for (int st = 0; st < min(nst, kStages); ++st) stage(st, std::true_type{});
    for (int st = kStages; st < nst; ++st) {
      if (st % kStages == 0) acc.flush();
      stage(st, std::false_type{});
    }
  }
}

// Recomputes the non-finite outputs of a wave (one copy of the code for its
// four blocks: it is rarely taken and would quadruple the epilogue).
template <int NPA, int NPB, typename SA, int LA, typename SB, int LB>
__device__ __forceinline__ void fix_nonfinite(SplitAcc<NPA, NPB>& acc, const Operand<SA>& A, const Operand<SB>& B,
                                              int wm0, int wn0, int K) {
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) bad |= !finite_f32(acc.c[i][j][v]);
  if (__builtin_expect(!__any(bad), 1)) return;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    block_acc x;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float lo = q & 1 ? acc.c[0][1][v] : acc.c[0][0][v], hi = q & 1 ? acc.c[1][1][v] : acc.c[1][0][v];
      x[v] = q & 2 ? hi : lo;
    }
    fp32_repair<SA, LA, SB, LB>(x, A, B, wm0 + (q >> 1) * 32, wn0 + (q & 1) * 32, K);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc.c[0][0][v] = q == 0 ? x[v] : acc.c[0][0][v];
      acc.c[0][1][v] = q == 1 ? x[v] : acc.c[0][1][v];
      acc.c[1][0][v] = q == 2 ? x[v] : acc.c[1][0][v];
      acc.c[1][1][v] = q == 3 ? x[v] : acc.c[1][1][v];
    }
  }
}

// How a product is formed: by the split alone, with its non-finite outputs
// recomputed, that and short contractions in fp64 (where only the device knows
// K), or in fp64 (launches of short contractions).
enum { kSplit = 0, kSplitRepair = 1, kSplitRepairShort = 2, kShort = 3 };

// The wave's blocks of a short contraction (those inside the output).
template <int NPA, int NPB, typename SA, int LA, typename SB, int LB>
__device__ __forceinline__ void short_blocks(SplitAcc<NPA, NPB>& acc, const Operand<SA>& A, const Operand<SB>& B,
                                             int wm0, int wn0, int K) {
  if (K <= 0) return;  // no active row: the sums are zero
  const int rows = LA == kLayoutRow ? A.rows : A.cols, cols = LB == kLayoutRow ? B.rows : B.cols;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      __builtin_amdgcn_sched_barrier(0);  // one block's registers at a time
      if (wm0 + 32 * i >= rows || wn0 + 32 * j >= cols) continue;
      acc.c[i][j] = fp64_product<SA, LA, SB, LB>(A, B, wm0 + 32 * i, wn0 + 32 * j, K);
    }
}

// Full k-loop of one 128 x 128 output tile; results in acc.c.  diag:
// diagonal tile of a symmetric output (squares and block sets of wave_role).
template <int MODE, typename SA, int LA, typename SB, int LB>
__device__ __forceinline__ void split_mma(SplitAcc<Planes<SA>::n, Planes<SB>::n>& acc, const Operand<SA>& A,
                                          const Operand<SB>& B, int m0, int n0, int K, char* smem, bool diag) {
  const int wave = threadIdx.x >> 6;
  const WaveRole ro = wave_role(wave, diag);
  constexpr bool SC = MODE != kSplit;
  if (MODE == kShort || (MODE == kSplitRepairShort && K <= kShortK)) {
    short_blocks<Planes<SA>::n, Planes<SB>::n, SA, LA, SB, LB>(acc, A, B, m0 + ro.wm, n0 + ro.wn, K);
    return;
  }
  if (ro.mode == kBlocksAll)
    split_loop<kBlocksAll, SC, SA, LA, SB, LB>(acc, A, B, m0, n0, K, smem, ro.wm, ro.wn);
  else if (ro.mode == kBlocksUpper)
    split_loop<kBlocksUpper, SC, SA, LA, SB, LB>(acc, A, B, m0, n0, K, smem, ro.wm, ro.wn);
  else if (ro.mode == kBlocksTopHalf)
    split_loop<kBlocksTopHalf, SC, SA, LA, SB, LB>(acc, A, B, m0, n0, K, smem, ro.wm, ro.wn);
  else
    split_loop<kBlocksBottomHalf, SC, SA, LA, SB, LB>(acc, A, B, m0, n0, K, smem, ro.wm, ro.wn);
  acc.template fold<SC>();
  if constexpr (MODE != kSplit && Planes<SA>::n + Planes<SB>::n > 2)
    fix_nonfinite<Planes<SA>::n, Planes<SB>::n, SA, LA, SB, LB>(acc, A, B, m0 + ro.wm, n0 + ro.wn, K);
}

}  // namespace shp
