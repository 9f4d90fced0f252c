// MFMA tile machinery for gfx950 (CDNA4): one workgroup computes a 128 x 128
// output tile C[m0:m0+128, n0:n0+128] = sum_k opA[m, k] * opB[k, n].
//
// Workgroup: 256 threads = 4 wave64s arranged 2 x 2, each owning a 64 x 64
// sub-tile.  This file holds what fp32 and fp64 products share (tile maps,
// wave roles, accumulator layouts) and the fp64 products: a wave's sub-tile is
// a grid of 4 x 4 blocks of 16 x 16 (v_mfma_f64_16x16x4_f64), and the k
// dimension is streamed through LDS in stages of kBK = 16, double-buffered:
// the global loads of stage s+1 are in flight in registers while the MFMAs of
// stage s run.  fp32 results are formed by split_mfma.hpp.
//
// Each operand stage is copied into LDS in its global orientation, with
// 16-byte loads and 16-byte LDS stores (no transpose):
//   kLayoutK   the stage is read from storage rows k0..k0+kBK, columns
//              i0..i0+128 (the operand's contraction index is its storage row:
//              B of C = A B, or A of C = A^T B, or any symmetric operand);
//              LDS [k][i], unpadded.
//   kLayoutRow the stage is read from storage rows i0..i0+128, columns
//              k0..k0+kBK (contraction index contiguous: A of C = A B,
//              B of C = A B^T); LDS [i][k] with a 16-byte row pad.
// Within a stage, lane group g (lanes with the same lane / kM) takes the
// contraction indices g*KS .. g*KS+KS-1 over the KS MFMA k-steps (a
// permutation of k shared by both operands, so the sum is unchanged).  A
// kLayoutRow fragment of a lane is then KS consecutive elements, read with
// 16-byte LDS loads one chunk of VP k-steps at a time; a kLayoutK fragment is
// one element per k-step.  Stages go through registers: full, aligned stages
// with 16-byte loads, others with bounds checks (out-of-range elements are
// loaded as 0).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace shp {

// Minimum waves per SIMD requested from the register allocator
// (__launch_bounds__ second argument): 2 for every product kernel (the fp32
// products hold 128 accumulator registers per lane, the fp64 ones 128).
constexpr int kMinWaves = 2;

constexpr int kTile = 128;
constexpr int kThreads = 256;
constexpr int kWaveTile = 64;

enum { kLayoutK = 0, kLayoutRow = 1 };

template <typename T>
struct Mfma;

template <>
struct Mfma<float> {
  static constexpr int kM = 32;   // MFMA block edge
  static constexpr int kAcc = 16; // accumulator elements per lane per block
  typedef float acc_t __attribute__((ext_vector_type(16)));
  // Position of accumulator element v of `lane` inside a 32 x 32 block.
  static __device__ __forceinline__ int row(int lane, int v) {
    return (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
  }
  static __device__ __forceinline__ int col(int lane) { return lane & 31; }
};

template <>
struct Mfma<double> {
  static constexpr int kBK = 16;  // k-depth of one LDS stage
  static constexpr int kM = 16;
  static constexpr int kK = 4;    // k-depth of one MFMA
  static constexpr int kAcc = 4;
  typedef double acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return v * 4 + (lane >> 4); }
  static __device__ __forceinline__ int col(int lane) { return lane & 15; }
};

// Row pitch (elements) of one LDS stage.  kLayoutK: [k][128] rows read as
// contiguous runs (no pad needed: measured conflict-free).  kLayoutRow:
// [128][kBK] rows padded by 16 bytes, so the 16-byte fragment reads of 8
// consecutive rows fall in distinct banks and every row stays 16-byte aligned.
template <typename T, int LAYOUT>
struct Pitch {
  static constexpr int value =
      LAYOUT == kLayoutK ? kTile : Mfma<T>::kBK + 16 / (int)sizeof(T);
};

// Elements of one operand stage in LDS.
template <typename T, int LAYOUT>
struct StageElems {
  static constexpr int value = (LAYOUT == kLayoutK ? Mfma<T>::kBK : kTile) * Pitch<T, LAYOUT>::value;
  static_assert(value * (int)sizeof(T) % 16 == 0, "stages must stay 16-byte aligned");
};


template <typename T, typename S>
__device__ __forceinline__ T cvt(S x) { return (T)x; }
template <>
__device__ __forceinline__ float cvt<float, uint16_t>(uint16_t x) {
  return __uint_as_float(((uint32_t)x) << 16);
}

// Global-memory (address space 1) access: keeps operand loads off the flat
// path, whose completion counter is shared with LDS and would make every LDS
// wait also wait for the prefetch of the next stage.
template <typename V>
__device__ __forceinline__ V gload(const void* p) {
  return *(const __attribute__((address_space(1))) V*)(p);
}
template <typename V>
__device__ __forceinline__ void gstore(void* p, V v) {
  *(__attribute__((address_space(1))) V*)(p) = v;
}

// A matrix operand as stored: row-major, `rows` x `cols`, row stride `ld`.
template <typename S>
struct Operand {
  const S* ptr;
  int64_t ld;
  int rows, cols;
  bool aligned;  // ptr and ld allow 16-byte vector loads (read by the fp64 staging)
};

// Per-thread staging registers for one operand stage (fp64).
template <typename T, int LAYOUT>
struct Loader {
  typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
  static constexpr int VE = 16 / (int)sizeof(T);
  static constexpr int BK = Mfma<T>::kBK;
  static constexpr int NVEC = BK * kTile / VE;
  static constexpr int PER = NVEC / kThreads;
  static constexpr int LDP = Pitch<T, LAYOUT>::value;
  static_assert(NVEC % kThreads == 0, "stage must split evenly over the workgroup");
  V buf[PER];

  // Storage coordinates (relative to the stage origin) of vector slot i.
  static __device__ __forceinline__ void slot(int tid, int i, int& sr, int& sc) {
    const int v = tid + i * kThreads;
    constexpr int VPR = (LAYOUT == kLayoutK ? kTile : BK) / VE;
    sr = v / VPR;
    sc = (v % VPR) * VE;
  }

  // Whether the stage with storage origin (r0, c0) lies inside the operand
  // and is 16-byte aligned (plain 16-byte loads, no bounds checks).
  static __device__ __forceinline__ bool full(const Operand<T>& op, int r0, int c0) {
    constexpr int SR = LAYOUT == kLayoutK ? BK : kTile;
    constexpr int SC = LAYOUT == kLayoutK ? kTile : BK;
    return op.aligned && (r0 + SR <= op.rows) && (c0 + SC <= op.cols);
  }

  // Global -> registers, the whole stage at (r0, c0): one branch for the
  // stage (a branch per slot makes the compiler wait for each 16-byte load
  // before issuing the next).
  __device__ __forceinline__ void load(const Operand<T>& op, int r0, int c0, int tid) {
    if (full(op, r0, c0)) {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        int sr, sc;
        slot(tid, i, sr, sc);
        buf[i] = gload<V>(op.ptr + (int64_t)(r0 + sr) * op.ld + (c0 + sc));
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        int sr, sc;
        slot(tid, i, sr, sc);
        const int gr = r0 + sr;
#pragma unroll
        for (int e = 0; e < VE; ++e) {
          const int gc = c0 + sc + e;
          buf[i][e] = (gr < op.rows && gc < op.cols) ? gload<T>(op.ptr + (int64_t)gr * op.ld + gc) : (T)0;
        }
      }
    }
  }

  // Registers -> LDS stage.
  __device__ __forceinline__ void store(T* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      int sr, sc;
      slot(tid, i, sr, sc);
      *reinterpret_cast<V*>(lds + sr * LDP + sc) = buf[i];
    }
  }
};

// Which MFMA blocks of its 64 x 64 square a wave computes.  On a diagonal
// tile of a symmetric output only the upper triangle is stored: the two
// waves on the diagonal skip their blocks below it, and the upper-right
// square is split by block rows between its own wave and the wave of the
// lower-left square (never stored), so no wave idles.
enum : int { kBlocksAll = 0, kBlocksUpper = 1, kBlocksTopHalf = 2, kBlocksBottomHalf = 3 };

template <int MODE, int NB>
__host__ __device__ constexpr bool block_used(int i, int j) {
  return MODE == kBlocksAll ? true
         : MODE == kBlocksUpper ? i <= j
         : MODE == kBlocksTopHalf ? i < NB / 2
                                  : i >= NB / 2;
}

// The wave's square (row and column offsets inside the 128 x 128 tile) and
// block set.
struct WaveRole {
  int wm, wn, mode;
};
__device__ __forceinline__ WaveRole wave_role(int wave, bool diag) {
  if (!diag) return {(wave >> 1) * kWaveTile, (wave & 1) * kWaveTile, kBlocksAll};
  if (wave == 0) return {0, 0, kBlocksUpper};
  if (wave == 3) return {kWaveTile, kWaveTile, kBlocksUpper};
  return {0, kWaveTile, wave == 1 ? kBlocksTopHalf : kBlocksBottomHalf};
}

// Accumulators of one wave: an NB x NB grid of MFMA blocks covering 64 x 64.
template <typename T>
struct WaveAcc {
  static constexpr int NB = kWaveTile / Mfma<T>::kM;
  typename Mfma<T>::acc_t c[NB][NB];

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < Mfma<T>::kAcc; ++v) c[i][j][v] = (T)0;
  }

  // The MFMA k-steps of one LDS stage (kBK / kK steps) over the wave's
  // NB x NB blocks.  MODE (kBlocks*): the blocks of the wave's square that
  // are computed.
  template <int LA, int LB, int LDPA, int LDPB, int MODE>
  __device__ __forceinline__ void stage(const T* __restrict__ a, const T* __restrict__ b, int wm0,
                                        int wn0, int lane) {
    constexpr int KS = Mfma<T>::kBK / Mfma<T>::kK;  // k-steps per stage
    constexpr int VP = 16 / (int)sizeof(T);         // elements per 16-byte LDS read
    constexpr int S0 = 0, S1 = KS;
    static_assert(KS % VP == 0, "row fragments are read 16 bytes at a time");
    typedef T vec_t __attribute__((ext_vector_type(VP)));
    const int g = lane / Mfma<T>::kM;  // this lane's k group: k = g * KS + s at k-step s
    const int ml = lane % Mfma<T>::kM;
    // kLayoutK fragments: one element per k-step, double-buffered in
    // registers so the reads of step s+1 are issued before the MFMAs of s.
    T fa[2][NB], fb[2][NB];
    const T* pa = a + g * KS * LDPA + wm0 + ml;
    const T* pb = b + g * KS * LDPB + wn0 + ml;
    if (LA == kLayoutK) {
#pragma unroll
      for (int i = 0; i < NB; ++i) fa[S0 & 1][i] = pa[S0 * LDPA + i * Mfma<T>::kM];
    }
    if (LB == kLayoutK) {
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[S0 & 1][j] = pb[S0 * LDPB + j * Mfma<T>::kM];
    }
    // kLayoutRow fragments: VP k-steps per 16-byte read, read per chunk of
    // VP steps (the registers of one chunk only)
#pragma unroll
    for (int cch = S0 / VP; cch < S1 / VP; ++cch) {
      vec_t ra[LA == kLayoutRow ? NB : 1], rb[LB == kLayoutRow ? NB : 1];
      if (LA == kLayoutRow) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
          ra[i] = *reinterpret_cast<const vec_t*>(a + (wm0 + i * Mfma<T>::kM + ml) * LDPA + g * KS + cch * VP);
      }
      if (LB == kLayoutRow) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
          rb[j] = *reinterpret_cast<const vec_t*>(b + (wn0 + j * Mfma<T>::kM + ml) * LDPB + g * KS + cch * VP);
      }
#pragma unroll
      for (int e = 0; e < VP; ++e) {
        const int s = cch * VP + e;
        const int cur = s & 1;
        if (s + 1 < S1) {
          if (LA == kLayoutK) {
#pragma unroll
            for (int i = 0; i < NB; ++i) fa[cur ^ 1][i] = pa[(s + 1) * LDPA + i * Mfma<T>::kM];
          }
          if (LB == kLayoutK) {
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[cur ^ 1][j] = pb[(s + 1) * LDPB + j * Mfma<T>::kM];
          }
        }
        if (LA == kLayoutK || LB == kLayoutK) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if (!block_used<MODE, NB>(i, j)) continue;
            c[i][j] = Mfma<T>::mma(LA == kLayoutRow ? ra[i][e] : fa[cur][i], LB == kLayoutRow ? rb[j][e] : fb[cur][j],
                                   c[i][j]);
          }
        if (LA == kLayoutK || LB == kLayoutK) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
};

// k-loop over LDS stages of one wave with square (wm0, wn0) and block set
// MODE (each block set is a separate loop, so the wave-uniform choice costs
// no registers inside the loop).  Stages alternate between two buffer pairs;
// at the start of stage st the registers loaded during stage st-1 are written
// as stage st+1, into the pair that stage st-1 read (every wave left it at
// the barrier ending that stage), and the loads of stage st+2 are issued.
template <int MODE, typename T, int LA, int LB>
__device__ __forceinline__ void tile_loop(WaveAcc<T>& acc, const Operand<T>& A, const Operand<T>& B, int m0, int n0,
                                          int K, T* a0, T* a1, T* b0, T* b1, int wm0, int wn0) {
  constexpr int BK = Mfma<T>::kBK;
  typedef Loader<T, LA> LdA;
  typedef Loader<T, LB> LdB;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  LdA la;
  LdB lb;
  const int nst = (K + BK - 1) / BK;
  auto load = [&](int k0) {
    if (LA == kLayoutK) la.load(A, k0, m0, tid); else la.load(A, m0, k0, tid);
    if (LB == kLayoutK) lb.load(B, k0, n0, tid); else lb.load(B, n0, k0, tid);
  };
  load(0);
  la.store(a0, tid);
  lb.store(b0, tid);
  if (nst > 1) load(BK);
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    const bool odd = st & 1;
    if (st + 1 < nst) {
      la.store(odd ? a0 : a1, tid);
      lb.store(odd ? b0 : b1, tid);
    }
    if (st + 2 < nst) load((st + 2) * BK);
    acc.template stage<LA, LB, LdA::LDP, LdB::LDP, MODE>(odd ? a1 : a0, odd ? b1 : b0, wm0, wn0, lane);
    __syncthreads();
  }
}

// Full k-loop of one 128 x 128 output tile.
//   A: layout LA; kLayoutK reads storage rows k (cols m0..), kLayoutRow
//      reads storage rows m0.. (cols k).
//   B: layout LB; kLayoutK reads storage rows k (cols n0..), kLayoutRow
//      reads storage rows n0.. (cols k).
// diag: diagonal tile of a symmetric output; the waves take the squares and
// block sets of wave_role (the epilogue must use the same roles).
template <typename T, int LA, int LB>
__device__ __forceinline__ void tile_mma(WaveAcc<T>& acc, const Operand<T>& A, const Operand<T>& B, int m0, int n0,
                                         int K, T* a0, T* a1, T* b0, T* b1, bool diag = false) {
  const WaveRole ro = wave_role(threadIdx.x >> 6, diag);
  if (ro.mode == kBlocksAll)
    tile_loop<kBlocksAll, T, LA, LB>(acc, A, B, m0, n0, K, a0, a1, b0, b1, ro.wm, ro.wn);
  else if (ro.mode == kBlocksUpper)
    tile_loop<kBlocksUpper, T, LA, LB>(acc, A, B, m0, n0, K, a0, a1, b0, b1, ro.wm, ro.wn);
  else if (ro.mode == kBlocksTopHalf)
    tile_loop<kBlocksTopHalf, T, LA, LB>(acc, A, B, m0, n0, K, a0, a1, b0, b1, ro.wm, ro.wn);
  else
    tile_loop<kBlocksBottomHalf, T, LA, LB>(acc, A, B, m0, n0, K, a0, a1, b0, b1, ro.wm, ro.wn);
}

// Workgroup id -> logical tile index so that consecutive logical tiles land
// on the same XCD (workgroups are dealt round-robin over the 8 XCDs, each
// with its own L2): XCD x receives the contiguous logical range
// [x*q + min(x, r), ...) where nwg = 8q + r.
__host__ __device__ __forceinline__ int xcd_remap(int b, int nwg) {
  const int q = nwg >> 3, r = nwg & 7;
  const int x = b & 7, s = b >> 3;
  return x * q + (x < r ? x : r) + s;
}

// Workgroup id -> logical index over two consecutive parts, [0, n1) and
// [n1, n1 + n2): XCD x runs its contiguous share of the first part (as
// xcd_remap), then its contiguous share of the second; -1 past both.  A
// launch needs 8 (ceil((n1 + n2) / 8) + 1) workgroups, since the two
// shares of one XCD round up separately.
__host__ __device__ __forceinline__ int xcd_split_remap(int b, int n1, int n2) {
  const int x = b & 7;
  int s = b >> 3;
  const int q1 = n1 >> 3, r1 = n1 & 7;
  const int c1 = q1 + (x < r1 ? 1 : 0);
  if (s < c1) return x * q1 + (x < r1 ? x : r1) + s;
  s -= c1;
  const int q2 = n2 >> 3, r2 = n2 & 7;
  if (s >= q2 + (x < r2 ? 1 : 0)) return -1;
  return n1 + x * q2 + (x < r2 ? x : r2) + s;
}

// Workgroup id -> logical index for launches whose tiles differ in cost
// (grouped problems of mixed sizes): chunks of kDealChunk consecutive
// indices are dealt round-robin over the 8 XCDs, so every XCD gets an even
// share of the work while its L2 still sees runs of neighbouring tiles.  A
// bijection on [0, 8 kDealChunk m) for every m: such launches pad their grid
// to a multiple of 8 kDealChunk, and ids mapped past the work return.
constexpr int kDealChunk = 8;
// Workgroup -> tile maps of the grouped GEMM: xcd_remap, deal_chunks, or
// (symmetric problems of one size) xcd_split_remap with the diagonal tiles
// last.
enum { kMapXcd = 0, kMapDeal = 1, kMapDiagLast = 2 };
__host__ __device__ __forceinline__ int deal_chunks(int b) {
  const int x = b & 7, s = b >> 3;
  return ((s / kDealChunk) * 8 + x) * kDealChunk + (s % kDealChunk);
}

// Index t of the upper-triangular tile list of a T x T tile grid (row-major
// over ti, tj >= ti) -> (ti, tj).
__host__ __device__ __forceinline__ void unrank_upper(int t, int T, int& ti, int& tj) {
  int i = 0;
  while (t >= T - i) {
    t -= T - i;
    ++i;
  }
  ti = i;
  tj = i + t;
}

// Index t of the strictly upper tile list of a T x T tile grid (row-major
// over ti, tj > ti) -> (ti, tj).
__host__ __device__ __forceinline__ void unrank_strict_upper(int t, int T, int& ti, int& tj) {
  int i = 0;
  while (t >= T - 1 - i) {
    t -= T - 1 - i;
    ++i;
  }
  ti = i;
  tj = i + 1 + t;
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    T w = __shfl_xor(v, o, 64);
    v = v > w ? v : w;
  }
  return v;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace shp
