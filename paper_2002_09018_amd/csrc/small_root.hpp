// Inverse p-th roots of matrices of at most 128 x 128 in fp32: the whole
// coupled Newton iteration of a matrix in one workgroup and one launch.
//
// What bounds it: the grouped path takes about 35 dependent launches and a
// host poll per iteration for such a matrix, each launch one 128 x 128 tile
// of work (7-10 us of launch and drain for under 3 us of products), so two
// 128 x 128 roots took 0.4 ms.  Here an iterate never leaves the compute
// unit: a matrix is NB x NB blocks of 32 x 32 (NB = ceil(n / 32)), wave
// (bi, bj) holds its block of X, M and P = M1^(2^s) in registers (16 values
// a lane each, in the MFMA accumulator layout), and a product publishes its
// operands as three bf16 planes in LDS in fragment order (split_mfma.hpp).
// The planes of two 128 x 128 operands (192 KB) exceed LDS, so a product of
// two matrices goes in two k-halves; a square publishes its one operand
// whole.  Waves of blocks on and above the diagonal multiply (10 of 16 at
// NB = 4, at most three to a SIMD); the others take the mirrored values
// through LDS, so iterates stay exactly symmetric.
//
// Once the residual is below 1/2 (where the subtraction is exact), M is held as
// E = M - I and the powers of M1 as Q = M1^(2^s) - I: products of matrices near
// I lose the small terms that the bf16 instruction sums together with a
// diagonal product (split_mfma.hpp); those of E and Q are small themselves.
// (Far from I the matrices themselves keep small eigenvalues to more bits: with
// E from the start and the Frobenius scaling p = 1 roots lost 40%, and with Q a
// 1 x 1 root of order 16 lost 4e-5.)  Roots of 24
// Wishart matrices of 32 x 32, error in 2^-24, before / now / fp32 instruction
// in the grouped path: p = 1 9.6 / 5.3 / 6.7, p = 2 3.7 / 1.4 / 2.9, p = 8 5.2 /
// 1.4 / 2.6; the number of products is the same.
#pragma once

#include "kernels.hpp"

namespace shp {

// Largest n, at any number of matrices.  Measured against grouped launches, us:
// 128 x 128 1: 466 -> 210, 400: 808 -> 420, 4000: 7680 -> 4400; 96 x 96 4000:
// 6630 -> 3070; 64 x 64 1: 445 -> 145, 10000: 10200 -> 2610; 8 x 8 1: 381 -> 149,
// 10000: 3780 -> 955.
constexpr int kSmallMax = 128;
// E shrinks below anything an M in 32 bits could show: a residual of at most
// this that was still above tol ends the iteration as the rounding floor.
constexpr float kSmallFloor = 0x1p-20f;
constexpr int kSmallExchange = 32 * 33;  // floats of one exchanged block (padded rows)

// A launch for matrices of at most NB x NB blocks: one wave per block, the
// planes of an operand pair, one exchange block per upper block, reductions.
// Launches of small matrices so share a compute unit: with the shape of NB = 4
// for all, a compute unit took one matrix at a time and 10000 roots of 8 x 8
// 3980 us, of 64 x 64 6000 (grouped launches 3780 and 10200); now 955 and 2610.
// Three waves per SIMD hold the iterates without spilling up to NB = 2 (two:
// 1055 and 3280, four: 965 and 2520 with 72 registers spilled, and a single
// root 4% slower).
constexpr int kSmallWaves = 3;
template <int NB>
struct SmallShape {
  static constexpr int threads = 64 * NB * NB;
  static constexpr int planes = 2 * NB * 3 * NB * kBlockB;
  static constexpr int shm = planes + NB * (NB + 1) / 2 * kSmallExchange * 4 + 16 * 8;
};

struct SmallRootArgs {
  int p, power, max_iters, eps_relative, esc_n;
  float tol;
  double eps;
  const float* esc_thr;
};

// Products of the iteration (SmallRoot::run), in the order they follow.
enum : int {
  kOpSquare0,  // power bound: P = M0 M0
  kOpSquare1,  //              X = P P
  kOpFirst4,   // first M update at p = 4 under the power bound, one product
  kOpX,        // X = X M1 = b X M + a X, or b X E + X
  kOpMM,       // P = M M, then P = M1 M1 and, for odd p, M = M1 M (or E E, Q and E)
  kOpY,        // M = P M, or E = (I + Q)(I + E) - I (bit s of p)
  kOpP         // P = P P, or Q = (I + Q)(I + Q) - I
};

// A small matrix's root is a chain of products with little work in each, run
// once: with every product inlined (75 KB of code) the kernel waited for
// instruction fetches (379 us for two 128 x 128 roots), so the products share
// one instance of the code, driven by the operation.
struct SmallRoot {
  typedef Mfma<float> F;
  typedef F::acc_t acc_t;
  typedef float blk[16];  // one block, accumulator layout

  char* smem;
  float* ex;
  double* red;
  int lane, wave, n;
  int nb, waves, upper;  // blocks per side, waves, upper blocks
  int bi, bj;            // this wave's block
  // Bits v of a lane's 16 values: inside the matrix, on its diagonal.  The
  // empty asm statements keep masks and addresses from being hoisted out of
  // the iteration, where they would not fit beside the iterates in the 128
  // registers of a 16-wave workgroup.
  int in_mask, dg_mask;

  static __device__ __forceinline__ int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
  }

  // The upper blocks first, row by row, then the strictly lower ones in the
  // order of their mirror blocks.
  __device__ __forceinline__ void place() {
    if (wave < upper) unrank_upper(wave, nb, bi, bj);
    else unrank_strict_upper(wave - upper, nb, bj, bi);
    in_mask = dg_mask = 0;
    const int c = bj * 32 + F::col(lane);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = bi * 32 + F::row(lane, v);
      if (r < n && c < n) in_mask |= 1 << v;
      if (r == c && r < n) dg_mask |= 1 << v;
    }
  }

  // Writes block x into an operand region holding the 16-deep steps
  // [k0, k0 + ks): element (r, c) is element (row c, k = r) of the symmetric
  // operand.
  __device__ __forceinline__ void publish(const blk& x, char* dst, int k0, int ks, int ln) const {
    const int pb = nb * kBlockB;
    dst += bj * kBlockB + (ln & 31) * 16 + (ln >> 5) * 8;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int s = 2 * bi + (g >> 1) - k0;
      if (s < 0 || s >= ks) continue;
      char* d = dst + s * 3 * pb + (g & 1) * kHalfB;
      u32x2 a, b, c;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        uint32_t t0, t1, t2;
        split_pair<false>(x[4 * g + 2 * e], x[4 * g + 2 * e + 1], t0, t1, t2);
        a[e] = t0;
        b[e] = t1;
        c[e] = t2;
      }
      *reinterpret_cast<u32x2*>(d) = a;
      *reinterpret_cast<u32x2*>(d + pb) = b;
      *reinterpret_cast<u32x2*>(d + 2 * pb) = c;
    }
  }

  __device__ __forceinline__ double sum(double x) {
    x = wave_sum(x);
    __syncthreads();
    if (lane == 0) red[wave] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll 1
    for (int w = 0; w < waves; ++w) s += red[w];
    return s;
  }
  __device__ __forceinline__ double max_(double x) {
    x = wave_max(x);
    __syncthreads();
    if (lane == 0) red[wave] = x;
    __syncthreads();
    double s = red[0];
#pragma unroll 1
    for (int w = 1; w < waves; ++w) s = s > red[w] ? s : red[w];
    return s;
  }
  // max |scale x - eye I| over the matrix (infinity for a non-finite entry)
  __device__ __forceinline__ float resid(const blk& x, float scale, float eye) {
    float m = 0.f;
    const int dg = fresh(dg_mask), in = fresh(in_mask);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float d = fabsf(scale * x[v] - ((dg >> v) & 1 ? eye : 0.f));
      d = d <= 3.0e38f ? d : INFINITY;
      m = fmaxf(m, (in >> v) & 1 ? d : 0.f);
    }
    return (float)max_((double)m);
  }
  // x^(1 / 2^k)
  static __device__ __forceinline__ double root2(double x, int k) {
#pragma unroll 1
    for (int i = 0; i < k; ++i) x = sqrt(x);
    return x;
  }

  __device__ __forceinline__ void run(const NewtonJob<float>& J, RootState& st, const SmallRootArgs& q) {
    const int p = q.p;
    blk X, M, P;
    // A_s = (A + A^T) / 2: its Frobenius norm, trace and smallest diagonal
    // entry (X and P hold A and A^T until M0 is formed)
    double ss = 0.0, tr = 0.0, dneg = -INFINITY;
    {
      const int in = fresh(in_mask), dg = fresh(dg_mask);
      const int r0 = bi * 32 + F::row(lane, 0), c0 = bj * 32 + F::col(lane);
      const float* pr = J.A + (int64_t)r0 * n + c0;
      const float* pc = J.A + (int64_t)c0 * n + r0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        X[v] = P[v] = 0.f;
        if ((in >> v) & 1) {
          X[v] = gload<float>(pr + F::row(0, v) * n);
          P[v] = gload<float>(pc + F::row(0, v));
        }
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const double s = 0.5 * ((double)X[v] + (double)P[v]);
        ss += s * s;
        if ((dg >> v) & 1) {
          tr += s;
          dneg = fmax(dneg, -s);
        }
      }
    }
    ss = sum(ss);
    tr = sum(tr);
    const double dmin = -max_(dneg);
    const double e = q.eps_relative ? st.eps_eff : q.eps;
    const double fro2 = ss + 2.0 * e * tr + (double)n * e * e;
    const bool lead = threadIdx.x == 0;
    if (!(dmin + e > 0.0) || !(fro2 > 0.0) || !isfinite(fro2)) {
      if (lead) {
        st.eps_eff = e;
        st.diag_min = dmin + e;
        st.status = kNotPD;
        st.z = 0.0;
      }
      return;
    }
    double z = (1.0 + p) / (2.0 * sqrt(fro2)), zc = 1.0;
    // M0 = z (A_s + e I)
    {
      const int dg = fresh(dg_mask);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        M[v] = (float)(z * (0.5 * ((double)X[v] + (double)P[v]) + (((dg >> v) & 1) ? e : 0.0)));
    }
    const double a = (p + 1.0) / p, b = -1.0 / p;
    int top = 0;
    while ((p >> (top + 1)) != 0) ++top;
    const bool pow2 = (p & (p - 1)) == 0;
    int iters = 0, status = kActive, bit = 0;
    float r = INFINITY, xs = 0.f, lift = 1.f;
    bool near = false;  // M holds E
    int op = q.power ? kOpSquare0 : -1;
    while (true) {
      if (op >= 0) {
        // T = (left) (right), exactly symmetric, in the wave's accumulators
        acc_t c, t;
        const int ln = fresh(lane);
        const int pb = nb * kBlockB;
        const bool square = op == kOpSquare0 || op == kOpSquare1 || op == kOpMM || op == kOpP;
        const int half = square ? 2 * nb : nb;  // 16-deep steps published at once
#pragma unroll
        for (int v = 0; v < 16; ++v) c[v] = t[v] = 0.f;
        char* rb = square ? smem : smem + nb * 3 * pb;
#pragma unroll 1
        for (int k0 = 0; k0 < 2 * nb; k0 += half) {
          if (k0) __syncthreads();  // every wave has multiplied the first half
#pragma unroll 1
          for (int o = 0; o < (square ? 1 : 2); ++o) {
            // left: M (first4, squares of M), X (op X) or P; right: P (first4) or M
            const int which = o ? (op == kOpFirst4 ? 2 : 1)
                                : (op == kOpX ? 0 : (op == kOpSquare1 || op == kOpY || op == kOpP ? 2 : 1));
            blk w;
#pragma unroll
            for (int v = 0; v < 16; ++v) w[v] = which == 0 ? X[v] : (which == 1 ? M[v] : P[v]);
            publish(w, o ? rb : smem, k0, half, ln);
          }
          __syncthreads();
          if (wave < upper) {
            const char* pa = smem + bi * kBlockB + ln * 16;
            const char* qb = rb + bj * kBlockB + ln * 16;
#pragma unroll 1
            for (int s = 0; s < half; ++s, pa += 3 * pb, qb += 3 * pb) {
              bf16x8 fa[3], fb[3];
#pragma unroll
              for (int u = 0; u < 3; ++u) {
                fa[u] = *reinterpret_cast<const bf16x8*>(pa + u * pb);
                fb[u] = *reinterpret_cast<const bf16x8*>(qb + u * pb);
              }
              // the leading product apart from the others (K <= 128: one run)
              c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[0], c, 0, 0, 0);
#pragma unroll
              for (int u = 1; u < 3; ++u)
#pragma unroll
                for (int w = 0; w <= u; ++w)
                  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[w], fb[u - w], t, 0, 0, 0);
            }
          }
        }
        // the affine term in X of op X and of the first update
        const float ca = op == kOpX ? (float)b : 1.f, cb = op == kOpX && !near ? (float)a : 1.f;
        const bool affine = op == kOpX || op == kOpFirst4;
        float* mine = ex + (wave < upper ? wave : 0) * kSmallExchange;
        if (wave < upper) {
          float* d = mine + F::row(ln, 0) * 33 + F::col(ln);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            c[v] = ca * (c[v] + t[v]);
            if (affine) c[v] += cb * X[v];
            d[F::row(0, v) * 33] = c[v];
          }
        }
        // the barrier also ends every wave's reads of the operand regions
        __syncthreads();
        // a strictly lower block is the mirror of upper block (bj, bi), and
        // so is the lower triangle of a diagonal block
        const float* src = wave < upper ? mine : ex + (bj * nb - bj * (bj - 1) / 2 + bi - bj) * kSmallExchange;
        src += F::col(ln) * 33 + F::row(ln, 0);
        const int lim = wave >= upper ? -1 : (bi == bj ? F::col(ln) - F::row(ln, 0) : 64);
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (F::row(0, v) > lim) c[v] = src[F::row(0, v)];

        if (op == kOpSquare1 || op == kOpX) {
#pragma unroll
          for (int v = 0; v < 16; ++v) X[v] = c[v];
        } else if (op == kOpY) {
#pragma unroll
          for (int v = 0; v < 16; ++v) M[v] = (near ? P[v] + M[v] : 0.f) + c[v];
        } else if (op == kOpP) {
#pragma unroll
          for (int v = 0; v < 16; ++v) P[v] = (near ? 2.f * P[v] : 0.f) + c[v];
        } else if (op == kOpFirst4) {
          const float c1 = (float)zc;
          const int dg = fresh(dg_mask);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            X[v] = xs * (-0.25f * (c1 * M[v]) + ((dg >> v) & 1 ? 1.25f : 0.f));
            M[v] = c[v];
          }
        } else {
#pragma unroll
          for (int v = 0; v < 16; ++v) P[v] = c[v];
        }
      }
      // what follows
      bool updated = false;  // M holds the next iterate
      if (op == kOpSquare0) {
        op = kOpSquare1;
        continue;
      }
      if (op == kOpSquare1) {
        // power bound: c = (p + 1) / (2 ||M0^4||_F^(1/4)), X = M0^4
        double s4 = 0.0;
#pragma unroll
        for (int v = 0; v < 16; ++v) s4 += (double)X[v] * (double)X[v];
        const double rho = root2(sum(s4), 3);
        const double c = (rho > 0.0 && isfinite(rho)) ? (1.0 + p) / (2.0 * rho) : 1.0;
        zc = c > 1.0 ? c : 1.0;
        z *= zc;
        op = -1;
      }
      if (op == -1) {
        // as x_lift
        const double x0 = pow2 ? root2(z, top) : pow(z, 1.0 / p);
        lift = x0 < 0x1p-64 ? 0x1p64f : 1.f;
        xs = (float)(x0 * lift);
        r = resid(M, (float)zc, 1.f);
        if (!(r <= kDivergeAt)) status = kDiverged;
        else if (r <= q.tol) status = kConverged;
        if (status != kActive) break;
        // the first iteration has no X product: X1 = z^(1/p) (a I + b M0)
        const float c1 = (float)zc, c2 = (float)(zc * zc), c4 = (float)(zc * zc * zc * zc);
        const int dg = fresh(dg_mask);
        if (q.power && p == 4) {
          // f(M0) = (a + b M0)^4 M0 = M0' (K3 M0^2 + K5 M0^4)
          //         + K1 M0 + K2 M0^2 + K4 M0^4, M0 = c M0'
          const float K1 = (float)(a * a * a * a), K2 = (float)(4.0 * a * a * a * b),
                      K3 = (float)(6.0 * a * a * b * b * zc), K4 = (float)(4.0 * a * b * b * b),
                      K5 = (float)(b * b * b * b * zc);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float m = c1 * M[v], m2 = c2 * P[v], m4 = c4 * X[v];
            P[v] = K3 * m2 + K5 * m4;
            X[v] = K1 * m + K2 * m2 + K4 * m4;
          }
          op = kOpFirst4;
          continue;
        }
        const float fa = (float)(p + 1) / (float)p, fb = -1.f / (float)p;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float m = c1 * M[v];
          X[v] = xs * (fb * m + ((dg >> v) & 1 ? fa : 0.f));
          M[v] = m;
          P[v] = c2 * P[v];
        }
        op = kOpMM;
        if (!q.power) continue;  // with the power bound, M0^2 = c^2 P is known
      }
      if (op == kOpX) {
        op = kOpMM;
        continue;
      }
      // M1^p M right to left over the bits of p: after M M, bit s: M = P M if
      // set, then P = P P below the top bit
      if (op == kOpFirst4) {
        updated = true;
      } else {
        if (op == kOpMM) {
          // M^2 -> M1^2 = b^2 M^2 + 2ab M + a^2 I, M1 M = b M^2 + a M;
          // E^2 -> M1^2 - I = b^2 E^2 + 2b E, M1 M - I = b E^2 + (1 + b) E
          bit = 0;
          const float b2 = (float)(b * b), ab2 = (float)(near ? 2.0 * b : 2.0 * a * b),
                      a2 = near ? 0.f : (float)(a * a), b1 = (float)b, a1 = (float)(near ? 1.0 + b : a);
          const int dg = fresh(dg_mask);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float m2 = P[v], m = M[v];
            P[v] = b2 * m2 + ab2 * m + ((dg >> v) & 1 ? a2 : 0.f);
            if (p & 1) M[v] = b1 * m2 + a1 * m;
          }
        }
        if (op == kOpMM || op == kOpP) {
          ++bit;
          if (bit > top) {
            updated = true;  // p = 1
          } else if ((p >> bit) & 1) {
            op = kOpY;
            continue;
          }
        }
        if (!updated) {  // bit's M product has run, or is not wanted
          if (bit < top) {
            op = kOpP;
            continue;
          }
          updated = true;
        }
      }
      const float prev = r;
      r = resid(M, 1.f, near ? 0.f : 1.f);
      ++iters;
      if (!(r <= kDivergeAt)) status = kDiverged;
      else if (r <= q.tol) status = kConverged;
      else if (prev < kStagGate && (r >= prev || prev <= kSmallFloor)) status = kStagnated;
      else if (iters >= q.max_iters) status = kMaxIter;
      else if (q.esc_thr && iters <= q.esc_n && r > q.esc_thr[iters - 1]) status = kMaxIter;
      if (status != kActive) break;
      if (!near && r < 0.5f) {
        near = true;
        const int dg = fresh(dg_mask);
#pragma unroll
        for (int v = 0; v < 16; ++v) M[v] -= (dg >> v) & 1 ? 1.f : 0.f;
      }
      op = kOpX;
    }
    // the last iterate, or X0 = z^(1/p) I
    {
      const int in = fresh(in_mask), dg = fresh(dg_mask);
      const float down = 1.f / lift;
      float* out = J.Xout + (int64_t)(bi * 32 + F::row(lane, 0)) * n + bj * 32 + F::col(lane);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if ((in >> v) & 1) gstore<float>(out + F::row(0, v) * n, down * (iters > 0 ? X[v] : (((dg >> v) & 1) ? xs : 0.f)));
    }
    if (lead) {
      st.eps_eff = e;
      st.diag_min = dmin + e;
      st.z = z;
      st.zc = zc;
      st.status = status;
      st.iters = iters;
      st.resid = r;
      st.parity = 0;  // the result is in the caller's X
      st.lift = 1.0;
    }
  }
};

// One workgroup per job from `first` on (n <= 32 NB, largest first); jobs that
// are not active (NOT_PD, sent to fp64 by the condition witness, kept from a warm
// start) are left alone.  Waves past the matrix's blocks end at once (a
// barrier counts the waves that are left).
template <int NB>
__global__ __launch_bounds__(SmallShape<NB>::threads, kSmallWaves) void newton_small_kernel(
    const NewtonJob<float>* __restrict__ jobs, int first, RootState* __restrict__ st, SmallRootArgs q) {
  __shared__ __attribute__((aligned(16))) char smem[SmallShape<NB>::shm];
  const int j = first + blockIdx.x;
  if (st[j].status != kActive) return;
  SmallRoot s;
  s.n = jobs[j].n;
  s.nb = (s.n + 31) / 32;
  s.waves = s.nb * s.nb;
  s.upper = s.nb * (s.nb + 1) / 2;
  s.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (s.wave >= s.waves) return;
  s.lane = threadIdx.x & 63;
  s.smem = smem;
  s.ex = reinterpret_cast<float*>(smem + SmallShape<NB>::planes);
  s.red = reinterpret_cast<double*>(s.ex + NB * (NB + 1) / 2 * kSmallExchange);
  s.place();
  s.run(jobs[j], st[j], q);
}

}  // namespace shp
