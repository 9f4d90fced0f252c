// Device kernels for embedding layers (appendix "Shampoo for embedding
// layers"): the sparse gradient of a lookup in compact form, and the reduce
// of split-K partial statistics.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace shp {

// Sort keys of the lookup entries: the table row, or `vocab` (sorts last)
// for an entry whose row or output feature is out of range; values are the
// entry indices, so a stable sort keeps the entries of one row in order.
__global__ __launch_bounds__(kThreads) void emb_keys_kernel(const int32_t* __restrict__ idx,
                                                           const int32_t* __restrict__ feat, int nnz,
                                                           int32_t vocab, int m, int32_t* __restrict__ keys,
                                                           int32_t* __restrict__ vals, int32_t* __restrict__ lens) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e >= nnz) return;
  const int32_t r = idx[e];
  const int32_t f = feat ? feat[e] : e;
  keys[e] = (r >= 0 && r < vocab && f >= 0 && f < m) ? r : vocab;
  vals[e] = e;
  lens[e] = 0;  // run lengths past the last run stay 0 for the offset scan
}

// Segment sums of the sorted entries in fixed chunks of kEmbChunk entries,
// one workgroup per chunk.  A run (the entries of one table row) that lies
// inside the chunk is summed into its row of U directly; the run holding
// the chunk's first entry, if it reaches outside the chunk, goes to partial
// slot 0 of the chunk, and the chunk's last run, if different and reaching
// past the end, to slot 1.  Entries are added in sorted (= entry) order.
constexpr int kEmbChunk = 64;

template <bool VEC>
__device__ __forceinline__ void emb_chunk_cols(int c, const int32_t* __restrict__ uniq, const int32_t* __restrict__ lens,
                                               const int32_t* __restrict__ offs, int R, const int32_t* __restrict__ vals,
                                               const int32_t* __restrict__ feat, const float* __restrict__ weight,
                                               const float* __restrict__ dy, int64_t ld_dy, int dim, int32_t vocab,
                                               int nnz, float* __restrict__ U, float* __restrict__ part) {
  const int t0 = c * kEmbChunk, t1 = min(t0 + kEmbChunk, nnz);
  // run holding t0: the last run starting at or before t0
  int lo = 0, hi = R - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (offs[mid] <= t0) lo = mid; else hi = mid - 1;
  }
  constexpr int W = VEC ? 4 : 1;
  for (int col = W * threadIdx.x; col < dim; col += W * kThreads) {
    int i = lo;
    int rs = offs[i], re = rs + lens[i];
    bool skip = uniq[i] == vocab;
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    auto flush = [&]() {
      if (skip) return;
      float* dst;
      if (rs >= t0 && re <= t1) dst = U + (int64_t)i * dim;              // whole run in this chunk
      else if (i == lo) dst = part + ((int64_t)c * 2 + 0) * dim;         // run of the first entry
      else dst = part + ((int64_t)c * 2 + 1) * dim;                      // last run, continues
      if (VEC) gstore<f4v>(dst + col, acc);
      else gstore<float>(dst + col, acc[0]);
    };
    for (int t = t0; t < t1; ++t) {
      if (t >= re) {
        flush();
        ++i;
        rs = offs[i];
        re = rs + lens[i];
        skip = uniq[i] == vocab;
        acc = f4v{0.f, 0.f, 0.f, 0.f};
      }
      if (skip) continue;
      const int e = vals[t];
      const int f = feat ? feat[e] : e;
      const float w = weight ? weight[e] : 1.f;
      const float* src = dy + (int64_t)f * ld_dy + col;
      if (VEC) acc += w * gload<f4v>(src);
      else acc[0] += w * gload<float>(src);
    }
    flush();
  }
}

__global__ __launch_bounds__(kThreads) void emb_chunk_kernel(
    const int32_t* __restrict__ uniq, const int32_t* __restrict__ lens, const int32_t* __restrict__ offs,
    const int32_t* __restrict__ nruns, const int32_t* __restrict__ vals, const int32_t* __restrict__ feat,
    const float* __restrict__ weight, const float* __restrict__ dy, int64_t ld_dy, int dim, int32_t vocab, int nnz,
    float* __restrict__ U, float* __restrict__ part) {
  const int c = blockIdx.x;
  if (c * kEmbChunk >= nnz) return;
  const int R = *nruns;
  if (R < 1) return;
  const bool vec = (dim & 3) == 0 && (ld_dy & 3) == 0 && (reinterpret_cast<uintptr_t>(dy) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(U) & 15) == 0;
  if (vec) emb_chunk_cols<true>(c, uniq, lens, offs, R, vals, feat, weight, dy, ld_dy, dim, vocab, nnz, U, part);
  else emb_chunk_cols<false>(c, uniq, lens, offs, R, vals, feat, weight, dy, ld_dy, dim, vocab, nnz, U, part);
}

// The row ids (-1 past the active rows), the counts (count[0] = active rows,
// count[1] = dropped entries), and for every run that spans several chunks
// the sum of its chunk partials in chunk order.  Workgroup b writes the ids
// of kThreads runs and sums the run that starts in chunk b and reaches past
// its end, if there is one (at most one per chunk, so about nnz / 64
// workgroups; one workgroup per potential run took 117 us for 65536 lookups,
// most of them to find nothing to do, and a Zipf head row's 110 partials were
// added one load at a time).  Rows of U at or past the active count are not
// written.
template <bool VEC>
__device__ __forceinline__ void emb_fix_cols(const float* __restrict__ part, int c0, int c1, bool first_slot1, int dim,
                                             float* __restrict__ dst) {
  constexpr int W = VEC ? 4 : 1;
  for (int col = W * threadIdx.x; col < dim; col += W * kThreads) {
    f4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int c = c0; c <= c1; ++c) {
      const float* src = part + ((int64_t)c * 2 + (c == c0 && first_slot1 ? 1 : 0)) * dim + col;
      if (VEC) acc += gload<f4v>(src);
      else acc[0] += gload<float>(src);
    }
    if (VEC) gstore<f4v>(dst + col, acc);
    else gstore<float>(dst + col, acc[0]);
  }
}

__global__ __launch_bounds__(kThreads) void emb_fix_kernel(const int32_t* __restrict__ uniq,
                                                          const int32_t* __restrict__ lens,
                                                          const int32_t* __restrict__ offs,
                                                          const int32_t* __restrict__ nruns, int dim, int32_t vocab,
                                                          int nnz, const float* __restrict__ part,
                                                          int32_t* __restrict__ rows, float* __restrict__ U,
                                                          int32_t* __restrict__ count) {
  const int R = *nruns;
  const bool tail_dropped = R > 0 && uniq[R - 1] == vocab;
  const int i0 = blockIdx.x * kThreads + threadIdx.x;
  if (i0 == 0) {
    count[0] = R - (tail_dropped ? 1 : 0);
    count[1] = tail_dropped ? lens[R - 1] : 0;
  }
  if (i0 < nnz) rows[i0] = i0 < R && uniq[i0] != vocab ? uniq[i0] : -1;
  const int c0 = blockIdx.x, t0 = c0 * kEmbChunk, t1 = t0 + kEmbChunk;
  if (R < 1 || t1 >= nnz) return;  // nothing reaches past the last chunk
  // the run holding entry t1 - 1
  int lo = 0, hi = R - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (offs[mid] <= t1 - 1) lo = mid; else hi = mid - 1;
  }
  const int rs = offs[lo], re = rs + lens[lo];
  if (rs < t0 || re <= t1 || uniq[lo] == vocab) return;
  float* dst = U + (int64_t)lo * dim;
  const bool vec = (dim & 3) == 0 && (reinterpret_cast<uintptr_t>(U) & 15) == 0;
  if (vec) emb_fix_cols<true>(part, c0, (re - 1) / kEmbChunk, rs != t0, dim, dst);
  else emb_fix_cols<false>(part, c0, (re - 1) / kEmbChunk, rs != t0, dim, dst);
}

// R = beta R + alpha * sum_s part[s] over all n elements, the partials added
// in split order (deterministic).  beta == 1 keeps R's old value exactly
// scaled by one.
__global__ __launch_bounds__(kThreads) void emb_reduce_kernel(const float* __restrict__ part, int splits,
                                                             int64_t stride, int64_t n, float alpha, float beta,
                                                             float* __restrict__ R) {
  const int64_t q = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
  if (q >= n) return;
  if (q + 4 <= n && (n & 3) == 0) {
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < splits; ++s) acc += gload<f4v>(part + s * stride + q);
    f4v r = gload<f4v>(R + q);
    gstore<f4v>(R + q, beta * r + alpha * acc);
  } else {
    for (int64_t k = q; k < q + 4 && k < n; ++k) {
      float acc = 0.f;
      for (int s = 0; s < splits; ++s) acc += gload<float>(part + s * stride + k);
      gstore<float>(R + k, beta * gload<float>(R + k) + alpha * acc);
    }
  }
}

}  // namespace shp
