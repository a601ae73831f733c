// The Gram finalize's sum of one bucket's partial slots, shared by the
// kernel that only writes the matrix and the one that solves it as well.
#pragma once

#include "internal.h"

namespace bkmoo {

namespace {

// The workgroup that adds up a bucket's slots: a thread each (kSumThreads), or one wavefront for all of them (the
// same sums in the same order) where a call has many buckets of few slots, of
// which most threads would only start and end: from four buckets a CU on and up
// to four chunks a bucket on average.  The Gram call, us, threads / wavefront:
// K=2 fp32, 20,000 buckets of 0.02 chunks 170 / 133, 2,048 of 0.9 60 / 59, 1,024
// of 3.9 95 / 95; K=10 fp32 8,192 of 0.02 197 / 182; but 256 buckets of 3.9
// 118 / 120, 16 of 7.9 32 / 36.
inline int sum_workgroup(const StreamArgs &a) {
  const bool small = a.B >= 4 * device_cu_count() && a.N / gram_chunk_elems(a.K, a.dt) <= 4 * (int64_t)a.B;
  return small && pairs(a.K) <= kWave ? kWave : kSumThreads;
}

// Partial loads a thread keeps in flight.  The sums wait for memory, not for
// bandwidth: with the loads one behind the other a group of 1024 slots of
// the K = 8 Gram took 40 us, the same slots in groups of 64 and batches of 16
// take 4 us.
constexpr int kSumBatch = 16;

// Sum over i = 0..n-1 of the P entries of slot c0 + i * step, for a whole
// workgroup of T threads, a thread per pair at least: entry q < rows * P (rows
// = kSumThreads / P) is pair q % P of the slots q / P, q / P + rows, ...
// ascending, then the rows are added ascending.  The order depends on n and P
// alone.  Thread p < P returns pair p's sum; `red` holds kSumThreads doubles of
// LDS (it may be reused after the next barrier).
template <int T>
__device__ __forceinline__ double sum_slots(const double *__restrict__ slots, int64_t c0, int64_t n, int64_t step,
                                            int P, double *red) {
  const int t = threadIdx.x, rows = kSumThreads / P;
  double s = 0.0;
  for (int q = t; q < rows * P; q += T) {
    const int r = q / P;
    const double *base = slots + c0 * P + (q - r * P);
    s = 0.0;
    for (int64_t i = r; i < n; i += (int64_t)rows * kSumBatch) {
      double x[kSumBatch];
#pragma unroll
      for (int u = 0; u < kSumBatch; ++u) {
        const int64_t j = i + (int64_t)u * rows;
        x[u] = j < n ? base[j * step * P] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < kSumBatch; ++u) s += x[u];
    }
    red[q] = s;
  }
  __syncthreads();
  if (t < P) {
    s = red[t];
    for (int q = 1; q < rows; ++q) s += red[q * P + t];
  }
  return s;
}

// Pair p's sum over bucket b, of its chunk slots or, in a bucket of sum_direct
// chunks and more, of its group sums.
template <int T>
__device__ __forceinline__ double sum_bucket(const double *__restrict__ partials, const int64_t *__restrict__ cs,
                                             int64_t b, int P, double *red) {
  const int64_t c0 = cs[b], n = cs[b + 1] - c0, step = n < sum_direct(P) ? 1 : kFinalizeGroup;
  return sum_slots<T>(partials, c0, (n + step - 1) / step, step, P, red);
}

// Task pair (i <= j) of entry p of the row-major upper triangle.
__device__ __forceinline__ void pair_of(int p, int K, int &i, int &j) {
  i = 0;
  while (p >= K - i) {
    p -= K - i;
    ++i;
  }
  j = i + p;
}

}  // namespace

}  // namespace bkmoo
