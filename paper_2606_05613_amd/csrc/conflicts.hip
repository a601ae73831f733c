// Per-bucket gradient-conflict diagnostics from the Gram matrices.
//
// Two task gradients conflict when their inner product (equivalently their
// cosine similarity) is negative (Section 2.1 and the appendix definition of
// conflicting gradients).  Figure 1 follows the mean and spread of the
// pairwise cosines and counts a conflict at a step when some pair is
// negative; per bucket these are the statistics below.  They read only the
// K x K Gram matrices the Gram pass already produced: B*K*K*8 bytes, no
// gradient traffic.  W lanes per bucket, W the power of two that holds its
// pairs (at most a wavefront: K <= 16 has 120), lane l of them the pairs l, l +
// W in fp64; sums go through a fixed butterfly, whose bits do not depend on W.
//
// A call waits for the roots and divisions of one bucket, so its pairs go side
// by side: by one thread K = 16 takes 103 us, by a wavefront 4.  It must not
// take more lanes than it has pairs either: launching a wavefront costs 0.5 ns
// of the chip, K=2, 400,000 buckets (one pair each) 6 us with W = 1, 204 with 64.
#include "internal.h"

namespace bkmoo {

namespace {

constexpr int kConflictThreads = kWave;

// Cosine of tasks i != j: G_ij / sqrt(G_ii G_jj) clipped to [-1, 1]; 0 when
// either gradient is zero.
__device__ __forceinline__ double pair_cos(const double *G, int K, int i, int j) {
  const double gii = G[i * K + i], gjj = G[j * K + j];
  if (!(gii > 0.0) || !(gjj > 0.0)) return 0.0;
  const double c = G[i * K + j] / sqrt(gii * gjj);
  return c < -1.0 ? -1.0 : (c > 1.0 ? 1.0 : c);
}

// Sum over a bucket's W lanes (every one of them).
template <int W>
__device__ __forceinline__ double lanes_sum(double x) {
#pragma unroll
  for (int off = W / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, W);
  return x;
}

template <int K, int W>
__global__ __launch_bounds__(kConflictThreads) void conflicts_kernel(
    int B, const double *__restrict__ gram, double *__restrict__ cosines, double *__restrict__ summary,
    int32_t *__restrict__ pairs) {
  constexpr int npairs = K * (K - 1) / 2, kPairsPerLane = (npairs + W - 1) / W;
  const int64_t b = ((int64_t)blockIdx.x * kConflictThreads + threadIdx.x) / W;
  if (b >= B) return;
  const int t = threadIdx.x % W;
  const double *G = gram + b * K * K;
  double *cb = cosines ? cosines + b * K * K : nullptr;

  int bad = 0;
  for (int q = t; q < K * K; q += W) bad |= !__builtin_isfinite(G[q]);
#pragma unroll
  for (int off = W / 2; off >= 1; off >>= 1) bad |= __shfl_xor(bad, off, W);
  if (bad) {
    const double nan = __builtin_nan("");
    if (cb)
      for (int q = t; q < K * K; q += W) cb[q] = nan;
    for (int q = t; q < 3; q += W) {
      if (summary) summary[3 * b + q] = nan;
      if (pairs) pairs[3 * b + q] = -1;
    }
    return;
  }

  if (cb)
    for (int i = t; i < K; i += W) cb[i * K + i] = G[i * K + i] > 0.0 ? 1.0 : 0.0;
  // this lane's pairs, in lexicographic order of (i, j): their cosines, the
  // least of them (`at`: its rank; a NaN, from a product of squared norms
  // out of range, is never less) and how many inner products are negative
  double c[kPairsPerLane], sum = 0.0, best = __builtin_inf();
  int at = kMaxK * kMaxK, count = 0;
#pragma unroll
  for (int u = 0; u < kPairsPerLane; ++u) {
    const int p = t + u * W;
    c[u] = 0.0;
    if (p < npairs) {
      int i = 0, rem = p;
      while (rem >= K - 1 - i) {
        rem -= K - 1 - i;
        ++i;
      }
      const int j = i + 1 + rem;
      c[u] = pair_cos(G, K, i, j);
      if (cb) cb[i * K + j] = cb[j * K + i] = c[u];
      sum += c[u];
      if (G[i * K + j] < 0.0) ++count;
      if (c[u] < best || (c[u] == best && p < at)) {
        best = c[u];
        at = p;
      }
    }
  }
  sum = lanes_sum<W>(sum);
#pragma unroll
  for (int off = W / 2; off >= 1; off >>= 1) {
    const double ob = __shfl_xor(best, off, W);
    const int oa = __shfl_xor(at, off, W);
    count += __shfl_xor(count, off, W);
    if (ob < best || (ob == best && oa < at)) {
      best = ob;
      at = oa;
    }
  }
  // the first pair stands unless another is less, also when it is a NaN
  const double first = __shfl(c[0], 0, W);
  if (at >= npairs || first != first) {
    best = first;
    at = 0;
  }
  const double mean = sum / npairs;
  double ss = 0.0;
#pragma unroll
  for (int u = 0; u < kPairsPerLane; ++u) {
    const double d = c[u] - mean;
    if (t + u * W < npairs) ss += d * d;
  }
  ss = lanes_sum<W>(ss);
  if (t == 0) {
    if (summary) {
      summary[3 * b] = mean;
      summary[3 * b + 1] = sqrt(ss / npairs);
      summary[3 * b + 2] = best;
    }
    if (pairs) {
      int i = 0, rem = at;
      while (rem >= K - 1 - i) {
        rem -= K - 1 - i;
        ++i;
      }
      pairs[3 * b] = i;
      pairs[3 * b + 1] = i + 1 + rem;
      pairs[3 * b + 2] = count;
    }
  }
}

template <int K>
void launch_conflicts_t(int B, const double *gram, double *cosines, double *summary, int32_t *pairs, hipStream_t s) {
  constexpr int npairs = K * (K - 1) / 2;
  constexpr int W = npairs <= 1 ? 1 : npairs <= 4 ? 4 : npairs <= 8 ? 8 : npairs <= 16 ? 16 : npairs <= 32 ? 32 : 64;
  const unsigned grid = (unsigned)(((int64_t)B * W + kConflictThreads - 1) / kConflictThreads);
  hipLaunchKernelGGL((conflicts_kernel<K, W>), dim3(grid), dim3(kConflictThreads), 0, s, B, gram, cosines, summary,
                     pairs);
}

}  // namespace

hipError_t launch_conflicts(int K, int B, const double *gram, double *cosines, double *summary,
                            int32_t *pairs, hipStream_t s) {
#define BKMOO_CONFLICTS_CASE(k) \
  case k: launch_conflicts_t<k>(B, gram, cosines, summary, pairs, s); break;
  switch (K) {
    BKMOO_CONFLICTS_CASE(2) BKMOO_CONFLICTS_CASE(3) BKMOO_CONFLICTS_CASE(4) BKMOO_CONFLICTS_CASE(5)
    BKMOO_CONFLICTS_CASE(6) BKMOO_CONFLICTS_CASE(7) BKMOO_CONFLICTS_CASE(8) BKMOO_CONFLICTS_CASE(9)
    BKMOO_CONFLICTS_CASE(10) BKMOO_CONFLICTS_CASE(11) BKMOO_CONFLICTS_CASE(12) BKMOO_CONFLICTS_CASE(13)
    BKMOO_CONFLICTS_CASE(14) BKMOO_CONFLICTS_CASE(15) BKMOO_CONFLICTS_CASE(16)
    default: return hipErrorInvalidValue;
  }
#undef BKMOO_CONFLICTS_CASE
  return hipGetLastError();
}

}  // namespace bkmoo
