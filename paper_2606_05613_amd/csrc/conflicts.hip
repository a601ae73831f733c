// Per-bucket gradient-conflict diagnostics from the Gram matrices.
//
// Two task gradients conflict when their inner product (equivalently their
// cosine similarity) is negative (Section 2.1 and the appendix definition of
// conflicting gradients).  Figure 1 follows the mean and spread of the
// pairwise cosines and counts a conflict at a step when some pair is
// negative; per bucket these are the statistics below.  They read only the
// K x K Gram matrices the Gram pass already produced: B*K*K*8 bytes, no
// gradient traffic.  One wavefront per bucket, lane l the pairs l, l + 64
// (K <= 16: at most 120) in fp64; sums go through a fixed butterfly.  One
// thread per bucket, as before, is a serial chain of 2 K(K-1)/2 roots and
// divisions: 103 us for K = 16.
#include "internal.h"

namespace bkmoo {

namespace {

// Cosine of tasks i != j: G_ij / sqrt(G_ii G_jj) clipped to [-1, 1]; 0 when
// either gradient is zero.
__device__ __forceinline__ double pair_cos(const double *G, int K, int i, int j) {
  const double gii = G[i * K + i], gjj = G[j * K + j];
  if (!(gii > 0.0) || !(gjj > 0.0)) return 0.0;
  const double c = G[i * K + j] / sqrt(gii * gjj);
  return c < -1.0 ? -1.0 : (c > 1.0 ? 1.0 : c);
}

constexpr int kPairsPerLane = (kMaxK * (kMaxK - 1) / 2 + kWave - 1) / kWave;

// Sum over the wavefront (every lane).
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

__global__ __launch_bounds__(kWave) void conflicts_kernel(
    int K, const double *__restrict__ gram, double *__restrict__ cosines, double *__restrict__ summary,
    int32_t *__restrict__ pairs) {
  const int64_t b = blockIdx.x;
  const int t = threadIdx.x;
  const double *G = gram + b * K * K;
  double *cb = cosines ? cosines + b * K * K : nullptr;

  bool finite = true;
  for (int q = t; q < K * K; q += kWave) finite = finite && __builtin_isfinite(G[q]);
  if (!__all(finite)) {
    const double nan = __builtin_nan("");
    if (cb)
      for (int q = t; q < K * K; q += kWave) cb[q] = nan;
    if (t < 3) {
      if (summary) summary[3 * b + t] = nan;
      if (pairs) pairs[3 * b + t] = -1;
    }
    return;
  }

  const int npairs = K * (K - 1) / 2;
  if (cb && t < K) cb[t * K + t] = G[t * K + t] > 0.0 ? 1.0 : 0.0;
  // this lane's pairs, in lexicographic order of (i, j): their cosines, the
  // least of them (`at`: its rank; a NaN, from a product of squared norms
  // out of range, is never less) and how many inner products are negative
  double c[kPairsPerLane], sum = 0.0, best = __builtin_inf();
  int at = kMaxK * kMaxK, count = 0;
#pragma unroll
  for (int u = 0; u < kPairsPerLane; ++u) {
    const int p = t + u * kWave;
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
  sum = wave_sum(sum);
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) {
    const double ob = __shfl_xor(best, off, kWave);
    const int oa = __shfl_xor(at, off, kWave);
    count += __shfl_xor(count, off, kWave);
    if (ob < best || (ob == best && oa < at)) {
      best = ob;
      at = oa;
    }
  }
  // the first pair stands unless another is less, also when it is a NaN
  const double first = __shfl(c[0], 0, kWave);
  if (at >= npairs || first != first) {
    best = first;
    at = 0;
  }
  const double mean = sum / npairs;
  double ss = 0.0;
#pragma unroll
  for (int u = 0; u < kPairsPerLane; ++u) {
    const double d = c[u] - mean;
    if (t + u * kWave < npairs) ss += d * d;
  }
  ss = wave_sum(ss);
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

}  // namespace

hipError_t launch_conflicts(int K, int B, const double *gram, double *cosines, double *summary,
                            int32_t *pairs, hipStream_t s) {
  hipLaunchKernelGGL(conflicts_kernel, dim3((unsigned)B), dim3(kWave), 0, s, K, gram, cosines, summary, pairs);
  return hipGetLastError();
}

}  // namespace bkmoo
