// The per-bucket MOO subproblem, solved from the bucket's Gram matrix alone.
//
// One wavefront per bucket, everything in fp64 in LDS and registers (the
// solvers are in solve_impl.h).  This file is compiled without
// floating-point contraction so every scalar expression rounds exactly as
// written.
#include "gram_sum.h"
#include "solve_impl.h"

namespace bkmoo {

namespace {

__global__ __launch_bounds__(kWave) void solve_kernel(int K, const double *__restrict__ gram,
                                                      int method, int iters, double c,
                                                      const int8_t *__restrict__ order,
                                                      float *__restrict__ weights,
                                                      double *__restrict__ aux) {
  __shared__ Shared S;
  const int64_t b = blockIdx.x;
  const int t = threadIdx.x;
  solver_load_gram<WaveSync>(S, K, gram + b * K * K, t, kWave);
  double wt, ax;
  solver_run<WaveSync>(S, K, method, iters, c, order, b, t, &wt, &ax);
  if (t < K) {
    weights[b * K + t] = (float)wt;
    if (aux) aux[b * K + t] = ax;
  }
}

// The same with K fixed at compile time: MGDA and CAGrad run the
// lane-parallel solvers (lane i holds task i's row, O(K) arithmetic per
// step and lane), PCGrad, the mean and non-finite Grams the sequential
// code above.  A K = 2 MGDA FW-20 solve of four buckets took 12.7 us with
// the sequential code, most of the smallest workload's step.
template <int K>
__global__ __launch_bounds__(kWave) void lane_solve_kernel(const double *__restrict__ gram, int method,
                                                           int iters, double c,
                                                           const int8_t *__restrict__ order,
                                                           float *__restrict__ weights,
                                                           double *__restrict__ aux) {
  __shared__ Shared S;
  const int64_t b = blockIdx.x;
  const int t = threadIdx.x;
  solver_load_gram<WaveSync>(S, K, gram + b * K * K, t, kWave);
  double wt = 0.0, ax = 0.0;
  if (S.bad || (method != MGDA && method != CAGRAD))
    solver_run<WaveSync>(S, K, method, iters, c, order, b, t, &wt, &ax);
  else if (method == MGDA)
    wt = ax = lane_solve_mgda<K>(S.G, iters, t);
  else
    lane_solve_cagrad<K>(S.G, iters, c, t, &wt, &ax);
  if (t < K) {
    weights[b * K + t] = (float)wt;
    if (aux) aux[b * K + t] = ax;
  }
}

// A resolve call's finalize and solve in one launch, a workgroup per bucket:
// the workgroup adds the bucket's partial slots (in the order of the Gram
// finalize, so the matrix is bit for bit what bkmoo_gram writes) into LDS,
// its first wavefront solves from there.  As two kernels with a launch each
// the smallest step spent 13 of its 41 us here.  KT = 0: K at run time, the
// sequential solvers (K > 10).
template <int KT, int T>
__global__ __launch_bounds__(T) void gram_solve_kernel(int Krt, const int64_t *__restrict__ cs,
                                                                 const double *__restrict__ partials,
                                                                 const uint32_t *__restrict__ err, int method,
                                                                 int iters, double c,
                                                                 const int8_t *__restrict__ order,
                                                                 double *__restrict__ gram,
                                                                 float *__restrict__ weights,
                                                                 double *__restrict__ aux) {
  __shared__ Shared S;
  __shared__ double red[kSumThreads];
  const int K = KT > 0 ? KT : Krt, P = K * (K + 1) / 2;
  const int64_t b = blockIdx.x;
  const int t = threadIdx.x;
  if (t == 0) S.bad = 0;
  double s = sum_bucket<T>(partials, cs, b, P, red);
  if (t < P) {
    if (*err & kErrOffsets) s = __builtin_nan("");
    int i, j;
    pair_of(t, K, i, j);
    S.G[i * K + j] = s;
    S.G[j * K + i] = s;
    if (!__builtin_isfinite(s)) S.bad = 1;
  }
  __syncthreads();
  if constexpr (T == kWave) {
    for (int e = t; e < K * K; e += T) gram[b * K * K + e] = S.G[e];
  } else if (t >= kWave) {  // the other wavefronts write the matrix
    for (int e = t - kWave; e < K * K; e += T - kWave) gram[b * K * K + e] = S.G[e];
    return;
  }
  double wt = 0.0, ax = 0.0;
  if constexpr (KT == 0) {
    solver_run<WaveSync>(S, K, method, iters, c, order, b, t, &wt, &ax);
  } else {
    if (S.bad || (method != MGDA && method != CAGRAD))
      solver_run<WaveSync>(S, K, method, iters, c, order, b, t, &wt, &ax);
    else if (method == MGDA)
      wt = ax = lane_solve_mgda<KT>(S.G, iters, t);
    else
      lane_solve_cagrad<KT>(S.G, iters, c, t, &wt, &ax);
  }
  if (t < K) {
    weights[b * K + t] = (float)wt;
    if (aux) aux[b * K + t] = ax;
  }
}

template <int K>
void launch_gram_solve_t(const StreamArgs &a, const double *partials, double *gram, int method, int max_iter, double c,
                         const int8_t *order, float *weights, double *aux, hipStream_t s) {
  const int T = sum_workgroup(a);
  hipLaunchKernelGGL((T == kWave ? gram_solve_kernel<K, kWave> : gram_solve_kernel<K, kSumThreads>),
                     dim3((unsigned)a.B), dim3((unsigned)T), 0, s, a.K, a.chunk_start, partials, a.err, method, max_iter, c, order, gram, weights, aux);
}

template <int K>
void launch_lane_solve(int B, const double *gram, int method, int max_iter, double c, const int8_t *order,
                       float *weights, double *aux, hipStream_t s) {
  hipLaunchKernelGGL(lane_solve_kernel<K>, dim3((unsigned)B), dim3(kWave), 0, s, gram, method, max_iter, c,
                     order, weights, aux);
}

}  // namespace

hipError_t launch_gram_solve(const StreamArgs &a, const double *partials, double *gram, int method, int max_iter,
                             double c, const int8_t *order, float *weights, double *aux, hipStream_t s) {
#define BKMOO_GS_CASE(k) \
  case k: launch_gram_solve_t<k>(a, partials, gram, method, max_iter, c, order, weights, aux, s); break;
  switch (a.K) {
    BKMOO_GS_CASE(2) BKMOO_GS_CASE(3) BKMOO_GS_CASE(4) BKMOO_GS_CASE(5) BKMOO_GS_CASE(6) BKMOO_GS_CASE(7)
    BKMOO_GS_CASE(8) BKMOO_GS_CASE(9) BKMOO_GS_CASE(10)
    default: launch_gram_solve_t<0>(a, partials, gram, method, max_iter, c, order, weights, aux, s);
  }
#undef BKMOO_GS_CASE
  return hipGetLastError();
}

hipError_t launch_solve(int K, int B, const double *gram, int method, int max_iter, double c,
                        const int8_t *order, float *weights, double *aux, hipStream_t s) {
  if (method == MGDA_EXACT || method == CAGRAD_EXACT)
    return launch_exact_solve(K, B, gram, method, c, weights, aux, s);
  switch (K) {
    case 2: launch_lane_solve<2>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 3: launch_lane_solve<3>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 4: launch_lane_solve<4>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 5: launch_lane_solve<5>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 6: launch_lane_solve<6>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 7: launch_lane_solve<7>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 8: launch_lane_solve<8>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 9: launch_lane_solve<9>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    case 10: launch_lane_solve<10>(B, gram, method, max_iter, c, order, weights, aux, s); break;
    default:
      hipLaunchKernelGGL(solve_kernel, dim3((unsigned)B), dim3(kWave), 0, s, K, gram, method, max_iter, c,
                         order, weights, aux);
  }
  return hipGetLastError();
}

}  // namespace bkmoo
