// Pass 1: per-bucket Gram matrices G_b[i][j] = <x_i, x_j> over the bucket.
//
// The bucket-level problems (Eq. shard-mgda, the local CAGrad problem and
// PCGrad's local conflict test, Section 3.2) depend on the local gradients
// only through these inner products, so this pass is the only one that
// needs all K rows at once.  It is HBM-bound: K*N*s bytes read, K(K+1)
// flops per element position, far below the fp32 vector ridge point, so
// it uses plain fp32 FMAs and no matrix cores.
//
// Design (gfx950): persistent workgroups of 4 wavefronts own contiguous
// runs of chunks.  Every thread issues K*R independent 128-bit
// non-temporal loads per iteration and accumulates all K(K+1)/2 products
// in fp32 registers over the chunk's iterations.  Lane sums are combined by
// a fixed xor butterfly across the wavefront, then in fp64 across the 4
// wavefronts through LDS in wave order, and land in a per-chunk slot.  The
// finalize adds a bucket's chunk slots in fp64 in an order fixed by the
// bucket's chunk count and N (where a bucket can have many chunks, groups of
// consecutive chunks first, then the groups); a resolve call adds them in
// the kernel that also solves the bucket's problem (solve.hip).  No atomics:
// the result is bitwise independent of the grid and of scheduling.
#include "chunk.h"
#include "gram_sum.h"

namespace bkmoo {

namespace {

template <int K, int DT>
__global__ __launch_bounds__(kThreads) void gram_partial_kernel(
    Rows<K> rows, const int64_t *__restrict__ offs, const int64_t *__restrict__ cs, int B,
    int shift, double *__restrict__ partials) {
  constexpr int64_t C = gram_chunk_elems(K, DT);
  constexpr int P = pairs(K);
  __shared__ double red[kThreads / kWave][P];

  int64_t c, cend;
  my_chunks(cs[B], c, cend);
  if (c >= cend) return;
  int b = find_bucket(cs, B, c);
  const int tid = threadIdx.x;

  for (; c < cend; ++c) {
    while (cs[b + 1] <= c) ++b;
    const int64_t lo = offs[b] + (c - cs[b]) * C;
    const int64_t hi = lo + C < offs[b + 1] ? lo + C : offs[b + 1];

    float acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] = 0.0f;

    gram_chunk<K, DT>(rows, lo, hi, shift, acc);

    // fixed-order reduction; the 4 wavefronts in order
    reduce_lanes<P>(acc, red);
    __syncthreads();
    for (int p = tid; p < P; p += kThreads) {
      double s = red[0][p];
#pragma unroll
      for (int w = 1; w < kThreads / kWave; ++w) s += red[w][p];
      partials[c * P + p] = s;
    }
    __syncthreads();
  }
}

// Finalize, level 1 (only where a bucket can have many chunks): one workgroup
// per group of up to kFinalizeGroup consecutive chunks of one bucket
// (grid-stride over the groups) leaves the group's sum in the slot of the
// group's first chunk, which only this workgroup reads.
__global__ __launch_bounds__(kSumThreads) void gram_group_kernel(int P, int B, const int64_t *__restrict__ cs,
                                                                 const int64_t *__restrict__ gs, double *partials) {
  __shared__ double red[kSumThreads];
  const int64_t total = gs[B];
  for (int64_t v = blockIdx.x; v < total; v += gridDim.x) {
    const int b = find_bucket(gs, B, v);
    const int64_t c0 = cs[b] + (v - gs[b]) * kFinalizeGroup, left = cs[b + 1] - c0;
    const double s = sum_slots<kSumThreads>(partials, c0, left < kFinalizeGroup ? left : kFinalizeGroup, 1, P, red);
    if ((int)threadIdx.x < P) partials[c0 * P + threadIdx.x] = s;
    __syncthreads();  // `red` before the next group
  }
}

// Finalize, level 2: one workgroup per bucket adds the bucket's chunk slots
// (step 1) or group sums (step kFinalizeGroup) and writes the symmetric
// K x K matrix (NaN everywhere when the offsets were rejected by the
// schedule).
__global__ __launch_bounds__(kSumThreads) void gram_finalize_kernel(int K, const int64_t *__restrict__ cs, int step,
                                                                    const double *__restrict__ partials,
                                                                    const uint32_t *__restrict__ err,
                                                                    double *__restrict__ gram) {
  __shared__ double red[kSumThreads];
  const int64_t b = blockIdx.x;
  const int P = K * (K + 1) / 2;
  double s = sum_slots<kSumThreads>(partials, cs[b], (cs[b + 1] - cs[b] + step - 1) / step, step, P, red);
  if ((int)threadIdx.x < P) {
    if (*err & kErrOffsets) s = __builtin_nan("");
    int i, j;
    pair_of((int)threadIdx.x, K, i, j);
    gram[(b * K + i) * K + j] = s;
    gram[(b * K + j) * K + i] = s;
  }
}

template <int K, int DT>
hipError_t launch_gram_t(const StreamArgs &a, double *partials, hipStream_t s) {
  Rows<K> rows;
  for (int i = 0; i < K; ++i) rows.p[i] = a.rows[i];
  auto kern = gram_partial_kernel<K, DT>;
  const int64_t C = gram_chunk_elems(K, DT);
  const int64_t cap = (a.N + C - 1) / C + a.B;
  static const int occ = occupancy(kern);
  int64_t grid = a.grid > 0 ? a.grid : (int64_t)device_cu_count() * occ;
  if (grid > cap) grid = cap;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), 0, s, rows, a.offsets,
                     a.chunk_start, a.B, a.shift, partials);
  return hipGetLastError();
}

template <int DT>
hipError_t dispatch_gram(const StreamArgs &a, double *partials, hipStream_t s) {
  switch (a.K) {
    case 2: return launch_gram_t<2, DT>(a, partials, s);
    case 3: return launch_gram_t<3, DT>(a, partials, s);
    case 4: return launch_gram_t<4, DT>(a, partials, s);
    case 5: return launch_gram_t<5, DT>(a, partials, s);
    case 6: return launch_gram_t<6, DT>(a, partials, s);
    case 7: return launch_gram_t<7, DT>(a, partials, s);
    case 8: return launch_gram_t<8, DT>(a, partials, s);
    case 9: return launch_gram_t<9, DT>(a, partials, s);
    case 10: return launch_gram_t<10, DT>(a, partials, s);
    case 11: return launch_gram_t<11, DT>(a, partials, s);
    case 12: return launch_gram_t<12, DT>(a, partials, s);
    case 13: return launch_gram_t<13, DT>(a, partials, s);
    case 14: return launch_gram_t<14, DT>(a, partials, s);
    case 15: return launch_gram_t<15, DT>(a, partials, s);
    case 16: return launch_gram_t<16, DT>(a, partials, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int gram_sum_step(int K, int dt, int64_t N) { return N / gram_chunk_elems(K, dt) < kSumDirect ? 1 : kFinalizeGroup; }

hipError_t launch_gram_partials(const StreamArgs &a, double *partials, hipStream_t s) {
  hipError_t e = a.dt == F32 ? dispatch_gram<F32>(a, partials, s) : dispatch_gram<BF16>(a, partials, s);
  if (e != hipSuccess || gram_sum_step(a.K, a.dt, a.N) == 1) return e;
  const int64_t groups = a.N / (gram_chunk_elems(a.K, a.dt) * kFinalizeGroup) + a.B;
  const int64_t limit = (int64_t)device_cu_count() * 4;
  hipLaunchKernelGGL(gram_group_kernel, dim3((unsigned)(groups < limit ? groups : limit)), dim3(kSumThreads), 0, s,
                     pairs(a.K), a.B, a.chunk_start, a.group_start, partials);
  return hipGetLastError();
}

hipError_t launch_gram_finalize(const StreamArgs &a, const double *partials, double *gram, hipStream_t s) {
  hipLaunchKernelGGL(gram_finalize_kernel, dim3((unsigned)a.B), dim3(kSumThreads), 0, s, a.K, a.chunk_start,
                     gram_sum_step(a.K, a.dt, a.N), partials, a.err, gram);
  return hipGetLastError();
}

}  // namespace bkmoo
