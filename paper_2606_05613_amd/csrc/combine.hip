// Pass 2: the resolved bucket updates d[o_b:o_{b+1}] = sum_i w_{b,i} x_i,
// concatenated over buckets (Algorithm 1: the per-strategy d_(k), then
// d = [d_(1), ..., d_(K)]).
//
// Bandwidth-bound: K*N*s bytes read, N*s_out written, 2K flops per
// element.  128-bit non-temporal loads as in the Gram pass, whose chunks are
// cut in kCombineParts (one schedule serves both passes: a schedule kernel of
// its own cost every two-pass call 5-6 us).  The schedule counts the parts: with
// two for every chunk, half of them empty where buckets are short, K=4 bf16,
// 20,000 buckets of 64 elements took 231 us instead of 136.  The K weights of a chunk's bucket are wave-uniform scalars.  Unlike the
// Gram pass, chunks are dealt round-robin (chunk c to workgroup c mod grid),
// so the whole grid sweeps the vector together: measured 1-2.5% faster
// than one contiguous run per workgroup on every workload shape here, in
// fast and slow buffer placements alike (the Gram pass gains nothing).
//
// Arithmetic.  For an fp32 output the sum is an fp32 FMA chain in task
// order.  For a bf16 output that is not enough: with bf16 inputs the exact
// sum of w_i x_i often lies within an fp32 rounding error of a bf16 tie
// (e.g. weights of 1/K), and an fp32 chain then rounds the wrong way on a
// few percent of elements.  So the bf16 path accumulates in fp64, where
// every product of an fp32 weight and an fp32/bf16 input is exact, and
// rounds once: fp64 -> fp32 with round-to-odd, then RNE to bf16.  Rounding
// to odd into a format with at least two more significand bits than the
// target makes the second rounding the correct single rounding.
#include "chunk.h"
#include "schedule.h"

namespace bkmoo {

namespace {

template <int K, int DT, int ODT, bool SELF>
__global__ __launch_bounds__(kThreads) void combine_kernel(
    Rows<K> rows, const int64_t *__restrict__ offs, const int64_t *__restrict__ gps, int B,
    int shift, ScheduleOut sched, const float *__restrict__ weights, void *out) {
  constexpr int64_t C = combine_chunk_elems(K, DT);

  __shared__ int64_t lps[SELF ? kSelfBuckets + 1 : 1];
  if constexpr (SELF) {
    if (!own_schedule<true>(offs, B, C * kCombineParts, sum_direct(pairs(K)), sched, lps)) return;
  }
  const int64_t *ps = SELF ? lps : gps;
  const int64_t total = ps[B];

  for (int64_t c = blockIdx.x; c < total; c += gridDim.x) {
    const int b = find_bucket(ps, B, c);
    const int64_t lo = offs[b] + (c - ps[b]) * C;
    const int64_t hi = lo + C < offs[b + 1] ? lo + C : offs[b + 1];
    float w[K];
#pragma unroll
    for (int i = 0; i < K; ++i) w[i] = weights[(int64_t)b * K + i];

    combine_chunk<K, DT, ODT, combine_shape(K).R, combine_shape(K).U>(rows, lo, hi, shift, w, out);
  }
}

template <int K, int DT, int ODT, bool SELF>
hipError_t launch_combine_s(const StreamArgs &a, const float *weights, void *out, hipStream_t s) {
  Rows<K> rows;
  for (int i = 0; i < K; ++i) rows.p[i] = a.rows[i];
  auto kern = combine_kernel<K, DT, ODT, SELF>;
  const int64_t C = combine_chunk_elems(K, DT);
  const int64_t cap = (a.N + C - 1) / C + a.B;
  static const int occ = occupancy(kern);
  constexpr int R = combine_shape(K).R;
  const bool alone = kCombineAlone<K, DT, ODT> &&
                     (DT != BF16 || ODT != BF16 || a.N / gram_chunk_elems(K, DT) >= 32 * (int64_t)a.B);
  int64_t grid = a.grid > 0 ? a.grid : stream_grid(a, R, kCombineParts, alone ? 1 : stream_wgs(K, R), occ, cap);
  if (grid > cap) grid = cap;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), 0, s, rows, a.offsets,
                     a.part_start, a.B, a.shift, ScheduleOut{a.N, a.chunk_start, a.group_start, a.part_start, a.err},
                     weights, out);
  return hipGetLastError();
}

template <int K, int DT, int ODT>
hipError_t launch_combine_t(const StreamArgs &a, const float *weights, void *out, hipStream_t s) {
  return a.scheduled ? launch_combine_s<K, DT, ODT, false>(a, weights, out, s)
                     : launch_combine_s<K, DT, ODT, true>(a, weights, out, s);
}

template <int DT, int ODT>
hipError_t dispatch_combine(const StreamArgs &a, const float *w, void *out, hipStream_t s) {
  switch (a.K) {
    case 2: return launch_combine_t<2, DT, ODT>(a, w, out, s);
    case 3: return launch_combine_t<3, DT, ODT>(a, w, out, s);
    case 4: return launch_combine_t<4, DT, ODT>(a, w, out, s);
    case 5: return launch_combine_t<5, DT, ODT>(a, w, out, s);
    case 6: return launch_combine_t<6, DT, ODT>(a, w, out, s);
    case 7: return launch_combine_t<7, DT, ODT>(a, w, out, s);
    case 8: return launch_combine_t<8, DT, ODT>(a, w, out, s);
    case 9: return launch_combine_t<9, DT, ODT>(a, w, out, s);
    case 10: return launch_combine_t<10, DT, ODT>(a, w, out, s);
    case 11: return launch_combine_t<11, DT, ODT>(a, w, out, s);
    case 12: return launch_combine_t<12, DT, ODT>(a, w, out, s);
    case 13: return launch_combine_t<13, DT, ODT>(a, w, out, s);
    case 14: return launch_combine_t<14, DT, ODT>(a, w, out, s);
    case 15: return launch_combine_t<15, DT, ODT>(a, w, out, s);
    case 16: return launch_combine_t<16, DT, ODT>(a, w, out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_combine(const StreamArgs &a, const float *weights, void *out, int out_dt,
                          hipStream_t s) {
  if (a.dt == F32)
    return out_dt == F32 ? dispatch_combine<F32, F32>(a, weights, out, s)
                         : dispatch_combine<F32, BF16>(a, weights, out, s);
  return out_dt == F32 ? dispatch_combine<BF16, F32>(a, weights, out, s)
                       : dispatch_combine<BF16, BF16>(a, weights, out, s);
}

}  // namespace bkmoo
