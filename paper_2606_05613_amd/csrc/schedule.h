// The bucket schedule on one workgroup: of the schedule kernel, or of every
// workgroup of a streaming pass that makes its own.
#pragma once

#include "internal.h"

namespace bkmoo {

namespace {

// Running sums over buckets: x their chunks; y their finalize groups (from bit
// 32 up) and how many of them end in the first half of a chunk, so that the last
// chunk has one combine part (the bits below, at most B < 2^31 in all).
struct Sums {
  int64_t x, y;
  __device__ __forceinline__ int64_t chunks() const { return x; }
  __device__ __forceinline__ int64_t groups() const { return y >> 32; }
  __device__ __forceinline__ int64_t parts() const { return kCombineParts * x - (y & 0xffffffff); }
};
static_assert(kCombineParts == 2, "a chunk's parts are its halves");

// Inclusive sums over the workgroup's threads: shuffles in the wavefront, then
// the wavefronts' totals (tot, two barriers).
template <int T>
__device__ __forceinline__ Sums block_scan(Sums s, Sums (&tot)[T / kWave]) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int64_t ax = __shfl_up(s.x, d, kWave), ay = __shfl_up(s.y, d, kWave);
    if (lane >= d) {
      s.x += ax;
      s.y += ay;
    }
  }
  __syncthreads();  // `tot` of the tile before
  if (lane == kWave - 1) tot[wave] = s;
  __syncthreads();
  for (int w = 0; w < wave; ++w) {
    s.x += tot[w].x;
    s.y += tot[w].y;
  }
  return s;
}

// Checks the offsets and calls put(b, s) for b = 0 .. B with the sums over the
// buckets before b (chunks of C elements, no finalize groups below `direct`); false
// (and no call) if the offsets are not 0 = o_0 <= ... <= o_B = N.
template <int T, typename Put>
__device__ __forceinline__ bool block_schedule(const int64_t *__restrict__ offs, int B, int64_t N, int64_t C,
                                               int64_t direct, Put put) {
  __shared__ Sums tot[T / kWave];
  const int tid = threadIdx.x;
  int bad = offs[0] != 0 || offs[B] != N;
  for (int b = tid; b < B; b += T) bad |= offs[b + 1] < offs[b];
  if (__syncthreads_or(bad)) return false;
  Sums carry{0, 0};
  for (int base = 0; base < B; base += T) {
    const int b = base + tid;
    const int64_t n = b < B ? offs[b + 1] - offs[b] : 0;
    const int64_t cnt = (n + C - 1) / C;
    const int64_t groups = cnt < direct ? 0 : (cnt + kFinalizeGroup - 1) / kFinalizeGroup;
    const bool half = n > 0 && n - (cnt - 1) * C <= C / kCombineParts;
    const Sums own{cnt, (groups << 32) + (half ? 1 : 0)};
    const Sums s = block_scan<T>(own, tot);
    if (b < B) put(b, Sums{carry.x + s.x - own.x, carry.y + s.y - own.y});
    for (int w = 0; w < T / kWave; ++w) {
      carry.x += tot[w].x;
      carry.y += tot[w].y;
    }
  }
  if (tid == 0) put(B, carry);
  return true;
}

// Invalid offsets: no chunk is processed, the error word says why.
__device__ __forceinline__ void reject_offsets(int B, int64_t *cs, int64_t *gs, int64_t *ps, uint32_t *err) {
  for (int b = threadIdx.x; b <= B; b += blockDim.x) {
    cs[b] = 0;
    if (gs) gs[b] = 0;
    if (ps) ps[b] = 0;
  }
  if (threadIdx.x == 0) {
    err[0] = kErrOffsets;
    err[1] = 0u;
  }
}

// A streaming pass's own schedule (SELF: at most kSelfBuckets buckets): every
// workgroup makes the prefix it needs for itself in LDS, of chunks or (PARTS) of
// combine parts; workgroup 0 also leaves these, the group prefix and the error
// word in the workspace for the kernels that follow.  As a kernel of its own the schedule takes 4.5 us and a launch
// of a step of 30 (K=2, 1M fp32); a workgroup that starts with it needs about
// 1.5 us, and finds a chunk's bucket in LDS rather than in memory.
constexpr int kSelfBuckets = 511;
struct ScheduleOut {
  int64_t N;
  int64_t *cs, *gs, *ps;
  uint32_t *err;
};
template <bool PARTS>
__device__ __forceinline__ bool own_schedule(const int64_t *__restrict__ offs, int B, int64_t C, int64_t direct,
                                             const ScheduleOut &o, int64_t (&lcs)[kSelfBuckets + 1]) {
  const bool writes = blockIdx.x == 0;
  const bool ok = block_schedule<kThreads>(offs, B, o.N, C, direct, [&](int b, Sums before) {
    lcs[b] = PARTS ? before.parts() : before.chunks();
    if (writes) {
      o.cs[b] = before.chunks();
      o.gs[b] = before.groups();
      o.ps[b] = before.parts();
    }
  });
  if (!ok) {
    if (writes) reject_offsets(B, o.cs, o.gs, o.ps, o.err);
    return false;
  }
  if (writes && threadIdx.x == 0) o.err[0] = o.err[1] = 0u;
  __syncthreads();
  return true;
}

}  // namespace

}  // namespace bkmoo
