// Bucket schedule: validates the bucket offsets and cuts every bucket into
// chunks of C elements that never straddle a bucket boundary (the partition
// of the parameter vector into disjoint contiguous buckets, Section 3.2).
#include "internal.h"

namespace bkmoo {

namespace {

constexpr int kSchedThreads = 1024;

// Inclusive sums of x and y over the workgroup's threads: shuffles in the
// wavefront, then the wavefronts' totals (tot, two barriers).
struct Sums {
  int64_t x, y;
};
__device__ __forceinline__ Sums block_scan(Sums s, Sums (&tot)[kSchedThreads / kWave]) {
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

// Workgroup 0.  chunk_start[b] = sum_{b' < b} ceil(n_b' / C) and, when
// group_start is given, group_start[b] = sum_{b' < b} ceil(chunks_b' / G)
// (groups of G consecutive chunks of one bucket, the Gram finalize's unit).
// On invalid offsets every entry is 0 (so no chunk is processed) and the
// error word gets kErrOffsets.  Otherwise the error word is cleared.  With a
// plan (plan.groups > 0) the word after it says whether the cooperative
// kernel runs its tiled form (see PipePlan).  The other workgroups zero
// `nsync` words at `sync`.
__global__ __launch_bounds__(kSchedThreads) void schedule_kernel(
    const int64_t *__restrict__ offs, int B, int64_t N, int64_t C, int64_t *__restrict__ cs,
    int64_t G, int64_t *__restrict__ gs, uint32_t *__restrict__ err, uint32_t *__restrict__ sync,
    int64_t nsync, PipePlan plan) {
  const int tid = threadIdx.x;
  if (blockIdx.x > 0) {
    const int64_t stride = (int64_t)(gridDim.x - 1) * kSchedThreads;
    for (int64_t i = (int64_t)(blockIdx.x - 1) * kSchedThreads + tid; i < nsync; i += stride) sync[i] = 0u;
    return;
  }
  __shared__ Sums tot[kSchedThreads / kWave];
  __shared__ unsigned long long load[kMaxPlanGroups];  // estimated ns of each group's buckets
  int bad = offs[0] != 0 || offs[B] != N;
  for (int b = tid; b < B; b += kSchedThreads) bad |= offs[b + 1] < offs[b];
  if (tid < kMaxPlanGroups) load[tid] = 0;
  if (__syncthreads_or(bad)) {
    for (int b = tid; b <= B; b += kSchedThreads) {
      cs[b] = 0;
      if (gs) gs[b] = 0;
    }
    if (tid == 0) {
      err[0] = kErrOffsets;
      err[1] = 0u;
    }
    return;
  }
  Sums carry{0, 0};
  for (int base = 0; base < B; base += kSchedThreads) {
    const int b = base + tid;
    const int64_t n = b < B ? offs[b + 1] - offs[b] : 0;
    const int64_t cnt = (n + C - 1) / C;
    const Sums own{cnt, (cnt + G - 1) / G};
    const Sums s = block_scan(own, tot);
    if (b < B) {
      cs[b] = carry.x + s.x - own.x;
      if (gs) gs[b] = carry.y + s.y - own.y;
      if (plan.groups > 0) atomicAdd(&load[b % plan.groups], (unsigned long long)plan.bucket_ns(n));
    }
    for (int w = 0; w < kSchedThreads / kWave; ++w) {
      carry.x += tot[w].x;
      carry.y += tot[w].y;
    }
  }
  __syncthreads();
  if (tid == 0) {
    cs[B] = carry.x;
    if (gs) gs[B] = carry.y;
    err[0] = 0u;
    unsigned long long most = 0;
    for (int g = 0; g < plan.groups; ++g) most = load[g] > most ? load[g] : most;
    err[1] = plan.groups > 0 && plan.tiled(most, N) ? 1u : 0u;
  }
}

}  // namespace

hipError_t launch_schedule(const int64_t *offsets, int B, int64_t N, int64_t C, int64_t *chunk_start,
                           int64_t *group_start, uint32_t *err, uint32_t *sync, int64_t nsync,
                           const PipePlan &plan, hipStream_t s) {
  // workgroup 0 schedules, up to 64 others clear
  const int64_t clear = (nsync + kSchedThreads - 1) / kSchedThreads;
  hipLaunchKernelGGL(schedule_kernel, dim3((unsigned)(1 + (clear < 64 ? clear : 64))), dim3(kSchedThreads), 0, s,
                     offsets, B, N, C, chunk_start, (int64_t)kFinalizeGroup, group_start, err, sync, nsync, plan);
  return hipGetLastError();
}

}  // namespace bkmoo
