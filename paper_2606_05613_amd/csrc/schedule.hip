// Bucket schedule: validates the bucket offsets and cuts every bucket into
// chunks of C elements that never straddle a bucket boundary (the partition
// of the parameter vector into disjoint contiguous buckets, Section 3.2).
#include "schedule.h"

namespace bkmoo {

namespace {

constexpr int kSchedThreads = 1024;

// Workgroup 0.  chunk_start[b] = sum_{b' < b} ceil(n_b' / C) and, when
// group_start is given, group_start[b] = the finalize groups of the buckets
// before b (none in a bucket of fewer than `direct` chunks), part_start[b]
// their combine parts.
// On invalid offsets every entry is 0 (so no chunk is processed) and the
// error word gets kErrOffsets.  Otherwise the error word is cleared.  With a
// plan (plan.groups > 0) the word after it says whether the cooperative
// kernel runs its tiled form (see PipePlan).  The other workgroups zero
// `nsync` words at `sync`.
__global__ __launch_bounds__(kSchedThreads) void schedule_kernel(
    const int64_t *__restrict__ offs, int B, int64_t N, int64_t C, int64_t direct, int64_t *__restrict__ cs,
    int64_t *__restrict__ gs, int64_t *__restrict__ ps, uint32_t *__restrict__ err, uint32_t *__restrict__ sync,
    int64_t nsync, PipePlan plan) {
  const int tid = threadIdx.x;
  if (blockIdx.x > 0) {
    const int64_t stride = (int64_t)(gridDim.x - 1) * kSchedThreads;
    for (int64_t i = (int64_t)(blockIdx.x - 1) * kSchedThreads + tid; i < nsync; i += stride) sync[i] = 0u;
    return;
  }
  __shared__ unsigned long long load[kMaxPlanGroups];  // estimated ns of each group's buckets
  if (tid < kMaxPlanGroups) load[tid] = 0;
  const bool ok = block_schedule<kSchedThreads>(offs, B, N, C, direct, [&](int b, Sums before) {
    cs[b] = before.chunks();
    if (gs) gs[b] = before.groups();
    if (ps) ps[b] = before.parts();
    if (plan.groups > 0 && b < B)
      atomicAdd(&load[b % plan.groups], (unsigned long long)plan.bucket_ns(offs[b + 1] - offs[b]));
  });
  if (!ok) {
    reject_offsets(B, cs, gs, ps, err);
    return;
  }
  __syncthreads();
  if (tid == 0) {
    err[0] = 0u;
    unsigned long long most = 0;
    for (int g = 0; g < plan.groups; ++g) most = load[g] > most ? load[g] : most;
    err[1] = plan.groups > 0 && plan.tiled(most, N) ? 1u : 0u;
  }
}

}  // namespace

hipError_t launch_schedule(const int64_t *offsets, int B, int64_t N, int64_t C, int64_t direct, int64_t *chunk_start,
                           int64_t *group_start, int64_t *part_start, uint32_t *err, uint32_t *sync, int64_t nsync,
                           const PipePlan &plan, hipStream_t s) {
  // workgroup 0 schedules, up to 64 others clear
  const int64_t clear = (nsync + kSchedThreads - 1) / kSchedThreads;
  hipLaunchKernelGGL(schedule_kernel, dim3((unsigned)(1 + (clear < 64 ? clear : 64))), dim3(kSchedThreads), 0, s,
                     offsets, B, N, C, direct, chunk_start, group_start, part_start, err, sync,
                     nsync, plan);
  return hipGetLastError();
}

}  // namespace bkmoo
