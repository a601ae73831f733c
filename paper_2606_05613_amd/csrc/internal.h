// Internal declarations shared by the bkmoo translation units (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace bkmoo {

constexpr int kMinK = 2;
constexpr int kMaxK = 16;
constexpr int kExactMaxK = 10;  // exact solvers: 2^K - 1 supports per bucket
constexpr int kHybridMaxK = 8;  // the pipelined cooperative resolve (hybrid.hip)
constexpr int kThreads = 256;          // streaming kernels: 4 wavefronts of 64
constexpr int kWave = 64;

enum Dtype : int { F32 = 0, BF16 = 1 };

// Vectors of 16 bytes: 4 fp32 or 8 bf16 elements.
constexpr int vec_elems(int dt) { return dt == F32 ? 4 : 8; }
constexpr int elem_bytes(int dt) { return dt == F32 ? 4 : 2; }

// Streaming-pass shapes.  A chunk is U iterations of kThreads * R 16-byte
// vectors per task row; chunks never straddle buckets, so bucket b holds
// ceil(n_b / C) chunks.  K * R bounds the registers holding loaded data (4
// per vector) next to the pass's accumulators; occupancy supplies the rest
// of the memory-level parallelism.  The two passes are tuned separately
// (measured on MI355X): the Gram pass prefers long chunks (fewer fixed-order
// reductions), the combine pass shorter ones.  Above K = 4 one vector per
// row and iteration keeps the Gram kernel under 256 VGPRs (two wavefronts
// per SIMD instead of one at K = 8: 19.5 ms instead of 23.5 ms for 128 GB)
// and speeds the combine by 5%.  R * U is the same for every K <= 8, and a
// lane visits its vectors of a chunk in the same order for R = 1 and R = 2,
// so the Gram sums do not depend on the shape.  Each thread accumulates
// R * U * V elements of a chunk in fp32 in the Gram pass.
struct PassShape {
  int R, U;
};
constexpr PassShape gram_shape(int K) { return K <= 4 ? PassShape{2, 8} : PassShape{1, 16}; }
constexpr PassShape combine_shape(int K) { return K <= 4 ? PassShape{2, 4} : PassShape{1, 8}; }

constexpr int64_t shape_elems(PassShape p, int dt) {
  return (int64_t)kThreads * p.R * p.U * vec_elems(dt);
}
constexpr int64_t gram_chunk_elems(int K, int dt) { return shape_elems(gram_shape(K), dt); }
constexpr int64_t combine_chunk_elems(int K, int dt) { return shape_elems(combine_shape(K), dt); }
// The combine pass cuts every Gram chunk into this many of its own (parts), so
// that one schedule serves both passes; a bucket's last chunk has one part if
// that holds its rest.
constexpr int kCombineParts = 2;
constexpr bool combine_parts_fit() {
  for (int K = kMinK; K <= kMaxK; ++K)
    for (int dt = 0; dt < 2; ++dt)
      if (gram_chunk_elems(K, dt) != kCombineParts * combine_chunk_elems(K, dt)) return false;
  return true;
}
static_assert(combine_parts_fit(), "a Gram chunk is kCombineParts combine chunks");

constexpr int pairs(int K) { return K * (K + 1) / 2; }

// Threads that add up a bucket's slots side by side in the Gram finalize: at
// K = 16 (136 pairs) three rows of them.
constexpr int kSumThreads = 512;
static_assert(kSumThreads >= pairs(kMaxK), "a thread per pair");

// The Gram finalize adds the chunk slots of a bucket of fewer than sum_direct
// chunks directly, one workgroup per bucket; in a longer bucket groups of
// kFinalizeGroup consecutive chunks come first (one workgroup per group, so that
// a single large bucket is not added by one), then the group sums.  Groups of
// 64 fill the chip sooner than the 1024 used before: K=8 bf16, one bucket of
// 124M elements (3,798 chunks), 40 + 5 us for the two kernels with 1024.
// Which of the two it is depends on the bucket (and K) alone, so its matrix is the
// same bits whatever else the call holds; and short buckets have no groups (K=2
// fp32, 20,000 buckets of one chunk, a group each: 209 us for the group kernel).
// The line, 64 slots a thread: groups save (or cost) us, ten buckets, K=16 at 190
// chunks -0.6, 260 1.4, 400 6.5; K=12 260 -1.0, 400 1.3; K=10 260 -1.0, 400 1.5;
// K=8 505 -0.4; K=4 and K=2 505 -2.4 and -3.6.
constexpr int kFinalizeGroup = 64;
constexpr int64_t kMaxSumDirect = 512;
__host__ __device__ constexpr int64_t sum_direct(int P) {
  return kSumThreads / P * kFinalizeGroup < kMaxSumDirect ? kSumThreads / P * kFinalizeGroup : kMaxSumDirect;
}
// Size of a finalize group in the workspace's layout (see Layout::part_start).
constexpr int kLayoutGroup = 1024;

// Partial-Gram slots the workspace always has room for (the pipelined
// cooperative kernel uses two sets of one slot per workgroup that holds data).
constexpr int64_t kCoopSlots = 1024;

// The cooperative kernel's per-bucket arrival counters and flags sit 128
// bytes apart (one per cache line): with 4-byte neighbours, device-scope
// atomics on one bucket's counter and polls of the next buckets' counters
// contend for the same line (measured: 1.4 ms of a 23 ms step).
constexpr int64_t kSyncStride = 32;  // uint32 words
// Copies of each bucket's weights flag on the cooperative path: ~500 data
// workgroups poll it, and one copy (one line, one memory channel) per
// eighth of them keeps the polls from queueing on one channel.
constexpr int kFlagCopies = 8;

// Workspace layout (every region 256-byte aligned):
//   [0, 256)            header: uint32 error word at byte 0, the tiled-form word at byte 4
//   chunk_start         int64 [B + 1]     (prefix sum of chunks per bucket)
//   gram                fp64  [B][K][K]   (used when the caller passes none)
//   weights             fp32  [B][K]      (used when the caller passes none)
//   partials            fp64  [cap][P]    cap = ceil(N / C) + B (at least kCoopSlots slots of P
//                                         rounded up to even)
//   group_start         int64 [B + 1]     (prefix sum of finalize groups per bucket)
//   part_start          int64 [B + 1]     (prefix sum of combine parts), in a region of fp64
//                       [cap / kLayoutGroup + B + 1][P]; the rest of it is unused, which keeps a
//                       workspace's size, and with it which calls the library's fixed scratch
//                       can hold, as callers know them
//   sync                uint32 [1 + kFlagCopies][B][kSyncStride]  cooperative path: arrival
//                       counters, then kFlagCopies copies of the flags
struct Layout {
  size_t err, chunk_start, gram, weights, partials, group_start, part_start, sync, total;
  int64_t cap_chunks;
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

inline Layout layout(int K, int64_t N, int B, int dt) {
  Layout L;
  const int64_t C = gram_chunk_elems(K, dt);  // the smallest chunk with partial slots
  L.cap_chunks = (N + C - 1) / C + B;
  // at least two sets of slots for up to 512 workgroups of a cooperative kernel
  if (L.cap_chunks < kCoopSlots) L.cap_chunks = kCoopSlots;
  size_t o = 0;
  L.err = o;            o += 256;
  L.chunk_start = o;    o = align256(o + sizeof(int64_t) * (size_t)(B + 1));
  L.gram = o;           o = align256(o + sizeof(double) * (size_t)B * K * K);
  L.weights = o;        o = align256(o + sizeof(float) * (size_t)B * K);
  // (the single-buffer cooperative kernel pads each slot to an even count)
  const int64_t part = L.cap_chunks * pairs(K) > kCoopSlots * (pairs(K) + (pairs(K) & 1))
                           ? L.cap_chunks * pairs(K) : kCoopSlots * (pairs(K) + (pairs(K) & 1));
  L.partials = o;       o = align256(o + sizeof(double) * (size_t)part);
  L.group_start = o;    o = align256(o + sizeof(int64_t) * (size_t)(B + 1));
  L.part_start = o;     o = align256(o + sizeof(double) * (size_t)(L.cap_chunks / kLayoutGroup + B + 1) * pairs(K));
  L.sync = o;           o = align256(o + sizeof(uint32_t) * (1 + kFlagCopies) * (size_t)B * kSyncStride);
  L.total = o;
  return L;
}

constexpr uint32_t kErrOffsets = 0x1u;
constexpr uint32_t kErrTimeout = 0x2u;

// Whether the refill kernel runs its pipelined or its tiled form, decided
// where the bucket sizes are known: on the device, from the offsets.
//
// The pipelined form deals bucket b to group b % groups of the workgroups,
// which the host can only size by the average bucket.  Where sizes differ,
// one group's buckets can outlast the others' by far (GPT-2 with a bucket per
// tensor, K=4 bf16: the 38.6M-element embedding of 124M on 17 of 512
// workgroups, 1.70 ms against 0.51 tiled), and a small bucket costs a hand-off
// whatever its size.  The tiled form reads everything twice but spreads every
// bucket over the chip.  Estimates, from times on MI355X: a bucket takes
// elem_ns an element on the whole chip (its group has 1/groups of that) and at
// least a hand-off; the tiled form tile_elem_ns an element and tile_fixed_ns.
// The first estimate is high where one group outlasts the others, as its
// workgroups are then faster than their share of the chip: the tiled form starts
// at 1.2 times.  At 1.1, 2.4 GiB of gradients in 40 buckets of which one holds a
// third took the tiled form (K=3 1,204 us against 1,028-1,106 pipelined, K=2
// 1,460 against 1,332; estimates 1.13 and 1.19 apart); of 706 calls of ragged
// buckets, K = 2 to 10, the form chosen now is at worst 7% behind the other.
// (The two-buffer kernel spreads every bucket over the chip as it is; on
// ragged buckets it stays within a few percent of two reads: K=8 bf16, 11
// to 45 buckets of 125-240 MiB on average, 0.95 to 1.10 times the two passes'
// speed.)
constexpr int kMaxPlanGroups = 32;
struct PipePlan {
  int groups;  // 0: no plan (another kernel, or the path is forced)
  double elem_ns, handoff_ns, tile_elem_ns, tile_fixed_ns;
  __host__ __device__ uint64_t bucket_ns(int64_t n) const {
    const double t = (double)n * elem_ns * groups;
    return n == 0 ? 0 : (uint64_t)(t > handoff_ns ? t : handoff_ns);
  }
  __host__ __device__ bool tiled(uint64_t longest_group_ns, int64_t N) const {
    return (double)longest_group_ns > 1.2 * ((double)N * tile_elem_ns + tile_fixed_ns);
  }
};

// Pointers of the K task rows, passed by value as kernel arguments.
template <int K>
struct Rows {
  const void *p[K];
};

// ---- launchers (host) -------------------------------------------------------

struct StreamArgs {
  int K;
  int dt;                      // input dtype
  const void *const *rows;     // host array of K device pointers
  int64_t N;
  int B;
  const int64_t *offsets;      // device [B+1]
  int64_t *chunk_start;        // device [B+1]
  int64_t *group_start;        // device [B+1] finalize groups
  int64_t *part_start;         // device [B+1] combine parts
  uint32_t *err;               // device error word
  bool scheduled;              // these four are there (else the pass makes them, B <= kSelfBuckets)
  int shift;                   // vectors start at elements n = shift (mod V): where the rows are 16-byte
                               // aligned (Gram pass: row 0) and, in the combine, the output's stores
  int grid;                    // workgroups (0: automatic)
};

// Validates offsets, writes chunk_start for chunks of C elements (and, where
// they are not null, the prefixes of finalize groups and of combine parts),
// sets the error word and, by `plan`, the word after it, and zeroes `nsync`
// words at `sync`.  direct: sum_direct.
hipError_t launch_schedule(const int64_t *offsets, int B, int64_t N, int64_t C, int64_t direct, int64_t *chunk_start,
                           int64_t *group_start, int64_t *part_start, uint32_t *err, uint32_t *sync, int64_t nsync,
                           const PipePlan &plan, hipStream_t s);
// Gram pass: per-chunk partials (and group sums, left in the slots of the
// groups' first chunks), then the per-bucket matrices.
hipError_t launch_gram_partials(const StreamArgs &a, double *partials, hipStream_t s);
hipError_t launch_gram_finalize(const StreamArgs &a, const double *partials, double *gram, hipStream_t s);
// The finalize and the solve (not the exact methods) in one kernel.
hipError_t launch_gram_solve(const StreamArgs &a, const double *partials, double *gram, int method, int max_iter,
                             double c, const int8_t *order, float *weights, double *aux, hipStream_t s);
hipError_t launch_solve(int K, int B, const double *gram, int method, int max_iter, double c,
                        const int8_t *order, float *weights, double *aux, hipStream_t s);
hipError_t launch_combine(const StreamArgs &a, const float *weights, void *out, int out_dt,
                          hipStream_t s);
hipError_t launch_conflicts(int K, int B, const double *gram, double *cosines, double *summary,
                            int32_t *pairs, hipStream_t s);
// Bucket slices and the slice-order sum of partial Grams.
hipError_t launch_slice_offsets(const int64_t *offsets, int B, int T, int64_t *out, hipStream_t s);
hipError_t launch_gram_reduce(int K, int B, int T, const double *partial, int bucket_major, double *gram,
                              hipStream_t s);
// Exact MGDA / CAGrad solvers by support enumeration (K <= kExactMaxK).
hipError_t launch_exact_solve(int K, int B, const double *gram, int method, double c, float *weights,
                              double *aux, hipStream_t s);

// Pipelined, partly resident resolve (K <= kHybridMaxK): cooperative grid (0 if the
// combination cannot run this way), and how many of its workgroups hold data
// (the rest solve); partials must hold 2 * data workgroups slots.
int hybrid_grid(int K, int dt, int out_dt);
int hybrid_data_workgroups(int grid);
// Data workgroups dispatched first onto their CU (0 unless the grid is two
// workgroups per CU): the ones a segment skew gives more data.  The
// kHybridSolvers workgroups dispatched right after them are the second
// residents of the solvers' CUs.
int hybrid_older_workgroups(int grid);
constexpr int kHybridSolvers = 4;  // workgroups of the hybrid grid that reduce and solve

// Segment [lo, hi) (relative to the bucket start) of slot w in a bucket of n
// elements, over gd segment slots in whole units of `unit` elements, and
// the number nseg of non-empty segments, which are always slots 0 ..
// nseg-1.  skew_pm = 0: equal shares.  Otherwise the first `older` slots
// take (1 + skew_pm/1000) times an equal share (rounded up) and the others
// split the rest evenly.
__host__ __device__ inline void hybrid_segment(int64_t n, int w, int gd, int older, int skew_pm, int64_t unit,
                                               int64_t &lo, int64_t &hi, int64_t &nseg) {
  const int64_t nu = (n + unit - 1) / unit;
  int64_t s, e;
  if (skew_pm <= 0 || older <= 0 || older >= gd) {
    const int64_t c = (nu + gd - 1) / gd;
    s = (int64_t)w * c;
    e = s + c;
    nseg = c > 0 ? (nu + c - 1) / c : 0;
  } else {
    const int64_t co = (nu * (1000 + skew_pm) + (int64_t)gd * 1000 - 1) / ((int64_t)gd * 1000);
    const int64_t rest = nu - (int64_t)older * co;
    const int gy = gd - older;
    const int64_t cy = rest > 0 ? (rest + gy - 1) / gy : 0;
    s = w < older ? (int64_t)w * co : (int64_t)older * co + (int64_t)(w - older) * cy;
    e = w < older ? s + co : s + cy;
    nseg = co == 0 ? 0 : rest <= 0 ? (nu + co - 1) / co : older + (cy > 0 ? (rest + cy - 1) / cy : 0);
  }
  lo = s * unit < n ? s * unit : n;
  hi = e * unit < n ? e * unit : n;
}

// How one call spreads each bucket over the hybrid kernel's data
// workgroups.  Data workgroup w holds segment slot(w) of nslots (none when
// slot(w) < 0).  Without `light` the slots are the workgroups themselves;
// with it the solvers' CU mates (the kHybridSolvers workgroups after the
// `older` ones) hold none and leave their CU to the solve.  skew_pm as in
// hybrid_segment.  Shared by the kernel and the host's traffic count.
struct HybLayout {
  int nslots, older, skew_pm, light;
  __host__ __device__ int slot(int w) const {
    return !light || w < older ? w : w < older + kHybridSolvers ? -1 : w - kHybridSolvers;
  }
  // segment of slot s (s < 0: the empty one at the bucket's end)
  __host__ __device__ void segment(int64_t n, int s, int64_t unit, int64_t &lo, int64_t &hi,
                                   int64_t &nseg) const {
    hybrid_segment(n, s < 0 ? nslots : s, nslots, older, skew_pm, unit, lo, hi, nseg);
  }
};
// Elements of its segment a data workgroup keeps on chip per bucket, and the
// granule segment lengths are rounded up to.
int64_t hybrid_held_elems(int K, int dt, int out_dt);
int64_t hybrid_unit_elems(int dt);
hipError_t launch_hybrid(int K, int dt, int out_dt, const void *const *rows, const int64_t *offs, int B,
                         int shift, int method, int iters, double c, const int8_t *order, double *gram,
                         float *weights, double *aux, void *out, double *partials, uint32_t *arrive,
                         uint32_t *flags, uint32_t *err, uint32_t spin_limit, int grid,
                         const HybLayout &layout, hipStream_t s);

int device_cu_count();

// Workgroups of a streaming pass over B buckets that cuts a Gram chunk into
// `parts` and has at most `cap` of these in all.  A long pass is
// fastest with no more wavefronts than keep about 128 KiB of loads in flight
// on a CU (a workgroup has 8 KiB per task and vector of a step, two steps at a
// time): further ones only spread the accesses over more of memory.  2 GiB
// read, Gram / combine, us, as many as fit (4-6 a CU) against two a CU: K=4
// fp32 371 / 569 -> 350 / 529, K=8 fp32 403 / 516 -> 365 / 496, K=10 fp32 377 /
// 491 -> 357 / 460, K=4 bf16 374 / 558 -> 357 / 552; K=2 bf16 374 / 705 -> 340
// / 675 with four, 432 / 782 with two.  A short pass (fewer than kLongPass
// whole parts for each of them) takes all that fit, and so does one of short
// buckets: it waits for latency at each, and where full and nearly empty chunks
// take turns a workgroup may be dealt only full ones, which further ones on its
// CU make up for.  Combine, all / two a CU, us: K=4 bf16, 0.7 GiB, buckets of
// 0.05 chunks 384 / 512, of 1.5 190 / 216, of 3 201 / 197; with one vector per
// row and step K=8 fp32, 2 GiB, buckets of 0.25 485 / 465, of 1.5 544 / 530, but
// 20,000 of 64 elements 125 / 143.
constexpr int kLongPass = 4;
constexpr int stream_wgs(int K, int R) {
  const int n = (16 + K * R / 2) / (K * R);
  return n < 2 ? 2 : n;
}
// The combine of eleven tasks and more, and of ten with bf16 rows and output, is
// fastest with one: two / one, 2 GiB in ten buckets, us, K=12 bf16 to fp32 532 /
// 502, K=14 fp32 to bf16 432 / 410, K=16 fp32 469 / 457, K=10 bf16 489 / 462.
// From bf16 to bf16, where an element costs K fp64 FMAs, only long buckets (32
// chunks) are: in 600 buckets K=12, 0.7 GiB, 178 / 201, K=16, 2 GiB, 498 / 500.
template <int K, int DT, int ODT>
constexpr bool kCombineAlone = K > 10 || (K == 10 && DT == BF16 && ODT == BF16);

inline int64_t stream_grid(const StreamArgs &a, int R, int parts, int wgs, int occ, int64_t cap) {
  const int64_t cus = device_cu_count(), few = cus * wgs;
  const int64_t chunks = a.N / gram_chunk_elems(a.K, a.dt), B = a.B;
  int64_t grid = cus * occ;
  if (grid > few && chunks * parts >= kLongPass * few && chunks >= (R > 1 ? 3 * B : B / 4)) grid = few;
  if (grid > cap) grid = cap;
  return grid < 1 ? 1 : grid;
}

// Resident workgroups of kThreads per CU for a kernel (at least 1).
template <typename Kern>
int occupancy(Kern kern) {
  int occ = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, kThreads, 0) != hipSuccess || occ < 1)
    occ = 1;
  return occ;
}

}  // namespace bkmoo
