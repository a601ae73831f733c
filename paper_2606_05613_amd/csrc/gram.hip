// Pass 1: per-bucket Gram matrices G_b[i][j] = <x_i, x_j> over the bucket.
//
// The bucket-level problems (Eq. shard-mgda, the local CAGrad problem and
// PCGrad's local conflict test, Section 3.2) depend on the local gradients
// only through these inner products, so this pass is the only one that
// needs all K rows at once.  It is HBM-bound: K*N*s bytes read, K(K+1)
// flops per element position, below the fp32 vector ridge point for fp32
// rows and for few tasks: there it uses plain fp32 FMAs (bf16 rows of many
// tasks: gram_mfma_kernel below).
//
// Design (gfx950): persistent workgroups of 4 wavefronts own contiguous
// runs of chunks.  Every thread issues K*R independent 128-bit
// non-temporal loads per iteration and accumulates all K(K+1)/2 products
// in fp32 registers over the chunk's iterations.  Lane sums are combined by
// a fixed xor butterfly across the wavefront, then in fp64 across the 4
// wavefronts through LDS in wave order, and land in a per-chunk slot.  The
// finalize adds a bucket's chunk slots in fp64 in an order fixed by the
// bucket's chunk count (in a bucket of many chunks groups of consecutive
// chunks first, then the groups); a resolve call adds them in
// the kernel that also solves the bucket's problem (solve.hip).  No atomics:
// the result is bitwise independent of the grid and of scheduling.
#include "chunk.h"
#include "gram_sum.h"
#include "schedule.h"

namespace bkmoo {

namespace {

template <int K, int DT, bool SELF>
__global__ __launch_bounds__(kThreads) void gram_partial_kernel(
    Rows<K> rows, const int64_t *__restrict__ offs, const int64_t *__restrict__ gcs, int B,
    int shift, ScheduleOut sched, double *__restrict__ partials) {
  constexpr int64_t C = gram_chunk_elems(K, DT);
  constexpr int P = pairs(K);
  __shared__ double red[kThreads / kWave][P];

  __shared__ int64_t lcs[SELF ? kSelfBuckets + 1 : 1];
  if constexpr (SELF) {
    if (!own_schedule<false>(offs, B, C, sum_direct(P), sched, lcs)) return;
  }
  const int64_t *cs = SELF ? lcs : gcs;
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

// The same partials of bf16 rows on the matrix cores, for kMfmaMinK tasks and
// more.  There the FMA kernel is bound by issue, not by memory: at K = 16 an
// element position costs 136 FMA and 16 conversions for 32 bytes, and its
// accumulators leave one wavefront a SIMD.  Here a 16x16x32 product X X^T
// takes 32 positions of 16 rows: lane l holds 16 bytes of row l % 16 (task l %
// 16 % K of slice l % 16 / K: 16 / K runs of positions side by side, of which
// the diagonal blocks count), the same register as left and as right operand,
// so which positions a lane holds does not matter as long as all rows agree.
// A wavefront reads a tile of 1 KiB of every row, lane after lane, and turns
// it through LDS (its own part: no barrier), with the next tile's loads in
// flight; read from memory in the operand's layout, 64 bytes of each row at a
// time, it reached 2.5-4 TB/s.  The tile's rows lie kRowPitch apart, so that
// eight lanes' 16-byte reads of eight rows fall on different banks.
//
// Products of bf16 are exact; an fp32 accumulator takes at most 256 of them
// and is then added to an fp64 one.  2 GiB in ten buckets, us, FMA / matrix:
// K=16 647 / 388, K=12 547 / 370, K=10 523 / 375, K=8 408 / 370, K=7 378 /
// 355; K=6 374 / 373 and K=5 354 / 388, where the FMA kernel is bound by
// memory.  Largest error relative to sqrt(G_ii G_jj) 1.5e-7 / 6e-9.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kMfmaMinK = 7;
constexpr int kRowPitch = kWave + 1;  // 16-byte vectors

template <int K, bool SELF>
__global__ __launch_bounds__(kThreads) void gram_mfma_kernel(Rows<K> rows, const int64_t *__restrict__ offs,
                                                             const int64_t *__restrict__ gcs, int B, int shift,
                                                             ScheduleOut sched, double *__restrict__ partials) {
  constexpr int64_t C = gram_chunk_elems(K, BF16);
  constexpr int P = pairs(K), V = vec_elems(BF16), S = 16 / K;
  constexpr int kWaves = kThreads / kWave, kStep = 4 * S;  // vectors of a row in a product
  constexpr int kSteps = kWave / kStep;                    // products in a tile (a vector of every row a lane)
  static_assert(K >= kMfmaMinK && kSteps * kStep == kWave, "one or two slices");
  __shared__ u32x4 tile[kWaves][K * kRowPitch];
  __shared__ double red[2][kWaves * S][P];

  __shared__ int64_t lcs[SELF ? kSelfBuckets + 1 : 1];
  if constexpr (SELF) {
    if (!own_schedule<false>(offs, B, C, sum_direct(P), sched, lcs)) return;
  }
  const int64_t *cs = SELF ? lcs : gcs;
  int64_t c, cend;
  my_chunks(cs[B], c, cend);
  if (c >= cend) return;
  int b = find_bucket(cs, B, c);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int row = lane & 15, g = lane / 16, slice = row / K, task = row - slice * K;
  const bool used = slice < S;
  u32x4 *own = tile[wave];
  const u32x4 *operand = own + (used ? task * kRowPitch + slice * 4 + g : 0);

  for (int parity = 0; c < cend; ++c, parity ^= 1) {
    while (cs[b + 1] <= c) ++b;
    const int64_t lo = offs[b] + (c - cs[b]) * C;
    const int64_t hi = lo + C < offs[b + 1] ? lo + C : offs[b + 1];
    const Split<V> sp(lo, hi, shift);
    double sum[4] = {0.0, 0.0, 0.0, 0.0};

    if (wave == 0 && sp.nh + sp.nt > 0) {  // the scalar head (group 0) and tail (group 1) in one product
      const uint16_t *mine = static_cast<const uint16_t *>(rows.p[0]);
#pragma unroll
      for (int i = 1; i < K; ++i) mine = task == i ? static_cast<const uint16_t *>(rows.p[i]) : mine;
      const int64_t at = g == 0 ? lo : sp.hi_a;
      const int n = slice == 0 ? (g == 0 ? sp.nh : g == 1 ? sp.nt : 0) : 0;
      uint16_t x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = e < n ? mine[at + e] : (uint16_t)0;
      const bf16x8 q = __builtin_bit_cast(bf16x8, x);
      const f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q, q, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] += (double)a[r];
    }
    u32x4 q[K];
    const auto load = [&](int v0) {
      const int v = v0 + lane;
      const bool in = v < sp.nv;
#pragma unroll
      for (int i = 0; i < K; ++i) {
        q[i] = u32x4{0u, 0u, 0u, 0u};
        if (in) q[i] = stream_load(static_cast<const uint16_t *>(rows.p[i]) + sp.lo_a, v);
      }
    };
    int v0 = wave * kWave;
    if (v0 < sp.nv) load(v0);
    for (; v0 < sp.nv; v0 += kWaves * kWave) {
#pragma unroll
      for (int i = 0; i < K; ++i) own[i * kRowPitch + lane] = q[i];
      if (v0 + kWaves * kWave < sp.nv) load(v0 + kWaves * kWave);
      // one wavefront's LDS accesses are executed in order: the compiler must
      // only keep them so
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      f32x4 a[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
      for (int u = 0; u < kSteps; ++u) {
        const bf16x8 x = __builtin_bit_cast(bf16x8, operand[u * kStep]);
        a[u & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, x, a[u & 1], 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] += (double)a[0][r] + (double)a[1][r];
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    // lane l holds entries (g * 4 + r, l % 16); the diagonal blocks' upper
    // triangles count
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = g * 4 + r - slice * K;
      if (used && i >= 0 && i <= task) red[parity][wave * S + slice][i * K - i * (i - 1) / 2 + task - i] = sum[r];
    }
    __syncthreads();
    if (tid < P) {
      double s = red[parity][0][tid];
#pragma unroll
      for (int w = 1; w < kWaves * S; ++w) s += red[parity][w][tid];
      partials[c * P + tid] = s;
    }
  }
}

// Finalize, level 1 (only buckets of sum_direct chunks and more): one workgroup
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

// Finalize, level 2: one workgroup per bucket adds the bucket's chunk slots or
// group sums and writes the symmetric K x K matrix (NaN everywhere when the
// offsets were rejected by the schedule).
template <int T>
__global__ __launch_bounds__(T) void gram_finalize_kernel(int K, const int64_t *__restrict__ cs,
                                                                    const double *__restrict__ partials,
                                                                    const uint32_t *__restrict__ err,
                                                                    double *__restrict__ gram) {
  __shared__ double red[kSumThreads];
  const int64_t b = blockIdx.x;
  const int P = K * (K + 1) / 2;
  double s = sum_bucket<T>(partials, cs, b, P, red);
  if ((int)threadIdx.x < P) {
    if (*err & kErrOffsets) s = __builtin_nan("");
    int i, j;
    pair_of((int)threadIdx.x, K, i, j);
    gram[(b * K + i) * K + j] = s;
    gram[(b * K + j) * K + i] = s;
  }
}

// Gram pass of one batch of buckets, by number of tasks and type.
template <int K, int DT, bool SELF>
constexpr auto gram_kernel() {
  if constexpr (DT == BF16 && K >= kMfmaMinK) return gram_mfma_kernel<K, SELF>;
  else return gram_partial_kernel<K, DT, SELF>;
}

template <int K, int DT, bool SELF>
hipError_t launch_gram_s(const StreamArgs &a, double *partials, hipStream_t s) {
  Rows<K> rows;
  for (int i = 0; i < K; ++i) rows.p[i] = a.rows[i];
  auto kern = gram_kernel<K, DT, SELF>();
  const int64_t C = gram_chunk_elems(K, DT);
  const int64_t cap = (a.N + C - 1) / C + a.B;
  static const int occ = occupancy(kern);
  int64_t grid = a.grid > 0 ? a.grid : stream_grid(a, gram_shape(K).R, 1, stream_wgs(K, gram_shape(K).R), occ, cap);
  if (grid > cap) grid = cap;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), 0, s, rows, a.offsets,
                     a.chunk_start, a.B, a.shift, ScheduleOut{a.N, a.chunk_start, a.group_start, a.part_start, a.err},
                     partials);
  return hipGetLastError();
}

template <int K, int DT>
hipError_t launch_gram_t(const StreamArgs &a, double *partials, hipStream_t s) {
  return a.scheduled ? launch_gram_s<K, DT, false>(a, partials, s) : launch_gram_s<K, DT, true>(a, partials, s);
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

hipError_t launch_gram_partials(const StreamArgs &a, double *partials, hipStream_t s) {
  hipError_t e = a.dt == F32 ? dispatch_gram<F32>(a, partials, s) : dispatch_gram<BF16>(a, partials, s);
  // the chunks that one bucket can have, and the groups of all that have them
  const int64_t chunks = (a.N + gram_chunk_elems(a.K, a.dt) - 1) / gram_chunk_elems(a.K, a.dt);
  const int64_t direct = sum_direct(pairs(a.K));
  if (e != hipSuccess || chunks < direct) return e;
  const int64_t groups = chunks / kFinalizeGroup + chunks / direct;
  const int64_t limit = (int64_t)device_cu_count() * 4;
  hipLaunchKernelGGL(gram_group_kernel, dim3((unsigned)(groups < limit ? groups : limit)), dim3(kSumThreads), 0, s,
                     pairs(a.K), a.B, a.chunk_start, a.group_start, partials);
  return hipGetLastError();
}

hipError_t launch_gram_finalize(const StreamArgs &a, const double *partials, double *gram, hipStream_t s) {
  const int T = sum_workgroup(a);
  hipLaunchKernelGGL(T == kWave ? gram_finalize_kernel<kWave> : gram_finalize_kernel<kSumThreads>, dim3((unsigned)a.B),
                     dim3((unsigned)T), 0, s, a.K, a.chunk_start, partials, a.err, gram);
  return hipGetLastError();
}

}  // namespace bkmoo
