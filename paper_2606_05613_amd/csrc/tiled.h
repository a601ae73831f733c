// The tiled form of the refill kernel, for buckets of very
// different sizes: every bucket is cut into the Gram pass's chunks, chunk c
// goes to data workgroup c % GD, and each chunk is read twice.
//
// Bound by memory like the two passes (2K reads and a write an element);
// GPT-2 with a bucket per tensor, K=4 bf16 in, fp32 out, 124M elements: 1.70
// ms pipelined (see PipePlan), 0.51 ms tiled.
//
// The chunks are taken in windows of whole buckets, at least GD chunks (one a
// workgroup) each: a data workgroup reads its chunks of window w + 1 (partial
// Gram matrices to the chunks' slots, one arrival per bucket it has finished)
// before it combines those of window w, so a bucket's sum and solve run while
// the next window is read.  Solver j takes buckets j, j + nsolv, ...: it waits
// for as many arrivals as the bucket has chunks, adds their slots in a fixed
// order, solves on one wavefront and publishes the weights in kFlagCopies
// records (coop_common.h), of which data workgroup d polls copy d %
// kFlagCopies.  Every wait is bounded: a solver whose wait runs out publishes
// NaN, a data workgroup whose wait runs out combines with NaN, both set the
// error word's timeout bit.
//
// No cycle of waits: the weights of window w need every workgroup's arrivals
// up to window w, and a workgroup arrives for window w + 1 before its first
// wait for window w; solvers wait only for arrivals, bucket by bucket upwards.
// The Gram sums are made chunk by chunk, with the Gram pass's chunks, so they do
// not depend on the grid.  They are not that pass's bits: the solver adds a
// bucket's slots in an order of its own, and bf16 rows of seven tasks and more go
// through FMAs here and through the matrix cores there.
#pragma once

#include "chunk.h"
#include "coop_common.h"
#include "solve_impl.h"

namespace bkmoo {

namespace {

struct TileArgs {
  const int64_t *offs, *cs;  // [B+1] bucket offsets, chunk prefix
  int B, shift, method, iters;
  double c;
  const int8_t *order;
  double *gram;
  float *weights;
  double *aux;
  void *out;
  double *partials;  // [chunks][P]
  uint32_t *arrive;  // [B] at stride kSyncStride, zero at launch
  uint32_t *recs;    // [kFlagCopies][B] at stride kSyncStride, zero at launch
  uint32_t *err;
  uint32_t spin_limit;
  int nsolv;  // workgroups 0 .. nsolv-1 solve, the others hold data
};

template <int K, int DT, int ODT>
struct Tiled {
  static constexpr int P = pairs(K);
  static constexpr int T = kThreads;
  static constexpr int64_t C = gram_chunk_elems(K, DT);
  static constexpr int NG = T / P;   // solver threads per Gram entry
  static constexpr int RB = 16;      // slot loads each keeps in flight
  static_assert(P <= kWave, "one wavefront stores a chunk's partial Gram (and publishes it)");

  struct Smem {
    double red[2][T / kWave][P];
    double sum[P][NG];
    Shared S;
    float wsh[2][K];
    int ok;
  };

  // Bucket of chunk c, which lies in buckets [lo, hi).
  static __device__ __forceinline__ int bucket_of(const int64_t *cs, int lo, int hi, int64_t c) {
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (cs[mid] <= c) lo = mid; else hi = mid;
    }
    return lo;
  }

  static __device__ __forceinline__ void arrived(const TileArgs &a, int b, uint32_t chunks) {
    if (threadIdx.x == 0) {
      publish_point();  // the chunks' slots (stored by this wavefront) before the arrival
      __hip_atomic_fetch_add(&a.arrive[(int64_t)b * kSyncStride], chunks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // This workgroup's chunks of buckets [wb, we): partial Gram matrices.
  static __device__ __forceinline__ void read(const Rows<K> &rows, const TileArgs &a, Smem &sm, int wb, int we, int64_t first, int GD,
                              int &parity) {
    const int t = threadIdx.x;
    const int64_t end = a.cs[we];
    int b = -1;
    uint32_t held = 0;  // chunks of bucket b not yet announced
    for (int64_t c = first; c < end; c += GD) {
      const int bc = bucket_of(a.cs, b < 0 ? wb : b, we, c);
      if (bc != b) {
        if (held) arrived(a, b, held);
        b = bc;
        held = 0;
      }
      const int64_t lo = a.offs[b] + (c - a.cs[b]) * C, end_b = a.offs[b + 1];
      float acc[P];
#pragma unroll
      for (int p = 0; p < P; ++p) acc[p] = 0.0f;
      gram_chunk<K, DT>(rows, lo, lo + C < end_b ? lo + C : end_b, a.shift, acc);
      double(*red)[P] = sm.red[parity];
      parity ^= 1;
      reduce_lanes<P>(acc, red);
      __syncthreads();
      if (t < P) {
        double s = red[0][t];
#pragma unroll
        for (int q = 1; q < T / kWave; ++q) s += red[q][t];
        store_agent(&a.partials[c * P + t], s);
      }
      ++held;
    }
    if (held) arrived(a, b, held);
  }

  // This workgroup's chunks of buckets [wb, we): the update.
  static __device__ __forceinline__ void combine(const Rows<K> &rows, const TileArgs &a, Smem &sm, int wb, int we, int64_t first,
                                 int d, int GD, int &parity) {
    const int t = threadIdx.x;
    const int64_t end = a.cs[we];
    int b = -1;
    float wv[K];
    for (int64_t c = first; c < end; c += GD) {
      const int bc = bucket_of(a.cs, b < 0 ? wb : b, we, c);
      if (bc != b) {
        b = bc;
        float *wsh = sm.wsh[parity];
        parity ^= 1;
        if (t == 0) {
          uint32_t x[K];
          const bool ok = poll_record<K, 16>(a.recs + ((int64_t)(d % kFlagCopies) * a.B + b) * kSyncStride, x, a.err,
                                             a.spin_limit);
#pragma unroll
          for (int i = 0; i < K; ++i) wsh[i] = ok ? word_weight(x[i]) : __builtin_nanf("");
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < K; ++i) wv[i] = wsh[i];
      }
      const int64_t lo = a.offs[b] + (c - a.cs[b]) * C, end_b = a.offs[b + 1];
      combine_chunk<K, DT, ODT, combine_shape(K).R, combine_shape(K).U * kCombineParts>(
          rows, lo, lo + C < end_b ? lo + C : end_b, a.shift, wv, a.out);
    }
  }

  static __device__ __forceinline__ void data(const Rows<K> &rows, const TileArgs &a, Smem &sm, int d, int GD) {
    int rp = 0, cp = 0;          // parity of the LDS copies
    int wb = 0, pb = 0, pe = 0;  // first bucket of the window to read, buckets of the one before it
    int64_t pfirst = 0;
    for (;;) {
      // the window: the fewest whole buckets with GD chunks, or all that are left
      int we = wb;
      int64_t first = 0;
      if (wb < a.B) {
        const int64_t c0 = a.cs[wb];
        int hi = a.B;  // the smallest bucket end in (wb, B] with GD chunks, else B
        for (int lo = wb; hi - lo > 1;) {
          const int mid = (lo + hi) >> 1;
          if (a.cs[mid] - c0 >= GD) hi = mid; else lo = mid;
        }
        we = hi;
        const int64_t m = c0 % GD;
        first = c0 + (d >= m ? d - m : d + GD - m);  // this workgroup's first chunk (c % GD == d) from c0 on
        read(rows, a, sm, wb, we, first, GD, rp);
      }
      if (pe > pb) combine(rows, a, sm, pb, pe, pfirst, d, GD, cp);
      if (we == wb) return;
      pb = wb;
      pe = we;
      pfirst = first;
      wb = we;
    }
  }

  static __device__ __forceinline__ void solve(const TileArgs &a, Smem &sm, int j) {
    const int t = threadIdx.x;
    __builtin_amdgcn_s_setprio(3);
    for (int b = j; b < a.B; b += a.nsolv) {
      const int64_t c0 = a.cs[b], n = a.cs[b + 1] - c0;
      if (t == 0) {
        uint32_t spins = 0;
        bool ok = true;
        while (load_agent(&a.arrive[(int64_t)b * kSyncStride]) < (uint32_t)n) {
          __builtin_amdgcn_s_sleep(1);
          if (++spins >= a.spin_limit) {
            note_timeout(a.err);
            ok = false;
            break;
          }
        }
        observe_point();  // the chunks' slots after the arrivals (loaded after the barrier)
        sm.ok = ok ? 1 : 0;
        sm.S.bad = ok ? 0 : 1;
      }
      __syncthreads();
      if (t < P * NG) {
        const int p = t % P, g = t / P;
        const double *slot = a.partials + c0 * P + p;
        double v = 0.0;
        for (int64_t i = g; i < n; i += (int64_t)RB * NG) {
          double x[RB];
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            const int64_t s = i + (int64_t)u * NG;
            x[u] = s < n ? load_agent(slot + s * P) : 0.0;
          }
#pragma unroll
          for (int u = 0; u < RB; ++u) v += x[u];
        }
        sm.sum[p][g] = v;
      }
      __syncthreads();
      if (t < P) {
        double v = 0.0;
        for (int g = 0; g < NG; ++g) v += sm.sum[t][g];
        if (!sm.ok) v = __builtin_nan("");  // some slots may be missing
        int i = 0, rem = t;
        while (rem >= K - i) {
          rem -= K - i;
          ++i;
        }
        const int jj = i + rem;
        sm.S.G[i * K + jj] = v;
        sm.S.G[jj * K + i] = v;
        if (!__builtin_isfinite(v)) sm.S.bad = 1;
      }
      __syncthreads();
      if (t < kWave) {
        double wt = 0.0, ax = 0.0;
        if (a.method == PCGRAD || sm.S.bad) {
          solver_run<WaveSync>(sm.S, K, a.method, a.iters, a.c, a.order, b, t, &wt, &ax);
        } else if (a.method == MGDA) {
          wt = ax = lane_solve_mgda<K>(sm.S.G, a.iters, t);
        } else if (a.method == CAGRAD) {
          lane_solve_cagrad<K>(sm.S.G, a.iters, a.c, t, &wt, &ax);
        } else {
          wt = ax = 1.0 / (double)K;
        }
        // lane i < K holds task i's weight; lanes r < kFlagCopies store record r
        float wk[K];
#pragma unroll
        for (int i = 0; i < K; ++i) wk[i] = (float)__shfl(wt, i, kWave);
        publish_point();  // nothing of this bucket in flight when its weights appear
        if (t < kFlagCopies) {
          uint32_t *rec = a.recs + ((int64_t)t * a.B + b) * kSyncStride;
#pragma unroll
          for (int i = 0; i < K; ++i) store_agent(rec + i, weight_word(wk[i]));
        }
        if (t < K) {
          a.weights[(int64_t)b * K + t] = (float)wt;
          if (a.aux) a.aux[(int64_t)b * K + t] = ax;
        }
      }
      for (int e = t; e < K * K; e += T) a.gram[(int64_t)b * K * K + e] = sm.S.G[e];
      __syncthreads();
    }
  }

  static __device__ __forceinline__ void run(const Rows<K> &rows, const TileArgs &a, Smem &sm) {
    const int GD = (int)gridDim.x - a.nsolv, d = (int)blockIdx.x - a.nsolv;
    if (d < 0) solve(a, sm, (int)blockIdx.x);
    else data(rows, a, sm, d, GD);
  }
};

}  // namespace

}  // namespace bkmoo
