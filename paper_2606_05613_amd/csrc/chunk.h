// One workgroup's work on one chunk of a bucket: its Gram products and its
// part of the update.  Shared by the two streaming passes and by the tiled
// form of the refill kernel.  Vectors start where `shift` puts them, on
// 16-byte boundaries of the rows where these share a phase; rows at other
// phases are read with 128-bit loads all the same.  Read element by element,
// as such rows were before, K=3 bf16, 30M elements in odd-length rows, took
// 149 us a step (now 100), K=8 bf16 of 90M 890 us (366).
#pragma once

#include "combine_impl.h"

namespace bkmoo {

namespace {

// acc[p] += the products of elements [lo, hi), at most U * R vectors a thread.
template <int K, int DT>
__device__ __forceinline__ void gram_chunk(const Rows<K> &rows, int64_t lo, int64_t hi, int shift,
                                           float (&acc)[pairs(K)]) {
  constexpr int V = vec_elems(DT), EB = elem_bytes(DT);
  constexpr int R = gram_shape(K).R, U = gram_shape(K).U;
  const int tid = threadIdx.x;
  const Split<V> sp(lo, hi, shift);
  if (tid < sp.nh + sp.nt) {
    const int64_t n = tid < sp.nh ? lo + tid : sp.hi_a + (tid - sp.nh);
    float x[K];
#pragma unroll
    for (int i = 0; i < K; ++i) x[i] = load_elem<DT>(rows.p[i], n);
    accumulate<K>(acc, x);
  }
#pragma unroll 2
  for (int u = 0; u < U; ++u) {
    const int vb = u * kThreads * R + tid;
    u32x4 buf[R][K];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int v = vb + r * kThreads;
      if (v < sp.nv) {
#pragma unroll
        for (int i = 0; i < K; ++i)
          buf[r][i] = stream_load(static_cast<const char *>(rows.p[i]) + sp.lo_a * EB, v);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int v = vb + r * kThreads;
      if (v < sp.nv) {
        float x[K][V];
#pragma unroll
        for (int i = 0; i < K; ++i) decode<DT>(buf[r][i], x[i]);
#pragma unroll
        for (int e = 0; e < V; ++e) {
          float xe[K];
#pragma unroll
          for (int i = 0; i < K; ++i) xe[i] = x[i][e];
          accumulate<K>(acc, xe);
        }
      }
    }
  }
}

// Lane sums of a workgroup: a fixed xor butterfly across the wavefront
// (fp32), the wavefronts' sums into red[wave][p] (fp64).
template <int P>
__device__ __forceinline__ void reduce_lanes(float (&acc)[P], double (*red)[P]) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) {
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] += __shfl_xor(acc[p], off, kWave);
  }
  if (lane == 0) {
#pragma unroll
    for (int p = 0; p < P; ++p) red[wave][p] = (double)acc[p];
  }
}

// The update of elements [lo, hi), at most U * R vectors a thread.  With many
// tasks (kCombineAlone) a vector's loads and its store share one condition: as
// two the compiler copies registers between them, for which the loads of the
// next step wait for the store (K=14 fp32 to bf16, 2 GiB, one workgroup a CU,
// 454 / 410 us).  With fewer, several workgroups hide that wait, and the loads of
// all vectors of a step go first.
template <int K, int DT, int ODT, int R, int U>
__device__ __forceinline__ void combine_chunk(const Rows<K> &rows, int64_t lo, int64_t hi, int shift, const float *w,
                                              void *out) {
  constexpr int V = vec_elems(DT), EB = elem_bytes(DT);
  const int tid = threadIdx.x;
  const Split<V> sp(lo, hi, shift);
  if (tid < sp.nh + sp.nt) {
    const int64_t n = tid < sp.nh ? lo + tid : sp.hi_a + (tid - sp.nh);
    float x[K];
#pragma unroll
    for (int i = 0; i < K; ++i) x[i] = load_elem<DT>(rows.p[i], n);
    store_elem<ODT>(out, n, wsum<K, ODT>(w, x));
  }
  const auto load = [&](int v, u32x4 (&q)[K]) {
#pragma unroll
    for (int i = 0; i < K; ++i) q[i] = stream_load(static_cast<const char *>(rows.p[i]) + sp.lo_a * EB, v);
  };
  const auto put = [&](int v, const u32x4 (&q)[K]) {
    float x[K][V];
#pragma unroll
    for (int i = 0; i < K; ++i) decode<DT>(q[i], x[i]);
    float y[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      float xe[K];
#pragma unroll
      for (int i = 0; i < K; ++i) xe[i] = x[i][e];
      y[e] = wsum<K, ODT>(w, xe);
    }
    store_vec<ODT, V>(out, sp.lo_a + (int64_t)v * V, y);
  };
#pragma unroll 2
  for (int u = 0; u < U; ++u) {
    const int vb = u * kThreads * R + tid;
    if constexpr (kCombineAlone<K, DT, ODT>) {
      static_assert(R == 1, "one vector per row and step");
      if (vb < sp.nv) {
        u32x4 buf[K];
        load(vb, buf);
        put(vb, buf);
      }
    } else {
      u32x4 buf[R][K];
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (vb + r * kThreads < sp.nv) load(vb + r * kThreads, buf[r]);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (vb + r * kThreads < sp.nv) put(vb + r * kThreads, buf[r]);
    }
  }
}

}  // namespace

}  // namespace bkmoo
