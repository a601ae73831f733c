// Exact solvers for the per-bucket problems, by support enumeration: the
// minimum-norm point of the simplex hull of the task gradients (Eq. mgda /
// Eq. shard-mgda over the simplex) and the minimiser of the CAGrad dual
// F(w) = b^T w + r ||g_w|| over the simplex (the local problem of Eq.
// cagrad through its dual), both from the bucket's Gram matrix alone.
//
// K <= 10, one wavefront per bucket, fp64, in two kernels: the first screens
// the supports, solves the one or two that can be the answer and leaves a
// bucket that it is not sure of to the second, which looks at every support
// (most often of no bucket: it then only reads one word each).  Both apply the
// rules below with the same arithmetic, so the split does not show in the
// results.
//
// The 2^K - 1 supports S are
// ranked in the order "by support size, then lexicographically", which fixes
// every tie-break, and dealt to the 64 lanes in rank order, so the lanes of
// a wavefront mostly hold supports of one size.  Each lane builds its
// support's small linear system in registers (a solver instantiated per
// support size, fully unrolled, row exchanges done by selects so every index
// is static) and solves it by Gaussian elimination with partial pivoting; a
// support whose system has an exactly zero pivot is skipped:
//
// MGDA.  On S the stationarity conditions G_SS a_S = mu 1, 1^T a_S = 1 form
// a bordered (|S|+1)-square system (non-singular exactly when the g_t, t in
// S, are affinely independent, which the smallest optimal support is).  A
// solution is kept if a_S >= -1e-10 and |sum a_S - 1| <= 1e-9; clipped at 0
// and renormalised it must satisfy (G a)_t >= a^T G a - 1e-9 for every t
// (the minimum-norm property); G is first divided by its largest diagonal
// entry.  Scanning the kept candidates in rank order, a later one replaces
// the current choice only if its a^T G a is smaller by more than 1e-12.  If
// none is kept (numerically degenerate input), 5000 Frank-Wolfe iterations
// of the iterative solver stand in.
//
// CAGrad.  Candidates are the K vertices and, when r > 0, for every S with
// |S| >= 2 the points v_S = G_SS^{-1} (lam 1 - b_S) / r for the two roots
// lam of v_S^T G_SS v_S = 1 (a quadratic in lam), kept if v_S >= -1e-12 and
// sum v_S > 0, clipped at 0 and normalised onto the simplex.  The candidate
// of least F wins, the first in rank order (vertices first, smaller root
// first) on exact ties.
#include "solve_impl.h"

namespace bkmoo {

namespace {

// Rank -> support (bit t = task t) tables for every K, built at compile
// time: the non-empty subsets of {0..K-1} ordered by size, then
// lexicographically (each size's combinations from {0..s-1} by the usual
// successor: raise the last index that can still rise, reset the rest
// right after it).  A lookup replaces unranking through binomial sums,
// whose integer divisions took half of the kernel's time (K=10, 6,564
// buckets: 2.45 -> 1.27 ms, identical results).
struct SupportTables {
  uint16_t m[kExactMaxK + 1][(1 << kExactMaxK) - 1];
};
constexpr SupportTables make_support_tables() {
  SupportTables T{};
  for (int K = 1; K <= kExactMaxK; ++K) {
    int r = 0;
    for (int s = 1; s <= K; ++s) {
      int c[kExactMaxK] = {};
      for (int i = 0; i < s; ++i) c[i] = i;
      for (;;) {
        uint16_t m = 0;
        for (int i = 0; i < s; ++i) m = (uint16_t)(m | (1u << c[i]));
        T.m[K][r++] = m;
        int i = s - 1;
        while (i >= 0 && c[i] == K - s + i) --i;
        if (i < 0) break;
        ++c[i];
        for (int j = i + 1; j < s; ++j) c[j] = c[j - 1] + 1;
      }
    }
  }
  return T;
}
__constant__ SupportTables kSupportTables = make_support_tables();

// Gaussian elimination with partial pivoting (the first entry of largest
// magnitude) on the N x (N + M) augmented matrix A, fully unrolled.  False if
// a pivot is exactly zero; otherwise the solutions overwrite columns N..N+M-1.
template <int N, int M>
__device__ __forceinline__ bool ge_solve(double (&A)[N][N + M]) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    double pv = fabs(A[k][k]);
    int p = k;
#pragma unroll
    for (int r = k + 1; r < N; ++r) {
      const double v = fabs(A[r][k]);
      const bool gt = v > pv;
      pv = gt ? v : pv;
      p = gt ? r : p;
    }
    ok = ok && pv != 0.0;
#pragma unroll
    for (int r = k + 1; r < N; ++r) {
      const bool sw = p == r;
#pragma unroll
      for (int c = k; c < N + M; ++c) {
        const double x = A[k][c], y = A[r][c];
        A[k][c] = sw ? y : x;
        A[r][c] = sw ? x : y;
      }
    }
    const double piv = pv != 0.0 ? A[k][k] : 1.0;
#pragma unroll
    for (int r = k + 1; r < N; ++r) {
      const double f = A[r][k] / piv;
#pragma unroll
      for (int c = k + 1; c < N + M; ++c) A[r][c] -= f * A[k][c];
      A[r][k] = 0.0;
    }
  }
#pragma unroll
  for (int j = N; j < N + M; ++j)
#pragma unroll
    for (int r = N - 1; r >= 0; --r) {
      double s = A[r][j];
#pragma unroll
      for (int c = r + 1; c < N; ++c) s -= A[r][c] * A[c][j];
      A[r][j] = s / (A[r][r] != 0.0 ? A[r][r] : 1.0);
    }
  return ok;
}

// Tasks of support m in increasing order.
template <int S>
__device__ __forceinline__ void support_tasks(uint32_t m, int (&idx)[S]) {
#pragma unroll
  for (int u = 0; u < S; ++u) {
    idx[u] = __builtin_ctz(m);
    m &= m - 1u;
  }
}

// MGDA on a support of S tasks of the normalised Gram Gn: solves the
// bordered system and runs the feasibility and minimum-norm checks.  On
// success a[0..S) holds the clipped, renormalised weights of the support's
// tasks in increasing task order and *q = a^T Gn a.
template <int S>
__device__ bool mgda_support(const double *Gn, int K, uint32_t m, double (&a)[S], double *q) {
  int idx[S];
  support_tasks<S>(m, idx);
  double A[S + 1][S + 2];
#pragma unroll
  for (int u = 0; u < S; ++u) {
#pragma unroll
    for (int v = 0; v < S; ++v) A[u][v] = Gn[idx[u] * K + idx[v]];
    A[u][S] = 1.0;
    A[u][S + 1] = 0.0;
  }
#pragma unroll
  for (int v = 0; v < S; ++v) A[S][v] = 1.0;
  A[S][S] = 0.0;
  A[S][S + 1] = 1.0;
  if (!ge_solve<S + 1, 1>(A)) return false;
  double amin = S < K ? 0.0 : A[0][S + 1], sum = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    amin = A[u][S + 1] < amin ? A[u][S + 1] : amin;
    sum += A[u][S + 1];
  }
  if (!(amin >= -1e-10) || !(fabs(sum - 1.0) <= 1e-9)) return false;
  double csum = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    a[u] = A[u][S + 1] > 0.0 ? A[u][S + 1] : 0.0;
    csum += a[u];
  }
#pragma unroll
  for (int u = 0; u < S; ++u) a[u] = a[u] / csum;
  // (Gn a)_t over every task, a^T Gn a, and the minimum-norm check
  double qq = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    double g = 0.0;
#pragma unroll
    for (int v = 0; v < S; ++v) g += Gn[idx[u] * K + idx[v]] * a[v];
    qq += a[u] * g;
  }
  for (int t = 0; t < K; ++t) {
    double g = 0.0;
#pragma unroll
    for (int v = 0; v < S; ++v) g += Gn[t * K + idx[v]] * a[v];
    if (!(g >= qq - 1e-9)) return false;
  }
  *q = qq;
  return true;
}

// CAGrad candidate `root` (0: smaller lam, 1: larger) on a support of S >= 2
// tasks: on success w[0..S) holds the simplex point on the support's tasks
// and *F its dual objective.
template <int S>
__device__ bool cagrad_support(const double *G, const double *bvec, double r, int K, uint32_t m,
                               int root, double (&w)[S], double *F) {
  int idx[S];
  support_tasks<S>(m, idx);
  double A[S][S + 2];  // [G_SS | 1 | b_S]
#pragma unroll
  for (int u = 0; u < S; ++u) {
#pragma unroll
    for (int v = 0; v < S; ++v) A[u][v] = G[idx[u] * K + idx[v]];
    A[u][S] = 1.0;
    A[u][S + 1] = bvec[idx[u]];
  }
  if (!ge_solve<S, 2>(A)) return false;
  double qa = 0.0, h1b = 0.0, hbb = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    qa += A[u][S];
    h1b += A[u][S] * bvec[idx[u]];
    hbb += bvec[idx[u]] * A[u][S + 1];
  }
  const double qb = -2.0 * h1b, qc = hbb - r * r;
  const double disc = qb * qb - 4.0 * qa * qc;
  if (!(qa > 0.0) || !(disc >= 0.0)) return false;
  const double sq = sqrt(disc);
  const double lam = root == 0 ? (-qb - sq) / (2.0 * qa) : (-qb + sq) / (2.0 * qa);
  double vmin = 0.0, vsum = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const double v = (lam * A[u][S] - A[u][S + 1]) / r;
    w[u] = v;
    vmin = u == 0 || v < vmin ? v : vmin;
    vsum += v;
  }
  if (!(vmin >= -1e-12) || !(vsum > 0.0)) return false;
  double csum = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    w[u] = w[u] > 0.0 ? w[u] : 0.0;
    csum += w[u];
  }
  double bw = 0.0, q = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) w[u] = w[u] / csum;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    bw += bvec[idx[u]] * w[u];
    double g = 0.0;
#pragma unroll
    for (int v = 0; v < S; ++v) g += w[v] * G[idx[v] * K + idx[u]];
    q += g * w[u];
  }
  const double f = bw + r * sqrt(q > 0.0 ? q : 0.0);
  if (!__builtin_isfinite(f)) return false;
  *F = f;
  return true;
}

// Size dispatch: run the support-size instantiation for |m| and, if `dst`
// is given, scatter its point onto the K tasks.
__device__ bool mgda_any(const double *Gn, int K, uint32_t m, double *q, double *dst) {
  switch (__builtin_popcount(m)) {
#define BKMOO_MGDA_CASE(n)                                                 \
  case n: {                                                                \
    double a[n];                                                           \
    if (!mgda_support<n>(Gn, K, m, a, q)) return false;                    \
    if (dst) {                                                             \
      int idx[n];                                                          \
      support_tasks<n>(m, idx);                                            \
      for (int i = 0; i < K; ++i) dst[i] = 0.0;                            \
      _Pragma("unroll") for (int u = 0; u < n; ++u) dst[idx[u]] = a[u];    \
    }                                                                      \
    return true;                                                           \
  }
    BKMOO_MGDA_CASE(1) BKMOO_MGDA_CASE(2) BKMOO_MGDA_CASE(3) BKMOO_MGDA_CASE(4) BKMOO_MGDA_CASE(5)
    BKMOO_MGDA_CASE(6) BKMOO_MGDA_CASE(7) BKMOO_MGDA_CASE(8) BKMOO_MGDA_CASE(9) BKMOO_MGDA_CASE(10)
#undef BKMOO_MGDA_CASE
    default: return false;
  }
}

__device__ bool cagrad_any(const double *G, const double *bvec, double r, int K, uint32_t m, int root,
                           double *F, double *dst) {
  switch (__builtin_popcount(m)) {
#define BKMOO_CAGRAD_CASE(n)                                                   \
  case n: {                                                                    \
    double w[n];                                                               \
    if (!cagrad_support<n>(G, bvec, r, K, m, root, w, F)) return false;        \
    if (dst) {                                                                 \
      int idx[n];                                                              \
      support_tasks<n>(m, idx);                                                \
      for (int i = 0; i < K; ++i) dst[i] = 0.0;                                \
      _Pragma("unroll") for (int u = 0; u < n; ++u) dst[idx[u]] = w[u];        \
    }                                                                          \
    return true;                                                               \
  }
    BKMOO_CAGRAD_CASE(2) BKMOO_CAGRAD_CASE(3) BKMOO_CAGRAD_CASE(4) BKMOO_CAGRAD_CASE(5)
    BKMOO_CAGRAD_CASE(6) BKMOO_CAGRAD_CASE(7) BKMOO_CAGRAD_CASE(8) BKMOO_CAGRAD_CASE(9)
    BKMOO_CAGRAD_CASE(10)
#undef BKMOO_CAGRAD_CASE
    default: return false;
  }
}

// (F, slot) is lexicographically smaller than (G, other).
__device__ __forceinline__ bool before(double f, int slot, double g, int other) {
  return f < g || (f == g && slot < other);
}

// ---- the screen -----------------------------------------------------------
// Solving every support's system from scratch is bound by fp64 issue (about
// 3,500 instructions for ten tasks, most of them the selects of the row
// exchanges, one wavefront a SIMD for its registers; 1,023 supports a bucket:
// K=10, 6,564 buckets, MGDA 1.19 ms, CAGrad 1.13), though all but one of them
// fail the answer's conditions by far.  With the screen 0.08 and 0.20 ms, K=8
// 0.41 -> 0.05, K=4 0.09 -> 0.025; where every bucket is left to the second
// kernel (K=10, a duplicated task in each) 1.14 -> 1.16, K=3 0.054 -> 0.061.  The screen finds
// that out with one symmetric sweep per support: sweeping task k into the
// tableau (D G D, D = diag(G_ii^-1/2)) extends the support by k in 55
// multiply-adds, sweeping it again takes it out, so lane l starts from the
// support given by its bits and walks the 2^(K-6) supports of the other
// tasks in Gray-code order.  With h = the swept right-hand side D 1, h_i (i in
// S) is the solution of G_SS y = 1 (y_i = d_i h_i) and h_t (t not in S) the
// residual 1 - G_tS y (times d_t): S is the minimum-norm support exactly if
// h_i >= 0 on S and h_t <= 0 off it.  For CAGrad, with e = the swept D b, the
// same signs are those of u = lam h - e for a root lam of u^T G u = r^2
// (u_i >= 0: the point is in the simplex; u_t <= 0: no other task's gradient
// entry is below lam), so one test serves both.
//
// A support is dropped only if some sign is wrong by more than kScreenTol of
// the entries' scale, above the tolerances under which the rules would still
// keep it.  That this is above the rounding of the sweeps as well, where the
// pivots (the squared distance of task k from the span of those before it,
// relative to its norm) stay above kScreenPivot, is measured and not a bound,
// as chains of nearly dependent tasks have condition numbers up to 1e12 with
// such pivots: on 20,000 buckets each of such chains, of triangular factors with
// equal off-diagonal entries, of noise on a low rank, of norms over eight
// decades and of near ties, every K and both methods, the results are the second
// kernel's, bit for bit.  One or two supports left are solved here;
// anything else (more, none, none of them kept, small pivots, a zero or
// non-finite diagonal, r = 0) leaves a mark in the bucket's first weight, a
// signalling NaN, which no conversion produces.
constexpr double kScreenTol = 1e-6, kScreenPivot = 1e-6;
constexpr uint32_t kUnsolved = 0x7f800001u;

template <int K, bool CAGRAD>
struct Tableau {
  static constexpr int LB = K < 6 ? K : 6;  // tasks chosen by the lane's bits
  double T[K][K];                           // upper triangle
  double h[K], e[K];

  __device__ __forceinline__ double &at(int i, int j) { return i <= j ? T[i][j] : T[j][i]; }

  // Sweep task k (in: sign = 1, out: -1) where `on`; true if the pivot is safe.
  __device__ __forceinline__ bool sweep(int k, bool on, double sign) {
    const double d = T[k][k];
    const bool safe = sign < 0.0 || d > kScreenPivot;
    const double inv = on ? 1.0 / d : 0.0;
    double f[K];
#pragma unroll
    for (int i = 0; i < K; ++i) f[i] = i == k ? 0.0 : at(i, k) * inv;
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
      for (int j = i; j < K; ++j)
        if (i != k && j != k) T[i][j] = __builtin_fma(-f[i], at(j, k), T[i][j]);
    const double hk = h[k], ek = CAGRAD ? e[k] : 0.0;
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (i != k) {
        h[i] = __builtin_fma(-f[i], hk, h[i]);
        if constexpr (CAGRAD) e[i] = __builtin_fma(-f[i], ek, e[i]);
        at(i, k) = on ? sign * f[i] : at(i, k);
      }
    T[k][k] = on ? -inv : d;
    h[k] = on ? sign * hk * inv : hk;
    if constexpr (CAGRAD) e[k] = on ? sign * ek * inv : ek;
    return !on || safe;
  }
};

// No u_i of the wrong sign for support m (u_i >= 0 in it, <= 0 off it) by more
// than c0 + c1 sum |u_i|.
template <int K>
__device__ __forceinline__ bool signs_fit(const double (&u)[K], uint32_t m, double c0, double c1) {
  double least = 0.0, sum = 0.0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const double s = (m >> i) & 1u ? u[i] : -u[i];
    least = s < least ? s : least;
    sum += fabs(u[i]);
  }
  return !(least < -(c0 + c1 * sum));  // (a NaN fits)
}

// Whether support a precedes b in rank order (by size, then lexicographically:
// the lowest task they differ in belongs to the first).
__device__ __forceinline__ bool ranks_before(uint32_t a, uint32_t b) {
  const int na = __builtin_popcount(a), nb = __builtin_popcount(b);
  if (na != nb) return na < nb;
  const uint32_t diff = a ^ b;
  return (a & (diff & (0u - diff))) != 0u;
}

// Gaussian elimination with the rows on lanes 0 .. n-1 (A[c], c < NM, and the
// right-hand sides z[.] in the lane's registers, n <= NM uniform): pivots, row
// exchanges and arithmetic are ge_solve's, element for element.  On success
// every lane holds the solutions in x[.][0 .. n-1].
template <int NM, int M>
__device__ __forceinline__ bool lane_ge_solve(double (&A)[NM], double (&z)[M], int n, int t, double (&x)[M][NM]) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < NM; ++k) {
    if (k < n) {
      double v = t >= k && t < n ? -fabs(A[k]) : 1.0;  // least = largest magnitude, lowest row first
      int p = t;
      argmin_step<kDppXor1>(v, p);
      argmin_step<kDppXor2>(v, p);
      argmin_step<kDppRor4>(v, p);
      argmin_step<kDppRor8>(v, p);
      p = __builtin_amdgcn_readfirstlane(p);
      const bool zero = lane_f64(v, 0) == 0.0;
      ok = ok && !zero;
      if (p != k) {
#pragma unroll
        for (int c = k; c < NM; ++c) {
          const double a = lane_f64(A[c], k), b = lane_f64(A[c], p);
          A[c] = t == k ? b : t == p ? a : A[c];
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
          const double a = lane_f64(z[j], k), b = lane_f64(z[j], p);
          z[j] = t == k ? b : t == p ? a : z[j];
        }
      }
      const double f = A[k] / (zero ? 1.0 : lane_f64(A[k], k));
#pragma unroll
      for (int c = k + 1; c < NM; ++c) {
        const double y = f * lane_f64(A[c], k);
        A[c] = t > k ? A[c] - y : A[c];
      }
#pragma unroll
      for (int j = 0; j < M; ++j) {
        const double y = f * lane_f64(z[j], k);
        z[j] = t > k ? z[j] - y : z[j];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < M; ++j)
#pragma unroll
    for (int r = NM - 1; r >= 0; --r) {
      if (r < n) {
        double s = z[j];
#pragma unroll
        for (int c = r + 1; c < NM; ++c)
          if (c < n) s -= A[c] * x[j][c];
        x[j][r] = lane_f64(s / (A[r] != 0.0 ? A[r] : 1.0), r);
      }
    }
  return ok;
}

// Lane t's task of support m: its t-th in increasing order.
template <int K>
__device__ __forceinline__ int support_task(uint32_t m, int t) {
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (i < t) m &= m - 1u;
  return m ? __builtin_ctz(m) : 0;
}

// mgda_support on a whole wavefront (m uniform): lane t < K gets task t's
// weight in *own.
template <int K>
__device__ __forceinline__ bool lane_mgda_support(const double *Gn, uint32_t m, int t, double *own, double *q) {
  const int n = __builtin_popcount(m), me = support_task<K>(m, t);
  double A[K + 1], z[1] = {t == n ? 1.0 : 0.0}, x[1][K + 1];
  int task[K];
#pragma unroll
  for (int c = 0; c <= K; ++c) {
    if (c < K) task[c < K ? c : 0] = __builtin_amdgcn_readlane(me, c);
    const double g = c < K && t < n && c < n ? Gn[me * K + task[c < K ? c : 0]] : 0.0;
    A[c] = t < n && c < n ? g : (t < n && c == n) || (t == n && c < n) ? 1.0 : 0.0;
  }
  if (!lane_ge_solve<K + 1, 1>(A, z, n + 1, t, x)) return false;
  double amin = n < K ? 0.0 : x[0][0], sum = 0.0;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) {
      amin = x[0][u] < amin ? x[0][u] : amin;
      sum += x[0][u];
    }
  if (!(amin >= -1e-10) || !(fabs(sum - 1.0) <= 1e-9)) return false;
  double a[K], csum = 0.0;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) {
      a[u] = x[0][u] > 0.0 ? x[0][u] : 0.0;
      csum += a[u];
    }
  const int at = __builtin_popcount(m & ((1u << (t & 31)) - 1u)), row = t < K ? t : 0;
  double mine = 0.0, g = 0.0;  // this lane's weight and (Gn a)_t
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) {
      a[u] = a[u] / csum;
      mine = u == at ? a[u] : mine;
      g += Gn[row * K + task[u]] * a[u];
    }
  double qq = 0.0;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) qq += a[u] * lane_f64(g, task[u]);
  if (!__all(t >= K || g >= qq - 1e-9)) return false;
  *own = t < K && (m >> t) & 1u ? mine : 0.0;
  *q = qq;
  return true;
}

// cagrad_support on a whole wavefront (m uniform, two tasks or more): even
// lanes try the smaller root, odd ones the larger; `kept` and *F are the
// lane's, w[u] its weight of the support's u-th task.
template <int K>
__device__ __forceinline__ bool lane_cagrad_support(const double *G, const double *bvec, double r, uint32_t m, int t,
                                                    double (&w)[K], double *F) {
  const int n = __builtin_popcount(m), me = support_task<K>(m, t);
  double A[K], z[2] = {1.0, bvec[me]}, x[2][K];
  int task[K];
#pragma unroll
  for (int c = 0; c < K; ++c) {
    task[c] = __builtin_amdgcn_readlane(me, c);
    A[c] = t < n && c < n ? G[me * K + task[c]] : 0.0;
  }
  if (!lane_ge_solve<K, 2>(A, z, n, t, x)) return false;
  double qa = 0.0, h1b = 0.0, hbb = 0.0;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) {
      const double b = bvec[task[u]];
      qa += x[0][u];
      h1b += x[0][u] * b;
      hbb += b * x[1][u];
    }
  const double qb = -2.0 * h1b, qc = hbb - r * r;
  const double disc = qb * qb - 4.0 * qa * qc;
  if (!(qa > 0.0) || !(disc >= 0.0)) return false;
  const double sq = sqrt(disc);
  const double lam = (t & 1) == 0 ? (-qb - sq) / (2.0 * qa) : (-qb + sq) / (2.0 * qa);
  double vmin = 0.0, vsum = 0.0, csum = 0.0;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) {
      const double v = (lam * x[0][u] - x[1][u]) / r;
      w[u] = v;
      vmin = u == 0 || v < vmin ? v : vmin;
      vsum += v;
    }
  const bool kept = vmin >= -1e-12 && vsum > 0.0;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) {
      w[u] = w[u] > 0.0 ? w[u] : 0.0;
      csum += w[u];
    }
  double bw = 0.0, q = 0.0;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) w[u] = w[u] / csum;
#pragma unroll
  for (int u = 0; u < K; ++u)
    if (u < n) {
      bw += bvec[task[u]] * w[u];
      double g = 0.0;
#pragma unroll
      for (int v = 0; v < K; ++v)
        if (v < n) g += w[v] * G[task[v] * K + task[u]];
      q += g * w[u];
    }
  const double f = bw + r * sqrt(q > 0.0 ? q : 0.0);
  if (!kept || !__builtin_isfinite(f)) return false;
  *F = f;
  return true;
}

template <int K, bool CAGRAD>
__global__ __launch_bounds__(kWave, CAGRAD && K == 10 ? 1 : 2) void exact_lanes_kernel(const double *__restrict__ gram, double c,
                                                                float *__restrict__ weights,
                                                                double *__restrict__ aux) {
  constexpr int LB = Tableau<K, CAGRAD>::LB, GB = K - LB;
  const int64_t b = blockIdx.x;
  const int t = threadIdx.x;
  __shared__ Shared S;
  __shared__ double d[K], db[K];  // D 1, D b
  __shared__ int found;
  __shared__ uint32_t mask[2];
  if (t == 0) found = 0;
  for (int i = t; i < K * K; i += kWave) S.G[i] = gram[b * K * K + i];
  WaveSync()();
  // the scale of the tolerances (MGDA: G over its largest diagonal entry, as
  // in the solve), b, r
  double dmax = 0.0, dmin = __builtin_inf(), bmax = 0.0, tot = 0.0;
#pragma unroll 1
  for (int i = 0; i < K; ++i) {
    const double x = S.G[i * K + i];
    dmax = x > dmax ? x : dmax;
    dmin = x < dmin ? x : dmin;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < K; ++j) s += S.G[i * K + j];
    tot += s;
    s = s / (double)K;
    bmax = fabs(s) > bmax ? fabs(s) : bmax;
    if (t == i) S.bvec[i] = s;
  }
  const double r = CAGRAD ? c * sqrt(tot > 0.0 ? tot / (double)(K * K) : 0.0) : 1.0;
  const double norm = CAGRAD ? 1.0 : dmax;
  // every entry finite, every norm positive and in range, a radius
  bool sure = dmin > 1e-12 * dmax && dmax < 1e200 && dmin > 1e-200 && __builtin_isfinite(tot) && r > 0.0;
  if (t < K) {
    d[t] = sqrt(norm / S.G[t * K + t]);
    db[t] = d[t] * S.bvec[t];
  }
  for (int i = t; i < K * K; i += kWave) {  // D G D (norm: G over it below)
    const double x = S.G[i] / sqrt(S.G[i / K * K + i / K] * S.G[i % K * K + i % K]);
    S.C[i] = x;
    // (not a NaN); two tasks of which one's pivot will be too small after the
    // other's, as it would be in every support of both: no need to walk them
    sure = sure && fabs(x) <= 1.0 + 1e-9 && (i % (K + 1) == 0 || x * x <= 1.0 - kScreenPivot);
  }
  if (!__all(sure)) {
    if (t == 0) reinterpret_cast<uint32_t *>(weights)[b * K] = kUnsolved;
    return;
  }
  WaveSync()();
  Tableau<K, CAGRAD> tb;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    tb.h[i] = d[i];
    tb.e[i] = CAGRAD ? db[i] : 0.0;
#pragma unroll
    for (int j = i; j < K; ++j) tb.T[i][j] = i == j ? 1.0 : S.C[i * K + j];
  }
  const double dM = sqrt(norm / dmin), dm = sqrt(norm / dmax);  // largest and smallest d
  // MGDA keeps a support with a_i >= -1e-10 and (G a)_t >= q - 1e-9, with a =
  // y / sum y and q = 1 / sum y: h_i >= -1e-10 sum y / d_i, h_t <= 1e-9 d_t sum y,
  // and sum y <= dM sum |h|.  CAGrad: v_i = d_i u_i / r >= -1e-12.
  const double c1 = CAGRAD ? kScreenTol : fmax(kScreenTol, fmax(2e-9 * dM * dM, 2e-10 * dM / dm));
  const uint32_t lane_mask = (uint32_t)t & ((1u << LB) - 1u);
  const bool active = t < (1 << LB);
#pragma unroll
  for (int k = 0; k < LB; ++k) {
    sure = tb.sweep(k, (lane_mask >> k) & 1u, 1.0) && sure;
    __builtin_amdgcn_sched_barrier(0);
  }

  if (!__all(sure || !active)) {
    if (t == 0) reinterpret_cast<uint32_t *>(weights)[b * K] = kUnsolved;
    return;
  }

  int mine = 0;
  uint32_t m0 = 0, m1 = 0;
#pragma unroll
  for (int g = 0; g < (1 << GB); ++g) {
    const uint32_t gray = (uint32_t)(g ^ (g >> 1));
    if (g > 0) {
      const int k = __builtin_ctz(g);
      sure = tb.sweep(LB + (k < GB ? k : 0), true, (gray >> k) & 1u ? 1.0 : -1.0) && sure;
    }
    __builtin_amdgcn_sched_barrier(0);  // states one after the other: overlapped, they spill
    const uint32_t m = lane_mask | (gray << LB);
    bool fits;
    if constexpr (!CAGRAD) {
      fits = signs_fit<K>(tb.h, m, kScreenTol * dM, c1);
    } else {
      double qa = 0.0, h1b = 0.0, hbb = 0.0;
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const double hi = (m >> i) & 1u ? tb.h[i] : 0.0, ei = (m >> i) & 1u ? tb.e[i] : 0.0;
        qa = __builtin_fma(d[i], hi, qa);
        h1b = __builtin_fma(db[i], hi, h1b);
        hbb = __builtin_fma(db[i], ei, hbb);
      }
      // qa lam^2 - 2 h1b lam + hbb = r^2; qa > 0, and the discriminant's
      // rounding must not hide a root
      const double disc = h1b * h1b - qa * (hbb - r * r);
      const double sq = sqrt(disc > 0.0 ? disc : 0.0);
      fits = false;
      if (m != 0 && !(disc < -1e-6 * (h1b * h1b + qa * r * r))) {
#pragma unroll
        for (int root = 0; root < 2; ++root) {
          const double lam = (root == 0 ? h1b - sq : h1b + sq) / qa;
          double u[K];
#pragma unroll
          for (int i = 0; i < K; ++i) u[i] = __builtin_fma(lam, tb.h[i], -tb.e[i]);
          const double c0 = kScreenTol * dM * (fabs(lam) + bmax) + 2e-12 * r / dm;
          fits = fits || signs_fit<K>(u, m, c0, c1);
        }
      }
    }
    if (fits && active && m != 0) {
      m1 = mine == 1 ? m : m1;
      m0 = mine == 0 ? m : m0;
      ++mine;
    }
  }
  WaveSync()();
  if (mine > 0) {
    const int at = atomicAdd(&found, mine);
    if (at < 2) mask[at] = m0;
    if (mine > 1 && at < 1) mask[1] = m1;
  }
  WaveSync()();
  // the supports left, in rank order
  const int n = found;
  if (!__all(sure || !active) || n < 1 || n > 2) {
    if (t == 0) reinterpret_cast<uint32_t *>(weights)[b * K] = kUnsolved;
    return;
  }
  uint32_t left[2] = {mask[0], n == 2 ? mask[1] : 0u};
  if (n == 2 && ranks_before(left[1], left[0])) {
    const uint32_t m = left[0];
    left[0] = left[1];
    left[1] = m;
  }
  double wt = 0.0, ax = 0.0;
  if constexpr (!CAGRAD) {
    for (int i = t; i < K * K; i += kWave) S.G[i] = S.G[i] / dmax;
    WaveSync()();
    bool some = false;
    double q = 0.0;
    for (int i = 0; i < n; ++i) {
      double own, qi;
      const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)left[i]);
      if (lane_mgda_support<K>(S.G, m, t, &own, &qi) && (!some || qi < q - 1e-12)) {
        some = true;
        q = qi;
        wt = ax = own;
      }
    }
    if (!some) {
      if (t == 0) reinterpret_cast<uint32_t *>(weights)[b * K] = kUnsolved;
      return;
    }
  } else {
    double all = 0.0;
    for (int i = 0; i < K * K; ++i) all += S.G[i];
    double g0sq = all / (double)(K * K);
    g0sq = g0sq > 0.0 ? g0sq : 0.0;
    const double rr = c * sqrt(g0sq);
    double bf = __builtin_inf();
    int bslot = 0x7fffffff;
    if (t < K) {  // the vertices
      const double gtt = S.G[t * K + t];
      bf = S.bvec[t] + rr * sqrt(gtt > 0.0 ? gtt : 0.0);
      bslot = t;
    }
    bool some = false;  // a support left is a vertex, or one of its points is kept
    for (int i = 0; i < n; ++i) {
      const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)left[i]);
      if (__builtin_popcount(m) < 2) {
        some = true;
        continue;
      }
      double w[K], f;
      const bool kept = lane_cagrad_support<K>(S.G, S.bvec, rr, m, t, w, &f);
      if (kept && t < 2) {
#pragma unroll
        for (int u = 0; u < K; ++u) S.C[(2 * i + t) * K + u] = w[u];
      }
      some = __any(kept) || some;
      if (kept && before(f, K + 2 * i + (t & 1), bf, bslot)) {
        bf = f;
        bslot = K + 2 * i + (t & 1);
      }
    }
    if (!some) {
      if (t == 0) reinterpret_cast<uint32_t *>(weights)[b * K] = kUnsolved;
      return;
    }
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
      const double of = __shfl_xor(bf, off, kWave);
      const int os = __shfl_xor(bslot, off, kWave);
      if (before(of, os, bf, bslot)) {
        bf = of;
        bslot = os;
      }
    }
    WaveSync()();
    if (t < K) {
      const uint32_t m = bslot < K ? 1u << bslot : left[(bslot - K) >> 1];
      const int at = __builtin_popcount(m & ((1u << t) - 1u));
      S.a[t] = !((m >> t) & 1u) ? 0.0 : bslot < K ? 1.0 : S.C[(bslot - K) * K + at];
    }
    WaveSync()();
    cagrad_primal<WaveSync>(S, K, rr, 1.0 / (double)K, t);
    if (t < K) {
      wt = S.C[t];
      ax = S.a[t];
    }
  }
  if (t < K) {
    weights[b * K + t] = (float)wt;
    if (aux) aux[b * K + t] = ax;
  }
}

constexpr int kMaxSupports = (1 << kExactMaxK) - 1;

// Every support of bucket b (a whole wavefront).
__device__ __forceinline__ void exact_solve_bucket(int K, int64_t b, const double *__restrict__ gram, int method,
                                                   double c, float *__restrict__ weights, double *__restrict__ aux) {
  __shared__ Shared S;
  __shared__ double Gn[kExactMaxK * kExactMaxK];
  __shared__ double qv[kMaxSupports];
  __shared__ uint32_t ok[kMaxSupports];  // mask | kept << 16
  __shared__ int choice;
  const int t = threadIdx.x;
  const int nsub = (1 << K) - 1;
  solver_load_gram<WaveSync>(S, K, gram + b * K * K, t, kWave);
  if (S.bad) {
    if (t < K) {
      weights[b * K + t] = __builtin_nanf("");
      if (aux) aux[b * K + t] = __builtin_nan("");
    }
    return;
  }
  double wt = 0.0, ax = 0.0;
  if (method == MGDA_EXACT) {
    double dmax = S.G[0];
    for (int i = 1; i < K; ++i) dmax = S.G[i * K + i] > dmax ? S.G[i * K + i] : dmax;
    const double scale = dmax > 1e-300 ? dmax : 1e-300;
    for (int i = t; i < K * K; i += kWave) Gn[i] = S.G[i] / scale;
    WaveSync()();
    for (int rk = t; rk < nsub; rk += kWave) {
      const uint32_t m = kSupportTables.m[K][rk];
      double q = 0.0;
      const bool kept = mgda_any(Gn, K, m, &q, nullptr);
      qv[rk] = q;
      ok[rk] = m | (kept ? 1u << 16 : 0u);
    }
    WaveSync()();
    if (t == 0) {
      int best = -1;
      double bq = 0.0;
      for (int rk = 0; rk < nsub; ++rk)
        if ((ok[rk] >> 16) && (best < 0 || qv[rk] < bq - 1e-12)) {
          best = rk;
          bq = qv[rk];
        }
      choice = best;
      if (best >= 0) {
        double q;
        mgda_any(Gn, K, ok[best] & 0xFFFFu, &q, S.a);
      }
    }
    WaveSync()();
    if (choice < 0) solve_mgda<WaveSync>(S, K, 5000, t);
    if (t < K) wt = ax = S.a[t];
  } else {  // CAGRAD_EXACT
    const double invK = 1.0 / (double)K;
    if (t < K) {
      double s = 0.0;
      for (int j = 0; j < K; ++j) s += S.G[t * K + j];
      S.bvec[t] = s / (double)K;
    }
    WaveSync()();
    double tot = 0.0;
    for (int i = 0; i < K * K; ++i) tot += S.G[i];
    double g0sq = tot / (double)(K * K);
    g0sq = g0sq > 0.0 ? g0sq : 0.0;
    const double r = c * sqrt(g0sq);
    // this lane's best candidate: slot t < K are the vertices; support rank
    // rk >= K gives slots K + 2 (rk - K) + root
    double bf = __builtin_inf();
    int bslot = 0x7fffffff;
    uint32_t bmask = 0;
    if (t < K) {
      const double gtt = S.G[t * K + t];
      bf = S.bvec[t] + r * sqrt(gtt > 0.0 ? gtt : 0.0);
      bslot = t;
    }
    if (r > 0.0)
      for (int rk = K + t; rk < nsub; rk += kWave) {
        const uint32_t m = kSupportTables.m[K][rk];
        for (int root = 0; root < 2; ++root) {
          double f;
          if (cagrad_any(S.G, S.bvec, r, K, m, root, &f, nullptr)) {
            const int slot = K + 2 * (rk - K) + root;
            if (before(f, slot, bf, bslot)) {
              bf = f;
              bslot = slot;
              bmask = m;
            }
          }
        }
      }
    for (int off = kWave / 2; off >= 1; off >>= 1) {
      const double of = __shfl_xor(bf, off, kWave);
      const int os = __shfl_xor(bslot, off, kWave);
      const uint32_t om = (uint32_t)__shfl_xor((int)bmask, off, kWave);
      if (before(of, os, bf, bslot)) {
        bf = of;
        bslot = os;
        bmask = om;
      }
    }
    // every lane now holds the winner; lane 0 rebuilds its point
    if (t == 0) {
      if (bslot < K) {
        for (int i = 0; i < K; ++i) S.a[i] = i == bslot ? 1.0 : 0.0;
      } else {
        double f;
        cagrad_any(S.G, S.bvec, r, K, bmask, (bslot - K) & 1, &f, S.a);
      }
    }
    WaveSync()();
    cagrad_primal<WaveSync>(S, K, r, invK, t);
    if (t < K) {
      wt = S.C[t];
      ax = S.a[t];
    }
  }
  if (t < K) {
    weights[b * K + t] = (float)wt;
    if (aux) aux[b * K + t] = ax;
  }
}

// The buckets that the first kernel left (or all of them).  With LOOP a wavefront
// looks at several, lane j at bucket blockIdx.x + j * gridDim.x, so that a call of
// very many buckets does not launch one for each just to end it; else one a
// wavefront, which saves the loop's spills around the support solvers' calls.
// Loop / one each, us, K=3 CAGrad: 60,000 buckets none of them left 130 / 146, all
// 673 / 618; 6,564 buckets none 25.5 / 25.2, all 87 / 78; K=10 MGDA, 6,564, all
// 1,347 / 1,230.
constexpr int kExactLoopBuckets = 16384;
template <bool LOOP>
__global__ __launch_bounds__(kWave) void exact_solve_kernel(int K, int B, int all, const double *__restrict__ gram,
                                                            int method, double c, float *weights,
                                                            double *__restrict__ aux) {
  const uint32_t *mark = reinterpret_cast<const uint32_t *>(weights);
  if constexpr (!LOOP) {
    const int64_t b = blockIdx.x;
    if (all || mark[b * K] == kUnsolved) exact_solve_bucket(K, b, gram, method, c, weights, aux);
    return;
  }
  for (int64_t first = blockIdx.x; first < B; first += (int64_t)gridDim.x * kWave) {
    const int64_t mine = first + (int64_t)threadIdx.x * gridDim.x;
    uint64_t todo = __ballot(mine < B && (all || mark[mine < B ? mine * K : 0] == kUnsolved));
    while (todo) {
      const int j = __builtin_ctzll(todo);
      todo &= todo - 1;
      exact_solve_bucket(K, first + (int64_t)j * gridDim.x, gram, method, c, weights, aux);
      WaveSync()();
    }
  }
}

template <bool CAGRAD>
hipError_t launch_lanes(int K, int B, const double *gram, double c, float *weights, double *aux, hipStream_t s) {
#define BKMOO_LANES_CASE(k)                                                                                \
  case k:                                                                                                   \
    hipLaunchKernelGGL((exact_lanes_kernel<k, CAGRAD>), dim3((unsigned)B), dim3(kWave), 0, s, gram, c, weights, aux); \
    break;
  switch (K) {
    BKMOO_LANES_CASE(2) BKMOO_LANES_CASE(3) BKMOO_LANES_CASE(4) BKMOO_LANES_CASE(5) BKMOO_LANES_CASE(6)
    BKMOO_LANES_CASE(7) BKMOO_LANES_CASE(8) BKMOO_LANES_CASE(9) BKMOO_LANES_CASE(10)
    default: return hipErrorInvalidValue;
  }
#undef BKMOO_LANES_CASE
  return hipGetLastError();
}

}  // namespace

hipError_t launch_exact_solve(int K, int B, const double *gram, int method, double c, float *weights,
                              double *aux, hipStream_t s) {
  if (K < kMinK || K > kExactMaxK) return hipErrorInvalidValue;
  const int fit = device_cu_count() * 4;  // wavefronts of the second kernel that fit at a time
  // two tasks have three supports, which it solves sooner than a screen and
  // another launch take (613 buckets 10.3 / 12.6 us), as long as all fit
  const int all = K == 2 && B <= fit;
  if (!all) {
    const hipError_t e = method == MGDA_EXACT ? launch_lanes<false>(K, B, gram, c, weights, aux, s)
                                              : launch_lanes<true>(K, B, gram, c, weights, aux, s);
    if (e != hipSuccess) return e;
  }
  const bool loop = B > kExactLoopBuckets;
  hipLaunchKernelGGL(loop ? exact_solve_kernel<true> : exact_solve_kernel<false>, dim3((unsigned)(loop ? fit : B)),
                     dim3(kWave), 0, s, K, B, all, gram, method, c, weights, aux);
  return hipGetLastError();
}

}  // namespace bkmoo
