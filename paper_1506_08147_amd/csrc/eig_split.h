// Lowest k eigenpairs of a tridiagonalised symmetric matrix, spread over many
// workgroups per matrix.  The eigenvalues are independent of one another, and
// so are the inverse iterations and the columns of the back-transformation;
// only the orthogonalisation inside clusters couples columns.  Stages, each
// one launch over all matrices of a batch:
//
//   eig_bisect     eigenvalues by multisection of the Sturm count
//   eig_invit      eigenvectors of the tridiagonal by inverse iteration
//   eig_cluster    modified Gram-Schmidt inside clusters of close eigenvalues
//   eig_back       Z := H_0 ... H_{n-3} Z for the Householder reflectors
//
// Every stage is a serial recurrence of length n per eigenvalue or vector, so
// what bounds it is the latency of that chain; in one workgroup per matrix
// (16 waves on one of 256 compute units) the chains of a matrix also queued
// behind one another.  Measured, 16 matrices of order 816, lowest 272: all
// four stages in one workgroup per matrix 28.5 ms, here 4.2 ms (bisect 1.2,
// invit 1.1, cluster 0.1, back 1.9).
#pragma once
#include "small_dense.h"

namespace dg {

// One matrix of a batch: reflectors of the tridiagonalisation below the
// subdiagonal of A (leading dimension n), work = d, e, tau (n each), then
// 4 n k doubles of the inverse iteration.  n = 0: nothing to do.
struct EigView {
  int n, k;
  double *A, *w, *Z, *work;
};

constexpr int EIG_MAXN = 832;              // orders handled here
constexpr int EIG_BIS_THREADS = 256;
constexpr int EIG_BIS_G = 32;              // lanes per eigenvalue
constexpr int EIG_BIS_COLS = EIG_BIS_THREADS / EIG_BIS_G;
constexpr int EIG_INV_COLS = 64;           // vectors per (one-wave) workgroup
constexpr int EIG_CL_THREADS = 1024;
constexpr int EIG_BT_THREADS = 512;
constexpr int EIG_BT_U = 2;                // columns per wave
constexpr int EIG_BT_COLS = EIG_BT_U * EIG_BT_THREADS / 64;
constexpr int EIG_BT_NB = 8;               // reflectors staged at a time

// 1/q to the last place or so: the hardware reciprocal and two Newton steps
// (half the dependent chain of an IEEE division; |q| is at least the pivot
// floor, so nothing overflows on the way).
__device__ __forceinline__ double recip(double q) {
  double r = __builtin_amdgcn_rcp(q);
  r = fma(fma(-q, r, 1.0), r, r);
  r = fma(fma(-q, r, 1.0), r, r);
  return r;
}

// Gershgorin interval, norm and pivot floor of the tridiagonal (d, e), the
// same for every thread of the workgroup.  red: LDS, >= 32 doubles.
struct TriBounds {
  double gl, gu, tnorm, pivmin;
};
template <class T>
__device__ __forceinline__ TriBounds tri_bounds(T& t, const double* d, const double* e, int n) {
  double gl = -1e300, gu = -1e300, em = 0.0;     // gl: largest -(lower end)
  for (int i = t.tid(); i < n; i += t.nt()) {
    const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i < n - 1 ? fabs(e[i]) : 0.0);
    gl = fmax(gl, -(d[i] - r));
    gu = fmax(gu, d[i] + r);
    if (i < n - 1) em = fmax(em, e[i] * e[i]);
  }
  TriBounds b;
  b.gl = -t.maxv(gl);
  b.gu = t.maxv(gu);
  em = t.maxv(em);
  b.tnorm = fmax(fabs(b.gl), fabs(b.gu));
  b.pivmin = fmax(1e-290, 1e-290 * em);
  const double eps = 2.220446049250313e-16;
  b.gl -= 2.0 * eps * b.tnorm * n + b.pivmin;
  b.gu += 2.0 * eps * b.tnorm * n + b.pivmin;
  return b;
}

// Eigenvalues [wg EIG_BIS_COLS, + EIG_BIS_COLS): G lanes per eigenvalue, each
// with one point of the interval, so a round divides the interval by G + 1 =
// 33 (a double's 53 bits in 11 rounds).  G = 32 against 16 with two points a lane
// (the same points): the second recurrence of a lane filled issue slots that the
// extra waves fill as well, and where there are few waves it only lengthened
// the step.  Lowest 32 of 96, 4 matrices: 95 -> 70 us; 272 of 816, 16 matrices:
// 1.29 -> 1.21 ms, with d and e^2 read from LDS ahead of the recurrence.
// lds: 2 n doubles.
__device__ __forceinline__ void eig_bisect_body(const EigView& m, int wg, double* lds, double* red) {
  const int n = m.n, k = m.k;
  if (wg * EIG_BIS_COLS >= k) return;
  DevTeam t{red};
  double* d = lds;
  double* e2 = lds + n;
  const double* dg = m.work;
  const double* eg = m.work + n;
  for (int i = t.tid(); i < n; i += t.nt()) {
    d[i] = gld(dg + i);
    e2[i] = i < n - 1 ? gld(eg + i) : 0.0;
  }
  t.sync();
  const TriBounds b = tri_bounds(t, d, e2, n);
  for (int i = t.tid(); i < n; i += t.nt()) e2[i] *= e2[i];
  t.sync();
  constexpr int G = EIG_BIS_G;
  const double eps = 2.220446049250313e-16, pivmin = b.pivmin;
  const int lane = threadIdx.x & 63, sidx = threadIdx.x % G;
  const int j = wg * EIG_BIS_COLS + threadIdx.x / G;
  const int base = lane - sidx;
  const unsigned long long gmask = ((1ull << G) - 1ull) << base;
  double lo = b.gl, hi = b.gu;
  bool done = j >= k;
  for (int it = 0; it < 200; ++it) {
    if (!done && hi - lo <= 2.0 * eps * fmax(fabs(lo), fabs(hi)) + pivmin) done = true;
    if (__all(done ? 1 : 0)) break;
    // points in ascending order over the lanes
    const double x = lo + (hi - lo) * (double)(sidx + 1) / (double)(G + 1);
    double q = d[0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    int c = q < 0.0;
    auto step = [&](double di, double ei) {
      q = fma(-ei, recip(q), di - x);
      if (fabs(q) < pivmin) q = -pivmin;
      c += q < 0.0;
    };
    // d and e^2 a chunk ahead of the recurrence
    constexpr int CH = 8;
    double df[CH], ef[CH];
    auto fetch = [&](int i0) {
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int i = i0 + u < n ? i0 + u : n - 1;
        df[u] = d[i];
        ef[u] = e2[i > 0 ? i - 1 : 0];
      }
    };
    int i = 1;
    fetch(i);
    for (; i + CH <= n; i += CH) {
      double dc[CH], ec[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        dc[u] = df[u];
        ec[u] = ef[u];
      }
      fetch(i + CH);
#pragma unroll
      for (int u = 0; u < CH; ++u) step(dc[u], ec[u]);
    }
    for (; i < n; ++i) step(d[i], e2[i - 1]);
    // points whose count is at most j lie below the eigenvalue
    const int cnt = __popcll(__ballot((!done && c <= j) ? 1 : 0) & gmask);
    const double a = __shfl(x, base + ((cnt - 1) & (G - 1)), 64);
    const double z = __shfl(x, base + (cnt & (G - 1)), 64);
    const double plo = cnt > 0 ? a : lo, phi = cnt < G ? z : hi;
    if (!done) {
      if (plo == lo && phi == hi) done = true;
      lo = plo;
      hi = phi;
    }
  }
  if (j < k && sidx == 0) gst(m.w + j, 0.5 * (lo + hi));
}

// Vectors [wg 64, + 64), one per lane of a one-wave workgroup: three inverse
// iterations from a fixed pseudo-random start.  The partial-pivoting LU of
// T - lambda I is fused with the forward substitution and carries its
// recurrences in registers; only U (as 1 / pivot and two superdiagonals) and
// x go through memory, interleaved over the lanes, and are read back CH rows
// ahead of the recurrence, as are d and e from LDS; no lane branches on its
// pivot.  Measured, k of n: 272 of 816 (16 matrices) 1.78 -> 1.06 ms against a
// branch per pivot and reads inside the recurrence, 32 of 96 (4) 168 -> 105 us.  lds: 2 n doubles + the 64 x 17 output tile.
constexpr int EIG_INV_TILE = 64 * 17;
__device__ __forceinline__ void eig_invit_body(const EigView& m, int wg, double* lds, double* red) {
  const int n = m.n, k = m.k;
  if (wg * EIG_INV_COLS >= k) return;
  DevTeam t{red};
  double* d = lds;
  double* e = lds + n;
  double* tile = lds + 2 * n;
  for (int i = t.tid(); i < n; i += t.nt()) {
    d[i] = gld(m.work + i);
    e[i] = i < n - 1 ? gld(m.work + n + i) : 0.0;
  }
  t.sync();
  const TriBounds b = tri_bounds(t, d, e, n);
  const int lane = threadIdx.x;
  const int j = wg * EIG_INV_COLS + lane;
  const int jc = j < k ? j : k - 1;        // idle lanes repeat the last vector and its stores
  const double lam = gld(m.w + jc);
  const double eps = 2.220446049250313e-16, tiny = eps * b.tnorm + 1e-290, rtiny = recip(tiny);
  const long long nk = (long long)n * k;
  double* W0 = m.work + 3 * (long long)n + jc;
  auto at = [&](int a, int i) { return W0 + a * nk + (long long)i * k; };
  constexpr int CH = 8;
  double sc = 1.0;                         // scale of the stored x
  for (int it = 0; it < 3; ++it) {
    // rows i0 .. i0 + CH - 1 of the start vector, d and e, a chunk ahead
    double xf[CH], df[CH], ef[CH];
    auto fetch = [&](int i0) {
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int i = i0 + c < n ? i0 + c : n - 1;
        xf[c] = it == 0 ? start_value(((unsigned long long)jc << 32) + i) : gld(at(3, i));
        df[c] = d[i];
        ef[c] = e[i];
      }
    };
    fetch(0);
    double ddi = df[0] - lam, dui = ef[0], xi = xf[0] * sc, bb = ef[0];
    fetch(1);
    auto chunk = [&](int i0, int rows) {
      double xb[CH], db[CH], eb[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        xb[c] = xf[c] * sc;
        db[c] = df[c] - lam;
        eb[c] = ef[c];
      }
      fetch(i0 + CH);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (c >= rows) break;
        const int i = i0 + c - 1;          // eliminates row i + 1
        const double ddn = db[c], dun = eb[c], xn = xb[c];   // e[n - 1] = 0
        // row i or i + 1 as the pivot row, without a branch: lanes differ
        const bool swap = !(fabs(ddi) >= fabs(bb) || fabs(bb) < 1e-290);
        if (!swap && fabs(ddi) < 1e-290) ddi = tiny;
        const double piv = swap ? bb : ddi, u1 = swap ? ddn : dui, u2 = swap ? dun : 0.0, xo = swap ? xn : xi;
        const double rp = recip(piv), f = (swap ? ddi : bb) * rp;
        ddi = fma(-f, u1, swap ? dui : ddn);
        xi = fma(-f, xo, swap ? xi : xn);
        dui = swap ? -f * dun : dun;
        gst(at(0, i), fabs(piv) < tiny ? (piv < 0 ? -rtiny : rtiny) : rp);
        gst(at(1, i), u1);
        gst(at(2, i), u2);
        gst(at(3, i), xo);
        bb = dun;
      }
    };
    int i0 = 1;
    for (; i0 + CH <= n; i0 += CH) chunk(i0, CH);
    if (i0 < n) chunk(i0, n - i0);
    if (fabs(ddi) < tiny) ddi = ddi < 0 ? -tiny : tiny;
    gst(at(0, n - 1), recip(ddi));
    gst(at(1, n - 1), 0.0);
    gst(at(2, n - 1), 0.0);
    gst(at(3, n - 1), xi);
    // the lane's own stores are read back below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    double x1 = 0.0, x2 = 0.0, smax = 0.0;
    double r[CH], u1[CH], u2[CH], v[CH], rf[CH], u1f[CH], u2f[CH], vf[CH];
    auto bfetch = [&](int i0) {
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int i = i0 - c > 0 ? i0 - c : 0;
        rf[c] = gld(at(0, i));
        u1f[c] = gld(at(1, i));
        u2f[c] = gld(at(2, i));
        vf[c] = gld(at(3, i));
      }
    };
    bfetch(n - 1);
    auto bchunk = [&](int i0, int rows) {
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        r[c] = rf[c];
        u1[c] = u1f[c];
        u2[c] = u2f[c];
        v[c] = vf[c];
      }
      bfetch(i0 - CH);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (c >= rows) break;
        const double s = fma(-u2[c], x2, fma(-u1[c], x1, v[c])) * r[c];
        gst(at(3, i0 - c), s);
        smax = fmax(smax, fabs(s));
        x2 = x1;
        x1 = s;
      }
    };
    int ib = n - 1;
    for (; ib >= CH - 1; ib -= CH) bchunk(ib, CH);
    if (ib >= 0) bchunk(ib, ib + 1);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const double is = 1.0 / smax;
    double nr[CH], nf[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      nr[c] = 0.0;
      nf[c] = gld(at(3, c < n ? c : n - 1));
    }
    for (int q = 0; q < n; q += CH) {
      double nv[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        nv[c] = nf[c] * is;
        nf[c] = gld(at(3, q + CH + c < n ? q + CH + c : n - 1));
      }
#pragma unroll
      for (int c = 0; c < CH; ++c)
        if (q + c < n) nr[c] = fma(nv[c], nv[c], nr[c]);
    }
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < CH; ++c) s += nr[c];
    sc = is / sqrt(s);
  }
  // columns to Z through a 16-row tile (contiguous stores)
  for (int i0 = 0; i0 < n; i0 += 16) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (i0 + r < n) tile[lane * 17 + r] = gld(at(3, i0 + r)) * sc;
    t.sync();
    for (int q = lane; q < 16 * EIG_INV_COLS; q += 64) {
      const int r = q & 15, c = q >> 4, jj = wg * EIG_INV_COLS + c;
      if (jj < k && i0 + r < n) gst(m.Z + (i0 + r) + (long long)n * jj, tile[c * 17 + r]);
    }
    t.sync();
  }
}

// Modified Gram-Schmidt inside clusters (neighbours closer than 1e-5 ||T||),
// columns in index order; one workgroup per matrix, one wave per cluster.
// lds: n doubles, then k ints of cluster starts.
__device__ __forceinline__ void eig_cluster_body(const EigView& m, double* lds, double* red) {
  const int n = m.n, k = m.k;
  if (n == 0) return;
  DevTeam t{red};
  double* w = lds;                         // k <= n
  int* first = (int*)(lds + n);            // 1: column starts a cluster
  const double* d = m.work;
  const double* e = m.work + n;
  // (the norm comes from global memory: two reads per row)
  const TriBounds b = tri_bounds(t, d, e, n);
  for (int j = t.tid(); j < k; j += t.nt()) w[j] = gld(m.w + j);
  t.sync();
  for (int j = t.tid(); j < k; j += t.nt()) first[j] = j == 0 || w[j] - w[j - 1] > 1e-5 * b.tnorm;
  t.sync();
  const int lane = t.tid() & 63, wv = t.tid() >> 6, nw = t.nt() >> 6;
  int cidx = 0;
  for (int j = 0; j < k;) {
    int jend = j + 1;
    while (jend < k && !first[jend]) ++jend;
    if (jend - j > 1 && (cidx++ % nw) == wv) {
      for (int a = j; a < jend; ++a) {
        double* ya = m.Z + (long long)n * a;
        for (int c = j; c < a; ++c) {
          const double* yc = m.Z + (long long)n * c;
          double s = 0.0;
          for (int i = lane; i < n; i += 64) s += gld(ya + i) * gld(yc + i);
          s = wave_sum_dpp(s);
          for (int i = lane; i < n; i += 64) gst(ya + i, gld(ya + i) - s * gld(yc + i));
        }
        double s = 0.0;
        for (int i = lane; i < n; i += 64) s += gld(ya + i) * gld(ya + i);
        s = 1.0 / sqrt(wave_sum_dpp(s));
        for (int i = lane; i < n; i += 64) gst(ya + i, gld(ya + i) * s);
      }
    }
    j = jend;
  }
}

// Columns [wg EIG_BT_COLS, + EIG_BT_COLS) of Z := H_0 ... H_{n-3} Z: each
// wave carries U columns in registers (R entries per lane), reflectors go
// through LDS NB at a time, the next NB in registers meanwhile.  Rows above a
// block's first reflector are left alone.  lds: NB (n + 1) doubles.
template <int R>
__device__ __forceinline__ void eig_back_body(const EigView& m, int wg, double* lds) {
  constexpr int U = EIG_BT_U, NB = EIG_BT_NB, NW = EIG_BT_THREADS / 64;
  constexpr int PF = (NB * 64 * R + EIG_BT_THREADS - 1) / EIG_BT_THREADS;
  const int n = m.n, k = m.k;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int j0 = wg * EIG_BT_COLS + wv;
  const double* tau = m.work + 2 * (long long)n;
  double* tl = lds + NB * n;
  double z[U][R];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = lane + 64 * r, j = j0 + u * NW;
      z[u][r] = (j < k && i < n) ? gld(m.Z + i + (long long)n * j) : 0.0;
    }
  // reflectors kl .. kl + NB - 1 (those past n - 3 are zero); entry q of a
  // staged block is row pi[u] & 0xffff of reflector pi[u] >> 16
  double pf[PF], pt = 0.0;
  int pi[PF];
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    const int q = tid + u * EIG_BT_THREADS, c = q / n;
    pi[u] = (c << 16) | (q - c * n);
  }
  auto fetch = [&](int kl) {
    const double* Ak = m.A + (long long)n * kl;
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int c = pi[u] >> 16, i = pi[u] & 0xffff, kk = kl + c;
      pf[u] = (c < NB && kk <= n - 3 && i > kk) ? gld(Ak + i + n * c) : 0.0;
    }
    if (tid < NB) pt = kl + tid <= n - 3 ? gld(tau + kl + tid) : 0.0;
  };
  int kl = n >= 3 ? ((n - 3) / NB) * NB : -1;
  if (kl >= 0) fetch(kl);
  for (; kl >= 0; kl -= NB) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int q = tid + u * EIG_BT_THREADS;
      if (q < NB * n) lds[q] = pf[u];
    }
    if (tid < NB) tl[tid] = pt;
    __syncthreads();
    if (kl > 0) fetch(kl - NB);
    const int r0 = __builtin_amdgcn_readfirstlane((kl + 1) >> 6);   // first row chunk touched
    for (int c = NB - 1; c >= 0; --c) {
      const double tk = tl[c];
      if (tk == 0.0) continue;
      const double* v = lds + c * n;
      double vv[R], s[U];
#pragma unroll
      for (int u = 0; u < U; ++u) s[u] = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        vv[r] = 0.0;
        if (r >= r0) {
          const int i = lane + 64 * r;
          vv[r] = i < n ? v[i] : 0.0;
#pragma unroll
          for (int u = 0; u < U; ++u) s[u] = fma(vv[r], z[u][r], s[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) s[u] = wave_sum_dpp(s[u]) * tk;
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r >= r0) {
#pragma unroll
          for (int u = 0; u < U; ++u) z[u][r] = fma(-s[u], vv[r], z[u][r]);
        }
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = lane + 64 * r, j = j0 + u * NW;
      if (j < k && i < n) gst(m.Z + i + (long long)n * j, z[u][r]);
    }
}

__device__ __forceinline__ void eig_back_any(const EigView& m, int wg, double* lds) {
  if (m.n == 0 || wg * EIG_BT_COLS >= m.k) return;
  if (m.n <= 128) eig_back_body<2>(m, wg, lds);
  else if (m.n <= 256) eig_back_body<4>(m, wg, lds);
  else if (m.n <= 448) eig_back_body<7>(m, wg, lds);
  else if (m.n <= 640) eig_back_body<10>(m, wg, lds);
  else eig_back_body<13>(m, wg, lds);
}

}  // namespace dg
