// Householder tridiagonalisation of symmetric matrices on the device (lower
// triangle read; reflector of step k left in column k below the diagonal as
// v with H_k = I - tau_k v v^T; d, e, tau in work).
//
//   tri_reg    orders up to TRI_REG_MAX: one workgroup holds the whole matrix
//              in its registers
//   tri_step   larger orders: tri_nwg(n) workgroups per matrix, one launch per
//              Householder step, until TRI_REG_MAX rows are left
//   tri_tail   those rows, as in tri_reg
//
// A step is a matrix-vector product of the trailing block and its rank-2
// update, each needing the one before: what bounds the reduction is the
// latency of a step, not its arithmetic ((4/3) n^3 flops in all).  Measured,
// with the stages of eig_split.h, against one workgroup per matrix up to order
// 512 and 8 workgroups of 256 lanes above: 32 matrices of order 432 18.4 ->
// 7.2 ms, 16 of order 816 38.6 -> 16.1 ms (a step there takes
// 30 us at its beginning, where it moves 85 MB: 3.9 TB/s); orders up to 96
// 1.5 -> 0.17 ms.
#pragma once
#include "eig_split.h"

namespace dg {

constexpr int TRI_REG_MAX = 192;
constexpr int TRI_REG_THREADS = 1024;
constexpr int TRI_REG_WAVES = TRI_REG_THREADS / 64;
constexpr int TRI_REG_LDS = (TRI_REG_WAVES + 4) * TRI_REG_MAX + 8;

// Lane l of wave w holds rows l + 64 r (r < RC) of columns w + 16 c (c < CC),
// both triangles, so a product with the matrix needs no second (column) sum
// and nothing of the matrix moves between steps.  Three barriers a step: the
// wave that owns column k forms reflector k alone (sums over its lanes); all
// waves apply the pending rank-2 update and form their share of A v in one
// pass over their registers; the shares are summed by row.  The update
// of step k - 1 is v q^T + q v^T with q = p - K v kept as (p, K, v).
// work: d, e, tau at a stride of wld.
// The caller fills vb[1] and pb with the pending update of a step before the
// first (or zeros), K with its v . p tau / 2, and synchronises.
template <int RC, int CC>
__device__ __forceinline__ void tri_reg_body(double* A0, int ld, int n, double* work, int wld, double K,
                                             double* lds) {
  constexpr int NW = TRI_REG_WAVES, LD = TRI_REG_MAX;
  double* part = lds;                 // [NW][LD] shares of A v
  double* vb = lds + NW * LD;         // [2][LD] reflectors, zero outside their rows
  double* pb = vb + 2 * LD;           // [LD] tau A v of the last step
  double* sc = pb + 2 * LD;           // tau and the sums of v . p by wave
  double* A = const_cast<double*>(uniform_ptr(A0));
  double *d = const_cast<double*>(uniform_ptr(work)), *e = d + wld, *tau = e + wld;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  double a[RC][CC];
#pragma unroll
  for (int c = 0; c < CC; ++c)
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      const int i = lane + 64 * r, j = wv + NW * c;
      a[r][c] = (i < n && j < n) ? gld(A + (i >= j ? i + ld * j : j + ld * i)) : 0.0;
    }
  for (int k = 0; k + 2 < n; ++k) {
    double* vo = vb + ((k & 1) ^ 1) * LD;
    double* v = vb + (k & 1) * LD;
    if (wv == k % NW) {
      const int ck = k / NW;
      const double vok = vo[k], qok = pb[k] - K * vok;
      double x[RC], s2 = 0.0, x0 = 0.0, ak = 0.0;
#pragma unroll
      for (int r = 0; r < RC; ++r) {
        const int i = lane + 64 * r;
        double y = 0.0;
#pragma unroll
        for (int c = 0; c < CC; ++c)
          if (c == ck) y = a[r][c];
        const double vi = vo[i], qi = pb[i] - K * vi;   // rows past n: zero
        y -= vi * qok + qi * vok;
        x[r] = y;
        if (i > k + 1) s2 += y * y;
        if (i == k + 1) x0 = y;
        if (i == k) ak = y;
      }
      s2 = wave_sum_dpp(s2);
      x0 = wave_sum_dpp(x0);
      ak = wave_sum_dpp(ak);
      double beta = x0, v0 = 0.0, tk = 0.0;
      if (s2 != 0.0) {
        const double nrm = sqrt(x0 * x0 + s2);
        beta = x0 >= 0.0 ? -nrm : nrm;
        v0 = x0 - beta;
        tk = 2.0 / (v0 * v0 + s2);
      }
#pragma unroll
      for (int r = 0; r < RC; ++r) {
        const int i = lane + 64 * r;
        const double vi = i <= k || s2 == 0.0 ? 0.0 : (i == k + 1 ? v0 : x[r]);
        v[i] = vi;
        if (i > k && i < n) gst(A + i + ld * k, vi);
      }
      if (lane == 0) {
        sc[0] = tk;
        d[k] = ak;
        e[k] = beta;
        tau[k] = tk;
      }
    }
    __syncthreads();
    const double tk = sc[0];
    double vi[RC], voi[RC], qoi[RC], acc[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      const int i = lane + 64 * r;
      vi[r] = v[i];
      voi[r] = vo[i];
      qoi[r] = pb[i] - K * voi[r];
      acc[r] = 0.0;
    }
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      const int j = wv + NW * c;
      if (j > k && j < n) {                      // wave-uniform
        const double vj = v[j], voj = vo[j], qoj = pb[j] - K * voj;
#pragma unroll
        for (int r = 0; r < RC; ++r) {
          a[r][c] -= voi[r] * qoj + qoi[r] * voj;
          acc[r] = fma(a[r][c], vj, acc[r]);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < RC; ++r) part[wv * LD + lane + 64 * r] = acc[r];
    __syncthreads();
    // pb is free: the pass above was its last reader
    if (wv < RC) {
      const int i = tid;
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += part[w * LD + i];
      s *= tk;
      if (i <= k) s = 0.0;                       // finished rows
      pb[i] = s;
      const double vp = wave_sum_dpp(s * v[i]);
      if (lane == 0) sc[1 + wv] = vp;
    }
    __syncthreads();
    K = 0.0;
#pragma unroll
    for (int r = 0; r < RC; ++r) K += sc[1 + r];
    K *= 0.5 * tk;
  }
  // last 2 x 2 (or 1 x 1) block, with the update still pending
  const int k0 = n >= 2 ? n - 2 : 0;
  const double* vo = vb + ((k0 & 1) ^ 1) * LD;
#pragma unroll
  for (int c = 0; c < CC; ++c)
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      const int i = lane + 64 * r, j = wv + NW * c;
      if (j >= k0 && j < n && i >= j && i < n) {
        const double vi = vo[i], vj = vo[j];
        const double y = a[r][c] - (vi * (pb[j] - K * vj) + (pb[i] - K * vi) * vj);
        if (i == j) d[i] = y; else e[j] = y;
      }
    }
  if (tid == 0) {
    e[n - 1] = 0.0;
    if (n >= 2) tau[n - 2] = 0.0;
  }
}

// vb and pb to zero (no barrier)
__device__ __forceinline__ void tri_reg_clear(double* lds) {
  for (int i = threadIdx.x; i < 4 * TRI_REG_MAX; i += TRI_REG_THREADS) lds[TRI_REG_WAVES * TRI_REG_MAX + i] = 0.0;
}

__device__ __forceinline__ void tri_reg(const EigView& m, double* lds) {
  if (m.n < 1) return;
  const int n = m.n;
  tri_reg_clear(lds);
  __syncthreads();
  if (n <= 64) tri_reg_body<1, 4>(m.A, n, n, m.work, n, 0.0, lds);
  else if (n <= 128) tri_reg_body<2, 8>(m.A, n, n, m.work, n, 0.0, lds);
  else tri_reg_body<3, 12>(m.A, n, n, m.work, n, 0.0, lds);
}

// ---------------------------------------------------------------------------
// Step k of the reduction by workgroup w of a matrix's tri_nwg(n) (launches
// k = 0 .. n - TRI_REG_MAX - 1; tri_tail does the rest).  A launch never waits for another workgroup: every
// workgroup of a matrix recomputes the small per-step vectors itself from
// what the previous launch left in device memory (double-buffered by the
// parity of k).  Thread i owns row k + i throughout:
//   A  reflector k-1 (vbuf) and the shares of p = A v (pcol, prow) -> the
//      update q of step k-1 still pending on the trailing block; workgroup 0
//      stores reflector k-1 into column k-1 of A;
//   B  column k with the pending update -> reflector k (d, e, tau, vbuf
//      written by workgroup 0);
//   C  the workgroup's columns j = w, w + NWG, ... of the trailing block:
//      pending update applied and stored, column sums (rows i >= j) and row
//      sums (columns j < i) of A v.
// The 16
// waves (8 up to order TRI_STEP_SPLIT) form four row groups (64-row chunks h,
// h + 4, ...) by four (two) column groups, U columns a pass.  Everything a launch reads that does not depend
// on its own sums -- the vectors of A, column k and the first columns of C
// -- is loaded up front, so a launch exposes one memory latency and the three
// barriers of its two sums.
// Lanes per workgroup (at least one per row): the orders of the two classes go
// to launches of their own.
constexpr int TRI_STEP_SPLIT = 512;
constexpr int TRI_STEP_THREADS = 1024;     // orders above TRI_STEP_SPLIT
constexpr int TRI_STEP_THREADS_S = 512;    // the others
constexpr int TRI_NWG_MAX = 16;
constexpr int TRI_NWG_S = 8;
// Workgroups per matrix: by its order alone, so that a matrix gives the same
// result in any batch; the rule has to serve few matrices, where a step is
// latency and more workgroups shorten it, and many, where the card is full and
// fewer have less to repeat.  Orders up to 512 on 8 and on 4 (all stages, ms):
//   count       1            32            64            100           200
//   300     2.63  3.24    3.59  4.10    4.32  4.73    5.96  5.53    9.34  8.92
//   432     4.87  6.65    7.02  8.79    8.64  9.38   12.8  11.7    21.3  20.3
//   480     5.94  8.26    8.46 10.7    10.6  11.6    15.9  14.5    26.9  25.9
//   512     6.66  9.38    9.34 11.8    12.1  13.0    18.8  17.2    31.7  30.7
// 8 costs at most 9% (100 matrices, which fill the card one and a half times) and
// saves up to 29%; six lie between.  (200 of order 432: one workgroup per matrix
// 24.4.)  Above 512, 16 of order 816: 21.8 ms on 8 workgroups, 17.8 on 16 (before
// tri_tail).  Workgroups of 1024 lanes up to order 512 instead of 512: 100 of order
// 480 19.9 on 4 and 25.3 on 8, only one of them fits a compute unit.
__host__ __device__ inline int tri_nwg(int n) { return n <= TRI_STEP_SPLIT ? TRI_NWG_S : TRI_NWG_MAX; }
__host__ __device__ inline int tri_step_ncw(int n) { return n / tri_nwg(n) + 1; }
// (grows with n, so the largest order of a launch sizes it for all)
__host__ __device__ inline size_t tri_step_lds(int n) {
  const int nc = (n <= TRI_STEP_SPLIT ? TRI_STEP_THREADS_S : TRI_STEP_THREADS) / 256;
  return sizeof(double) * ((3 + nc) * (size_t)n + 4 * (size_t)(n / 4 + 1) + 40);
}

template <int R, int U, int NWG, int TPB>
__device__ __forceinline__ void tri_step_body(double* A, int n, int k, int w, double* work, double* lds) {
  constexpr int NC = TPB / 256;            // column groups
  double *d = work, *e = work + n, *tau = work + 2 * n;
  double* pcol = work + 3 * (long long)n;                      // [2][n]
  double* prow = work + 5 * (long long)n;                      // [2][NWG][n]
  double* vbuf = work + (5 + 2 * NWG) * (long long)n;      // [2][n]
  const int par = k & 1, opar = par ^ 1;
  const int ncw_max = tri_step_ncw(n);
  double* vo = lds;
  double* qo = lds + n;
  double* v = lds + 2 * n;
  double* prt = lds + 3 * n;                                   // [NC][n]
  double* pcl = prt + NC * n;                                  // [4][ncw_max]
  double* sc = pcl + 4 * ncw_max;                              // sums by wave, rows 0 and 1
  const int i = threadIdx.x, lane = i & 63;
  const int wv = __builtin_amdgcn_readfirstlane(i >> 6);
  const int mo = n - k, m = mo - 1;                            // rows of reflectors k-1 and k
  const bool upd = k > 0;
  double* A2 = A + (long long)(k + 1) + (long long)n * (k + 1);
  // columns of this wave in phase C: t-th is j = w + NWG (cg + NC t)
  const int h = wv & 3, cg = wv >> 2;
  const int ncw = w < m ? (m - w + NWG - 1) / NWG : 0; // columns of the workgroup
  // ---- loads that depend on nothing computed here
  const double tko = upd ? gld(tau + k - 1) : 0.0;
  double vi = 0.0, s = 0.0, ai = 0.0;
  if (i < mo) {
    ai = gld(A + (long long)(k + i) + (long long)n * k);
    if (upd) {
      vi = gld(vbuf + (long long)opar * n + i);
      s = gld(pcol + (long long)opar * n + i);
      const double* pr = prow + (long long)opar * NWG * n + i;
      double t[NWG];
#pragma unroll
      for (int q = 0; q < NWG; ++q) t[q] = gld(pr + (long long)q * n);
#pragma unroll
      for (int q = 0; q < NWG; ++q) s += t[q];
    }
  }
  double xn[U][R];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = cg + NC * (t0 + u), j = w + NWG * t;
      const double* col = A2 + (long long)n * (t < ncw ? j : 0);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int cb = 64 * (h + 4 * r);
        double a = 0.0;
        if (t < ncw && cb + 63 >= j && cb < m) {               // wave-uniform chunk test
          const int row = cb + lane;
          if (row >= j && row < m) a = gld(col + row);
        }
        xn[u][r] = a;
      }
    }
  };
  fetch(0);
  // ---- A: q = tau p - (tau / 2) (v . tau p) v of step k-1
  const double pp = tko * s;
  {
    const double t = wave_sum_dpp(vi * pp);
    if (lane == 0) sc[wv] = t;
    if (i == 0) { sc[32] = vi; sc[33] = pp; }
  }
  if (w == 0 && upd && i < mo) gst(A + (long long)(k + i) + (long long)n * (k - 1), vi);
  __syncthreads();
  double K = 0.0;
#pragma unroll
  for (int q = 0; q < TPB / 64; ++q) K += sc[q];
  K *= 0.5 * tko;
  const double qi = pp - K * vi;
  const double vo0 = sc[32], qo0 = sc[33] - K * vo0;
  if (i < mo) {
    vo[i] = vi;
    qo[i] = qi;
  }
  // ---- B: column k -> reflector k
  ai -= vi * qo0 + qi * vo0;
  {
    const double t = wave_sum_dpp(i >= 2 && i < mo ? ai * ai : 0.0);
    if (lane == 0) sc[16 + wv] = t;
    if (i == 1) sc[34] = ai;
  }
  __syncthreads();
  double a2 = 0.0;
#pragma unroll
  for (int q = 0; q < TPB / 64; ++q) a2 += sc[16 + q];
  const double x0 = sc[34];
  double beta = x0, v0 = 0.0, tk = 0.0;
  if (a2 != 0.0) {
    const double nrm = sqrt(x0 * x0 + a2);
    beta = x0 >= 0.0 ? -nrm : nrm;
    v0 = x0 - beta;
    tk = 2.0 / (v0 * v0 + a2);
  }
  if (i >= 1 && i < mo) {
    const double x = a2 == 0.0 ? 0.0 : (i == 1 ? v0 : ai);
    v[i - 1] = x;
    if (w == 0) gst(vbuf + (long long)par * n + i - 1, x);
  }
  if (w == 0 && i == 0) {
    d[k] = ai;
    e[k] = beta;
    tau[k] = tk;
  }
  __syncthreads();
  // ---- C: this workgroup's columns of the trailing block
  double vr[R], acc[R], vor[R], qor[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = 64 * (h + 4 * r) + lane;
    vr[r] = row < m ? v[row] : 0.0;
    vor[r] = row < m ? vo[row + 1] : 0.0;
    qor[r] = row < m ? qo[row + 1] : 0.0;
    acc[r] = 0.0;
  }
  for (int t0 = 0; cg + NC * t0 < ncw; t0 += U) {
    double x[U][R], sm[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r) x[u][r] = xn[u][r];
    if (cg + NC * (t0 + U) < ncw) fetch(t0 + U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = cg + NC * (t0 + u);
      const int j = t < ncw ? w + NWG * t : 0;
      const double vj = v[j], voj = vo[j + 1], qoj = qo[j + 1];
      double* col = A2 + (long long)n * j;
      sm[u] = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int cb = 64 * (h + 4 * r), row = cb + lane;
        if (t < ncw && cb + 63 >= j && cb < m) {
          if (row >= j && row < m) {
            double a = x[u][r];
            a -= vor[r] * qoj + qor[r] * voj;
            if (upd) gst(col + row, a);
            sm[u] = fma(a, vr[r], sm[u]);
            if (row > j) acc[r] = fma(a, vj, acc[r]);
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) sm[u] = wave_sum_dpp(sm[u]);
    if (lane == 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = cg + NC * (t0 + u);
        if (t < ncw) pcl[h * ncw_max + t] = sm[u];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = 64 * (h + 4 * r) + lane;
    if (row < m) prt[cg * n + row] = acc[r];
  }
  __syncthreads();
  if (i < m) {
    double t = prt[i];
#pragma unroll
    for (int q = 1; q < NC; ++q) t += prt[q * n + i];
    gst(prow + ((long long)par * NWG + w) * n + i, t);
  }
  if (i < ncw)
    gst(pcol + (long long)par * n + w + NWG * i,
        ((pcl[i] + pcl[ncw_max + i]) + pcl[2 * ncw_max + i]) + pcl[3 * ncw_max + i]);
}

template <bool WIDE>
__device__ __forceinline__ void tri_step(const EigView& m, int k, int w, double* lds) {
  if ((m.n > TRI_STEP_SPLIT) != WIDE || k >= m.n - TRI_REG_MAX || w >= tri_nwg(m.n)) return;
  if constexpr (WIDE) {
    if (m.n <= 768) tri_step_body<3, 3, 16, TRI_STEP_THREADS>(m.A, m.n, k, w, m.work, lds);
    else tri_step_body<4, 2, 16, TRI_STEP_THREADS>(m.A, m.n, k, w, m.work, lds);
  } else {
    if (m.n <= 256) tri_step_body<1, 6, TRI_NWG_S, TRI_STEP_THREADS_S>(m.A, m.n, k, w, m.work, lds);
    else tri_step_body<2, 3, TRI_NWG_S, TRI_STEP_THREADS_S>(m.A, m.n, k, w, m.work, lds);
  }
}

// The last TRI_REG_MAX rows after the launches of tri_step, in the registers of
// one workgroup, starting from the update that the last of them left pending: a
// step here takes 2.7 us, a launch there at least 7.  Measured, all stages: 32
// matrices of order 432 8.36 -> 7.23 ms, 16 of order 816 17.0 -> 16.1 ms.
__device__ __forceinline__ void tri_tail(const EigView& m, double* lds) {
  constexpr int LD = TRI_REG_MAX;
  const int n = m.n, k = n - LD, nwg = tri_nwg(n), i = threadIdx.x;   // k >= 1
  const long long opar = (k & 1) ^ 1;
  const double* pcol = m.work + 3 * (long long)n + opar * n;
  const double* prow = m.work + 5 * (long long)n + opar * nwg * n;
  const double* vbuf = m.work + (5 + 2 * nwg) * (long long)n + opar * n;
  double* vb = lds + TRI_REG_WAVES * LD;
  double* pb = vb + 2 * LD;
  double* sc = pb + 2 * LD;
  tri_reg_clear(lds);
  __syncthreads();
  const double tko = gld(m.work + 2 * (long long)n + k - 1);
  if (i < LD) {
    const double vi = gld(vbuf + i);
    double s = gld(pcol + i);
    for (int q = 0; q < nwg; ++q) s += gld(prow + (long long)q * n + i);
    const double pp = tko * s;
    vb[LD + i] = vi;
    pb[i] = pp;
    gst(m.A + (long long)(k + i) + (long long)n * (k - 1), vi);
    const double t = wave_sum_dpp(vi * pp);
    if ((i & 63) == 0) sc[1 + (i >> 6)] = t;
  }
  __syncthreads();
  const double K = 0.5 * tko * (sc[1] + sc[2] + sc[3]);
  tri_reg_body<3, 12>(m.A + (long long)k * (n + 1), n, LD, m.work + k, n, K, lds);
}

}  // namespace dg
