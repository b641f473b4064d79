// Per-element LOBPCG kernels other than the operator and the block products:
// residuals and their norms, the band kinetic energies of the Teter
// preconditioner, block orthonormalisation coefficients (CholQR / SVQB),
// the Rayleigh-Ritz step with the next search direction, and the final
// restriction + SVD truncation to ALBs (Sec. II.A after Eq. localproblem,
// Sec. II.B "Generation of the ALB functions").
//
// Small dense work (size J or 3J) runs one workgroup per element on the
// cooperative routines of small_dense.h, all FP64.
#include "common.h"
#include "small_dense.h"
#include "chol.h"
#include "tri.h"

namespace dg {

constexpr double CHOL_TOL = 1e-10;   // smallest admissible pivot of a unit-diagonal Gram
constexpr int SMALL_THREADS = 1024;
// LDS of the one-workgroup eigensolver (doubles)
constexpr int EIG_LDS = 10240;

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// R = HX - X diag(theta) into block `out_slot`; resid = ||R_j||, xhx = x_j.hx_j,
// vx = sum V x_j^2.  Work item: (element, column j).
//
// One pass over the columns, so memory should bound it; but a call can have
// fewer columns than the card has CUs, and then the loads in flight of one
// workgroup do.  Hence RESID_THREADS lanes with RESID_NP points each at a time,
// all loads ahead of the arithmetic.  Measured: 144 columns of 36x36x60 (one
// workgroup on about half of the CUs), 256 lanes with one point at a time
// 196 us, this 51 us.
constexpr int RESID_NP = 4;
extern "C" __global__ void __launch_bounds__(RESID_THREADS)
dg_resid(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
         int na, int xs, int hxs, int out_slot, int write_r) {
  constexpr int NW = RESID_THREADS / 64;
  __shared__ double red[3][NW];
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const Elem& e = E[active[ai]];
  int j = b - prefix[ai];
  const double* x = bp(e, xs) + (long long)j * e.ld;
  const double* hx = bp(e, hxs) + (long long)j * e.ld;
  double* r = bp(e, out_slot) + (long long)j * e.ld;
  const double* V = e.V;
  const double th = e.theta[j];
  const int ng = e.ng;
  double s0 = 0, s1 = 0, s2 = 0;
  for (int i0 = threadIdx.x; i0 < ng; i0 += RESID_THREADS * RESID_NP) {
    double xv[RESID_NP], hv[RESID_NP], vv[RESID_NP];
#pragma unroll
    for (int u = 0; u < RESID_NP; ++u) {
      const int i = i0 + u * RESID_THREADS, ic = i < ng ? i : i0;
      xv[u] = gld(x + ic);
      hv[u] = gld(hx + ic);
      vv[u] = gld(V + ic);
    }
#pragma unroll
    for (int u = 0; u < RESID_NP; ++u) {
      const int i = i0 + u * RESID_THREADS;
      if (i >= ng) break;
      const double rv = hv[u] - th * xv[u];
      if (write_r) gst(r + i, rv);
      s0 += rv * rv;
      s1 += xv[u] * hv[u];
      s2 += vv[u] * xv[u] * xv[u];
    }
  }
  s0 = wave_sum(s0); s1 = wave_sum(s1); s2 = wave_sum(s2);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) { red[0][w] = s0; red[1][w] = s1; red[2][w] = s2; }
  __syncthreads();
  if (threadIdx.x < 3) {
    double s = 0;
    for (int k = 0; k < NW; ++k) s += red[threadIdx.x][k];
    if (threadIdx.x == 0) e.resid[j] = sqrt(s);
    if (threadIdx.x == 1) e.xhx[j] = s;
    if (threadIdx.x == 2) e.vx[j] = s;
  }
}

// Band kinetic energy of the unit Ritz vector x_j from quantities already at
// hand: T_j = x_j^T H x_j - sum V x_j^2 - sum_p gamma_p (beta_p^T x_j)^2,
// floored at the smallest nonzero planewave energy.  One workgroup per element.
extern "C" __global__ void __launch_bounds__(256)
dg_teter_energy(Elem* __restrict__ E, const int* __restrict__ active, int na) {
  const Elem& e = E[active[blockIdx.x]];
  for (int j = threadIdx.x; j < e.J; j += 256) {
    double t = e.xhx[j] - e.vx[j];
    for (int p = 0; p < e.n_proj; ++p) {
      double b = e.projx[p + (long long)e.n_proj * j];
      t -= e.gamma[p] * b * b;
    }
    e.tkin[j] = fmax(t, e.tfloor);
  }
}

// Passes over the small matrices (order n = kJ) run on RR_NY workgroups per
// element (grid (elements, RR_NY)), by columns or by 32 x 32 tiles of the lower
// triangle: one workgroup per element spent 0.1-2 ms on each pass of an order
// 800 matrix at the latency of its few loads in flight.
constexpr int RR_NY = 64;
constexpr int SYT = 32;
struct SymTile {
  double v[SYT][SYT + 1];
};

// f(bi, bj) for this workgroup's tiles, block row bi >= block column bj.
template <class F>
__device__ __forceinline__ void for_sym_tiles(int n, F f) {
  const int nb = cdiv(n, SYT), nt = nb * (nb + 1) / 2;
  for (int q = blockIdx.y; q < nt; q += gridDim.y) {
    int bi = (int)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);
    while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
    while (bi * (bi + 1) / 2 > q) --bi;
    f(bi, q - bi * (bi + 1) / 2);
  }
}

// v[c][r] = A[br SYT + r][bc SYT + c] (256 lanes).
__device__ __forceinline__ void load_tile(SymTile& t, const double* A, int n, int br, int bc) {
  const int r = threadIdx.x % SYT, row = br * SYT + r;
#pragma unroll
  for (int c = threadIdx.x / SYT; c < SYT; c += 256 / SYT) {
    const int col = bc * SYT + c;
    t.v[c][r] = (row < n && col < n) ? gld(A + row + (long long)n * col) : 0.0;
  }
}

// f(r, c) over the entries of a tile, lanes along r.
template <class F>
__device__ __forceinline__ void for_tile(F f) {
#pragma unroll
  for (int c = threadIdx.x / SYT; c < SYT; c += 256 / SYT) f((int)(threadIdx.x % SYT), c);
}

// Orthonormalising transform of a block Y with Gram G = Y^T Y (J x J, upper
// triangle in SM_G): T = D^-1 L^-T from a Cholesky of the unit-diagonal
// D^-1 G D^-1 = L L^T (CholQR), or, if a pivot falls below CHOL_TOL, the
// eigenvalue form T = D^-1 U Lambda^-1/2 with Lambda clamped (SVQB).
// Output T in SM_T (ld J).  init = 1: a fallback marks breakdown instead;
// init = 2 (the P block of a Rayleigh-Ritz step): a failed pivot test sets
// T = 0 and counts a P drop (the step then runs on [X W] alone).
extern "C" __global__ void __launch_bounds__(SMALL_THREADS)
dg_cholqr(Elem* __restrict__ E, const int* __restrict__ active, int na, int init) {
  __shared__ double red[32];
  __shared__ double lds[CH_LDS];
  DevTeam t{red};
  const Elem& e = E[active[blockIdx.x]];
  const int n = e.J;
  double* G = sm(e, SM_G);
  double* Ls = sm(e, SM_L);
  double* Tm = sm(e, SM_T);
  double* vec = sm(e, SM_V);
  double* dm = vec + 6 * n;
  static_assert((SMALL_THREADS / 64) * SYM_TILE_LDS <= CH_LDS, "tiles of the symmetric fill");
  sym_from_upper_tiles(t, G, n, n, lds);
  for (int i = t.tid(); i < n; i += t.nt()) {
    double d = sqrt(fmax(G[i + (long long)n * i], 0.0));
    dm[i] = d > 0.0 ? d : 1.0;
  }
  t.sync();
  const int lane = t.tid() & 63, wv = t.tid() >> 6, nw = t.nt() >> 6;
  for (int j = wv; j < n; j += nw)
    for (int i = lane; i < n; i += 64)
      gst(Ls + i + (long long)n * j, gld(G + i + (long long)n * j) / (dm[i] * dm[j]));
  t.sync();
  int ok = chol_any(t, Ls, n, n, CHOL_TOL, lds);
  if (ok) {
    double* Lt = sm(e, SM_A);
    tri_inv_t_any(t, Ls, n, Lt, n, n, lds);   // Lt = L^-T
    for (int j = wv; j < n; j += nw)
      for (int i = lane; i < n; i += 64) gst(Tm + i + (long long)n * j, gld(Lt + i + (long long)n * j) / dm[i]);
    if (init == 2 && t.tid() == 0) e.fl[FL_PDROP_NOW] = 0;
    t.sync();
    return;
  }
  if (init == 2) {
    for (int p = t.tid(); p < n * n; p += t.nt()) Tm[p] = 0.0;
    if (t.tid() == 0) {
      e.fl[FL_P_DROP] += 1;
      e.fl[FL_PDROP_NOW] = 1;
    }
    t.sync();
    return;
  }
  if (t.tid() == 0) {
    if (init) e.fl[FL_BREAKDOWN] = 1;
    else e.fl[FL_W_SVQB] += 1;
  }
  // SVQB: eigen-decomposition of the scaled Gram, clamped spectrum
  for (int p = t.tid(); p < n * n; p += t.nt()) {
    int i = p % n, j = p / n;
    Ls[p] = G[p] / (dm[i] * dm[j]);
  }
  t.sync();
  double* w = vec + 7 * n;
  double* Z = sm(e, SM_Z);
  int qok = syev(t, Ls, n, n, w, Z, n, n, sm(e, SM_U), vec);
  if (!qok && t.tid() == 0) e.fl[FL_QL_FAIL] += 1;
  double lmax = w[n - 1] > 1e-300 ? w[n - 1] : 1e-300;
  for (int p = t.tid(); p < n * n; p += t.nt()) {
    int i = p % n, j = p / n;
    double l = fmax(w[j], CHOL_TOL * lmax);
    Tm[p] = Z[p] / (sqrt(l) * dm[i]);
  }
  t.sync();
}

// Rayleigh-Ritz on S = [X P W] (k blocks: 1 for the initial/final step on X,
// 2 without P, 3 with P): lowest J of Hh c = theta M c with Hh = S^T HS and
// M = S^T S (upper triangles in SM_H, SM_M, ld n = kJ).  Produces theta, the
// coefficients C (n x J) in SM_C[:, 0:J] and, for k > 1, the next search
// direction D (n x J) in SM_C[:, J:2J]: the part of S [0; C_P; C_W] that is
// M-orthogonal to S C, normalised through a scaled Cholesky of its M-Gram.
//
// Launch sequence (host: rr_step).  The per-element decisions and
// factorisations run one workgroup per element; the products of size n^3,
// n^2 J and n J^2 run on dg_sgemm over many workgroups.  Reduction paths
// (fl[FL_RR_PATH]):
//   2  the blocks of S are orthonormalised as they are built, so M = I + E;
//      when ||E||_F <= 1e-8 (and not the step on X alone) the problem is
//      reduced to first order, T = I - E/2 with T^T M T = I + O(E^2):
//      A = Hh - sym(E Hh), C = Y - E Y / 2;
//   3  when 1e-8 < ||E||_F <= 1e-4: T = M^-1/2 by its binomial series to
//      third order, T = I - E/2 + 3E^2/8 - 5E^3/16 (T^T M T = I + O(E^4),
//      <= 1e-16), A = T Hh T, C = T Y, all products on dg_sgemm;
//   0  exact reduction with a Cholesky factor of the scaled M:
//      A = L^-1 D^-1 Hh D^-1 L^-T, C = D^-1 L^-T Y (L^-T kept in SM_T);
//   1  M not numerically SPD: reduction to the eigenvectors of the scaled M
//      above CHOL_TOL times the largest, finished inside dg_rr_reduce.
// (Y, theta): lowest J eigenpairs of A from the eigensolver stages.
constexpr double NEAR_ORTHO = 1e-8;
constexpr double SERIES_ORTHO = 1e-4;
// The [X P] Gram blocks formed from small matrices are used while the
// largest residual of the element's wanted states is at least CARRY_RES;
// closer to convergence both products are formed in full over the grid
// (measured: carried blocks down to the tolerance cost the slowest elements
// of a block without guard columns extra iterations).  An element with guard
// columns carries them to the end (measured on the slab: same iterations,
// 1.5% less time).
constexpr double CARRY_RES = 3e-5;

// Lower triangles of Hh and M from their upper ones; beyond the step on X alone
// also E = M - I (SM_L) and this workgroup's share of ||E||_F^2 (SM_W0[y]).
extern "C" __global__ void __launch_bounds__(256)
dg_rr_fill(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  __shared__ SymTile th, tm;
  __shared__ double red[4];
  const Elem& e = E[active[blockIdx.x]];
  const int n = (single ? 1 : (has_p(e) ? 3 : 2)) * e.J;
  double* H = sm(e, SM_H);
  double* M = sm(e, SM_M);
  double* L = sm(e, SM_L);
  double ef = 0.0;
  for_sym_tiles(n, [&](int bi, int bj) {
    load_tile(th, H, n, bj, bi);
    load_tile(tm, M, n, bj, bi);
    __syncthreads();
    for_tile([&](int r, int c) {
      const int row = bi * SYT + r, col = bj * SYT + c;
      if (row < n && col < n && row > col) {
        const double mv = tm.v[r][c];
        gst(H + row + (long long)n * col, th.v[r][c]);
        gst(M + row + (long long)n * col, mv);
        if (!single) gst(L + row + (long long)n * col, mv);
        ef += 2.0 * mv * mv;
      }
      const int ur = bj * SYT + r, uc = bi * SYT + c;
      if (!single && ur < n && uc < n && ur <= uc) {
        const double v = tm.v[c][r] - (ur == uc ? 1.0 : 0.0);
        gst(L + ur + (long long)n * uc, v);
        if (ur == uc) ef += v * v;
      }
    });
    __syncthreads();
  });
  if (single) return;
  ef = wave_sum(ef);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ef;
  __syncthreads();
  if (threadIdx.x == 0) sm(e, SM_W0)[blockIdx.y] = (red[0] + red[1]) + (red[2] + red[3]);
}

extern "C" __global__ void __launch_bounds__(SMALL_THREADS)
dg_rr_reduce(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  __shared__ double red[32];
  __shared__ double lds[CH_LDS];
  DevTeam t{red};
  const Elem& e = E[active[blockIdx.x]];
  const int J = e.J;
  const int kb = single ? 1 : (has_p(e) ? 3 : 2);
  const int n = kb * J;
  double* H = sm(e, SM_H);
  double* M = sm(e, SM_M);
  double* A = sm(e, SM_A);
  double* Lm = sm(e, SM_L);
  double* U = sm(e, SM_U);
  double* Cm = sm(e, SM_C);
  double* Tm = sm(e, SM_T);
  double* Z = sm(e, SM_Z);
  double* vec = sm(e, SM_V);
  double* dm = vec + 6 * n;
  double* w = vec + 7 * n;
  // a step on X alone (start, final check) leaves nothing to carry
  if (single && t.tid() == 0) e.fl[FL_CARRY] = 0;
  if (!single) {
    const double* part = sm(e, SM_W0);
    double ef = 0.0;
    for (int q = 0; q < RR_NY; ++q) ef += part[q];
    ef = sqrt(ef);          // ||E||_F >= ||E||_2; E = M - I is in SM_L (dg_rr_fill)
    if (ef <= SERIES_ORTHO) {
      if (t.tid() == 0) {
        e.fl[FL_RR_PATH] = ef <= NEAR_ORTHO ? 2 : 3;
        e.fl[FL_RR_NSERIES] += 1;
      }
      return;
    }
  }
  if (t.tid() == 0 && !single) e.fl[FL_RR_NCHOL] += 1;
  for (int i = t.tid(); i < n; i += t.nt()) {
    double d = sqrt(fmax(M[i + (long long)n * i], 0.0));
    dm[i] = d > 0.0 ? d : 1.0;
  }
  t.sync();
  const int lane = t.tid() & 63, wv = t.tid() >> 6, nw = t.nt() >> 6;
  for (int j = wv; j < n; j += nw)
    for (int i = lane; i < n; i += 64) {
      const long long p = i + (long long)n * j;
      const double dd = dm[i] * dm[j];
      gst(Lm + p, gld(M + p) / dd);
      gst(A + p, gld(H + p) / dd);       // D^-1 Hh D^-1
    }
  t.sync();
  int ok = chol_any(t, Lm, n, n, CHOL_TOL, lds);
  int nk = n;
  if (ok) {
    tri_inv_t_any(t, Lm, n, Tm, n, n, lds);   // Tm = L^-T; products follow on dg_sgemm
    if (t.tid() == 0) e.fl[FL_RR_PATH] = 0;
    t.sync();
    return;
  } else {
    if (t.tid() == 0) e.fl[FL_RR_FALLBACK] += 1;
    // reduce to the eigenvectors of D^-1 M D^-1 above CHOL_TOL * max
    for (int p = t.tid(); p < n * n; p += t.nt()) {
      int i = p % n, j = p / n;
      Lm[p] = M[p] / (dm[i] * dm[j]);
    }
    t.sync();
    double* wm = vec + 8 * n;
    int qok = syev(t, Lm, n, n, wm, Z, n, n, U, vec);
    if (!qok && t.tid() == 0) e.fl[FL_QL_FAIL] += 1;
    double lmax = wm[n - 1];
    int first = n;
    for (int i = 0; i < n; ++i)
      if (wm[i] > CHOL_TOL * lmax) { first = i; break; }
    nk = n - first;
    if (nk < J) {
      if (t.tid() == 0) e.fl[FL_BREAKDOWN] = 1;
      nk = J < n ? J : n;
      first = n - nk;
    }
    // T (n x nk) = D^-1 V_k Lambda_k^-1/2
    for (int p = t.tid(); p < n * nk; p += t.nt()) {
      int i = p % n, j = p / n;
      double l = fmax(wm[first + j], 1e-300);
      Tm[p] = Z[i + (long long)n * (first + j)] / (sqrt(l) * dm[i]);
    }
    t.sync();
    gemm(t, 0, 0, n, nk, n, 1.0, H, n, Tm, n, 0.0, U, n);     // U = Hh T
    gemm(t, 1, 0, nk, nk, n, 1.0, Tm, n, U, n, 0.0, A, nk);   // A = T^T Hh T
    sym_from_upper(t, A, nk, nk);
    int q2 = syev(t, A, nk, nk, w, Z, nk, J, U, vec);
    if (!q2 && t.tid() == 0) e.fl[FL_QL_FAIL] += 1;
    gemm(t, 0, 0, n, J, nk, 1.0, Tm, n, Z, nk, 0.0, Cm, n);   // C = T Y
  }
  for (int j = t.tid(); j < J; j += t.nt()) e.theta[j] = w[j];
  if (t.tid() == 0) e.fl[FL_RR_PATH] = 1;
}

// Path 2: A = Hh - (U + U^T)/2 with U = E Hh, the lower triangle (all that
// the tridiagonalisation reads).
extern "C" __global__ void __launch_bounds__(256)
dg_rr_form(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  __shared__ SymTile tu;
  const Elem& e = E[active[blockIdx.x]];
  if (e.fl[FL_RR_PATH] != 2) return;
  const int n = (single ? 1 : (has_p(e) ? 3 : 2)) * e.J;
  const double* H = sm(e, SM_H);
  const double* U = sm(e, SM_U);
  double* A = sm(e, SM_A);
  for_sym_tiles(n, [&](int bi, int bj) {
    load_tile(tu, U, n, bj, bi);
    __syncthreads();
    for_tile([&](int r, int c) {
      const int row = bi * SYT + r, col = bj * SYT + c;
      const long long p = row + (long long)n * col;
      if (row < n && row >= col) gst(A + p, gld(H + p) - 0.5 * (gld(U + p) + tu.v[r][c]));
    });
    __syncthreads();
  });
}

// [X P] block of S^T S and S^T H S from the last step: with X' = S C and
// P' = S D, [X' P']^T [X' P'] = [C D]^T M [C D] and likewise for H, which the
// last step left in SM_MC and SM_HC.  Overwrites the leading kc x kc block of
// both products (the tiles there were not computed).
extern "C" __global__ void __launch_bounds__(256)
dg_carry_in(Elem* __restrict__ E, const int* __restrict__ active, int na) {
  const Elem& e = E[active[blockIdx.x]];
  const int kc = carried_cols(e);
  if (kc == 0) return;
  const int n = (e.fl[FL_HASP] ? 3 : 2) * e.J, ldc = 2 * e.J;
  double* M = sm(e, SM_M);
  double* H = sm(e, SM_H);
  const double* Mc = sm(e, SM_MC);
  const double* Hc = sm(e, SM_HC);
  for (int j = blockIdx.y; j < kc; j += gridDim.y)
    for (int i = threadIdx.x; i < kc; i += 256) {
      gst(M + i + (long long)n * j, gld(Mc + i + (long long)ldc * j));
      gst(H + i + (long long)n * j, gld(Hc + i + (long long)ldc * j));
    }
}

// The eigensolver of the Rayleigh-Ritz step: tridiagonalisation (tri.h: in
// registers up to order TRI_REG_MAX, else one launch per Householder step),
// then the stages of eig_split.h, for orders up to EIG_MAXN; larger orders
// stay in one workgroup (dg_rr_eig_large).

// Where the matrices of a batch are: the Rayleigh-Ritz matrices of elements
// (kind 0), the restricted Grams of elements (1), or a plain batch (2: copies
// and workspaces of dgdft_small_syev).
struct EigSrc {
  int kind;
  const Elem* E;
  const int* active;
  int single;
  double *work, *w, *Z;
  int n, k;
};

__host__ __device__ inline long long syev_stride(int n, int k) { return 2LL * n * n + 8LL * n + 6LL * n * k; }

__device__ __forceinline__ EigView eig_view(const EigSrc& s, int b) {
  EigView m{};
  if (s.kind == 2) {
    m.n = s.n;
    m.k = s.k;
    m.A = s.work + b * syev_stride(s.n, s.k);
    m.work = m.A + (long long)s.n * s.n;
    m.w = s.w + (long long)b * s.n;
    m.Z = s.Z + (long long)b * s.n * s.k;
    return m;
  }
  const Elem& e = s.E[s.active[b]];
  const int n = (s.kind == 1 || s.single ? 1 : (has_p(e) ? 3 : 2)) * e.J;
  if ((s.kind == 0 && e.fl[FL_RR_PATH] == 1) || n > EIG_MAXN) return m;
  m.n = n;
  m.k = s.kind == 1 ? e.nalb : e.J;
  m.A = sm(e, SM_A);
  m.Z = sm(e, SM_Z);
  m.w = sm(e, SM_V) + 7 * n;
  m.work = sm(e, SM_W0);       // and SM_W1, which follows it
  return m;
}

// Stage kernels: `per` workgroups per matrix (the largest of the batch needs
// them all), 2 nmax doubles of LDS and what the stage adds.
extern "C" __global__ void __launch_bounds__(EIG_BIS_THREADS)
dg_eig_bisect(EigSrc s, int per) {
  extern __shared__ double dyn[];
  __shared__ double red[32];
  eig_bisect_body(eig_view(s, blockIdx.x / per), blockIdx.x % per, dyn, red);
}

extern "C" __global__ void __launch_bounds__(EIG_INV_COLS)
dg_eig_invit(EigSrc s, int per) {
  extern __shared__ double dyn[];
  __shared__ double red[32];
  eig_invit_body(eig_view(s, blockIdx.x / per), blockIdx.x % per, dyn, red);
}

extern "C" __global__ void __launch_bounds__(EIG_CL_THREADS)
dg_eig_cluster(EigSrc s) {
  extern __shared__ double dyn[];
  __shared__ double red[32];
  eig_cluster_body(eig_view(s, blockIdx.x), dyn, red);
}

extern "C" __global__ void __launch_bounds__(EIG_BT_THREADS)
dg_eig_back(EigSrc s, int per) {
  extern __shared__ double dyn[];
  eig_back_any(eig_view(s, blockIdx.x / per), blockIdx.x % per, dyn);
}

extern "C" __global__ void __launch_bounds__(TRI_REG_THREADS)
dg_tri_reg(EigSrc s) {
  __shared__ double lds[TRI_REG_LDS];
  const EigView m = eig_view(s, blockIdx.x);
  if (m.n > TRI_REG_MAX) return;           // dg_tri_step's matrix
  tri_reg(m, lds);
}

// After the last dg_tri_step (wide) or dg_tri_step_s of a matrix.
extern "C" __global__ void __launch_bounds__(TRI_REG_THREADS)
dg_tri_tail(EigSrc s, int wide) {
  __shared__ double lds[TRI_REG_LDS];
  const EigView m = eig_view(s, blockIdx.x);
  if (m.n <= TRI_REG_MAX || (m.n > TRI_STEP_SPLIT) != (wide != 0)) return;
  tri_tail(m, lds);
}

// tri_nwg(nmax) workgroups per matrix and tri_step_lds(nmax) bytes of LDS, nmax
// the largest order of the launch's class.
extern "C" __global__ void __launch_bounds__(TRI_STEP_THREADS)
dg_tri_step(EigSrc s, int k) {
  extern __shared__ double dyn[];
  const int b = blockIdx.x / TRI_NWG_MAX;
  tri_step<true>(eig_view(s, b), k, blockIdx.x - b * TRI_NWG_MAX, dyn);
}

extern "C" __global__ void __launch_bounds__(TRI_STEP_THREADS_S)
dg_tri_step_s(EigSrc s, int k) {
  extern __shared__ double dyn[];
  const int b = blockIdx.x / TRI_NWG_S;
  tri_step<false>(eig_view(s, b), k, blockIdx.x - b * TRI_NWG_S, dyn);
}

// Orders above EIG_MAXN: the whole eigensolver in one workgroup.
extern "C" __global__ void __launch_bounds__(SMALL_THREADS)
dg_rr_eig_large(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  __shared__ double red[32];
  __shared__ double lds[EIG_LDS];
  DevTeam t{red};
  const Elem& e = E[active[blockIdx.x]];
  if (e.fl[FL_RR_PATH] == 1) return;
  const int n = (single ? 1 : (has_p(e) ? 3 : 2)) * e.J;
  if (n <= EIG_MAXN) return;
  double* vec = sm(e, SM_V);
  syev_lowest(t, sm(e, SM_A), n, n, e.J, vec + 7 * n, sm(e, SM_Z), n, sm(e, SM_W0), (int*)(vec + 10 * n), lds,
              EIG_LDS);
}

// Path 3: T = I - E/2 + 3 E^2/8 - 5 E^3/16 from E (SM_L), E^2 (SM_U) and
// E^3 (SM_A), into SM_T.
extern "C" __global__ void __launch_bounds__(256)
dg_rr_series(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  const Elem& e = E[active[blockIdx.x]];
  if (e.fl[FL_RR_PATH] != 3) return;
  const int J = e.J;
  const int n = (single ? 1 : (has_p(e) ? 3 : 2)) * J;
  const double* Em = sm(e, SM_L);
  const double* E2 = sm(e, SM_U);
  const double* E3 = sm(e, SM_A);
  double* Tm = sm(e, SM_T);
  for (int j = blockIdx.y; j < n; j += gridDim.y)
    for (int i = threadIdx.x; i < n; i += 256) {
      const long long p = i + (long long)n * j;
      gst(Tm + p, (i == j ? 1.0 : 0.0) - 0.5 * gld(Em + p) + 0.375 * gld(E2 + p) - 0.3125 * gld(E3 + p));
    }
}

// Path 2: C = Y (the E Y / 2 correction follows on dg_sgemm).
extern "C" __global__ void __launch_bounds__(256)
dg_rr_cinit(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  const Elem& e = E[active[blockIdx.x]];
  if (e.fl[FL_RR_PATH] != 2) return;
  const int J = e.J;
  const int n = (single ? 1 : (has_p(e) ? 3 : 2)) * J;
  const double* Z = sm(e, SM_Z);
  double* Cm = sm(e, SM_C);
  for (int p = blockIdx.y * 256 + threadIdx.x; p < n * J; p += gridDim.y * 256) gst(Cm + p, gld(Z + p));
}

// Ritz values; path 0: undo the diagonal scaling of C.
extern "C" __global__ void __launch_bounds__(256)
dg_rr_post(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  const Elem& e = E[active[blockIdx.x]];
  const int J = e.J;
  const int kb = single ? 1 : (has_p(e) ? 3 : 2);
  const int n = kb * J;
  const int path = e.fl[FL_RR_PATH];
  double* Cm = sm(e, SM_C);
  double* vec = sm(e, SM_V);
  const double* dm = vec + 6 * n;
  const double* w = vec + 7 * n;
  if (path == 0)
    for (int j = blockIdx.y; j < J; j += gridDim.y)
      for (int i = threadIdx.x; i < n; i += 256) Cm[i + (long long)n * j] /= dm[i];
  if (blockIdx.y > 0) return;
  if (path != 1)
    for (int j = threadIdx.x; j < J; j += 256) e.theta[j] = w[j];
  if (kb == 1 && threadIdx.x == 0) e.fl[FL_HASP_NEXT] = 0;
}

// ---------------------------------------------------------------------------
// With guard columns, the basis of a LOBPCG step is S = [X P W] with X the
// Ritz vectors, W the preconditioned residuals made orthonormal and
// orthogonal to X, and P the previous step's search direction in the form of
// Knyazev's method,
// P' = [P W] [C_P; C_W] (formed together with X' = X C_X + P' in one pass
// over the blocks), which is neither normalised nor orthogonal to X.  Before
// the Rayleigh-Ritz reduction the P block is orthonormalised against
// Q = [X W] in small space: P~ = (P - Q Z) T_P with Z = (2I - M_QQ) M_QP,
// the projection coefficients M_QQ^-1 M_QP to first order in M_QQ - I (Q is
// orthonormal to FP64 rounding; the mixed form, whose FP32 products leave
// it orthonormal only to ~1e-6, keeps the orthonormalised direction), T_P
// from a scaled Cholesky of S_P = M_PP - M_QP^T Z, i.e.
// S~ = S B with B the identity except for its P column block
// B_P = [-Z_X T_P; T_P; -Z_W T_P]; then Hh~ = B^T Hh B, M~ = B^T M B (close
// to I), the Rayleigh-Ritz step gives C~, and C = B C~ in the basis S.  The
// span of S, hence the step, is that of the method with an orthonormalised
// search direction; only its representation differs.  (Without guard
// columns the slowest wanted states leave this P nearly dependent on [X W]
// near convergence, and so do residuals well below 1e-7 with guards: S_P
// then loses P's independent part to cancellation and P is dropped step
// after step.  Such blocks keep the orthonormalised direction, dg_rr_dchol,
// and project W against [X P].)

// Block copies inside the small workspace.  Dimension codes as for dg_sgemm
// (0: n = kJ, 1: J, 2: 2J, 3: n - J); offsets in units of J (-1: the last
// block, k - 1).  mode 0: D = alpha S, 1: D = alpha S^T, 2: D = alpha I,
// 3: D = 0.  gate as dg_sgemm's gate_carry.
struct CpArgs {
  int ms, rs, cs, ls;
  int md, rd, cd, ld;
  int dr, dc;
  double alpha;
  int mode;
  int gate;
  int single;
};

extern "C" __global__ void __launch_bounds__(256)
dg_small_copy(Elem* __restrict__ E, const int* __restrict__ active, int na, CpArgs a) {
  const Elem& e = E[active[blockIdx.x]];
  if ((a.gate & 1) && carried_cols(e) == 0) return;
  if ((a.gate & 2) && !has_p(e)) return;
  const int J = e.J;
  const int kb = a.single ? 1 : (has_p(e) ? 3 : 2);
  const int n = kb * J;
  const int R = sg_dim(a.dr, n, J), Cn = sg_dim(a.dc, n, J);
  const int lds = sg_dim(a.ls, n, J), ldd = sg_dim(a.ld, n, J);
  auto off = [&](int c) { return (c >= 0 ? c : kb - 1) * J; };
  const double* S = sm(e, a.ms) + (long long)off(a.cs) * lds + off(a.rs);
  double* D = sm(e, a.md) + (long long)off(a.cd) * ldd + off(a.rd);
  for (int j = blockIdx.y; j < Cn; j += gridDim.y)
    for (int i = threadIdx.x; i < R; i += 256) {
      double v;
      switch (a.mode) {
        case 0: v = gld(S + i + (long long)lds * j); break;
        case 1: v = gld(S + j + (long long)lds * i); break;
        case 2: v = i == j ? 1.0 : 0.0; break;
        default: v = 0.0;
      }
      gst(D + i + (long long)ldd * j, a.alpha * v);
    }
}

// Start of the Rayleigh-Ritz step: full symmetric S^T S and S^T H S from
// their upper triangles, kept as formed in SM_MO / SM_HO (the carried blocks
// of the next step are taken from them); with P, M_PP into SM_G (ld J) as the
// start of its Schur complement.
extern "C" __global__ void __launch_bounds__(256)
dg_rr_prep(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  __shared__ SymTile th, tm;
  const Elem& e = E[active[blockIdx.x]];
  const int J = e.J;
  const bool p3 = has_p(e);
  const int n = (p3 ? 3 : 2) * J;
  double* M = sm(e, SM_M);
  double* H = sm(e, SM_H);
  double* Mo = sm(e, SM_MO);
  double* Ho = sm(e, SM_HO);
  double* G = sm(e, SM_G);
  for_sym_tiles(n, [&](int bi, int bj) {
    load_tile(th, H, n, bj, bi);
    load_tile(tm, M, n, bj, bi);
    __syncthreads();
    for_tile([&](int r, int c) {
      // lower entry (row, col) from the transposed tile
      const int row = bi * SYT + r, col = bj * SYT + c;
      if (row < n && col < row) {
        const long long p = row + (long long)n * col;
        const double hv = th.v[r][c], mv = tm.v[r][c];
        gst(H + p, hv);
        gst(Ho + p, hv);
        gst(M + p, mv);
        gst(Mo + p, mv);
        if (p3 && col >= J && row < 2 * J) gst(G + (row - J) + J * (col - J), mv);
      }
      // upper entry
      const int ur = bj * SYT + r, uc = bi * SYT + c;
      if (uc < n && ur <= uc) {
        const long long p = ur + (long long)n * uc;
        const double mv = tm.v[c][r];
        gst(Ho + p, th.v[c][r]);
        gst(Mo + p, mv);
        if (p3 && ur >= J && uc < 2 * J) gst(G + (ur - J) + J * (uc - J), mv);
      }
    });
    __syncthreads();
  });
}

// P column block of B^T Hh B and B^T M B: from U_H = Hh B_P (SM_U, n x J),
// B_P^T U_H (SM_A, J x J), U_M = M B_P (SM_Z) and B_P^T U_M (SM_W0), write
// the upper triangles of Hh and M (elements with P): the X-P block, the P-W
// block (transposed, by tiles) and the P-P block; dg_rr_fill follows.
// When the step dropped P (B_P = 0), the P-P blocks become M = I and
// Hh = sigma I with no coupling, sigma = 2 max_i |Hh_ii| + 1 over the X and W
// rows: every Ritz value of [X W] that the step keeps lies below sigma (the
// J-th is at most theta_J, an X diagonal entry, by interlacing), so the
// lowest J eigenpairs are those of [X W] with zero P rows, and M stays
// nearly the identity instead of singular.
extern "C" __global__ void __launch_bounds__(256)
dg_rr_pscatter(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  __shared__ double red[4];
  __shared__ SymTile th, tm;
  const Elem& e = E[active[blockIdx.x]];
  if (!has_p(e)) return;
  const int J = e.J, n = 3 * J;
  double* H = sm(e, SM_H);
  double* M = sm(e, SM_M);
  const double* Uh = sm(e, SM_U);
  const double* Um = sm(e, SM_Z);
  const double* Hpp = sm(e, SM_A);
  const double* Mpp = sm(e, SM_W0);
  const bool dropped = e.fl[FL_PDROP_NOW] != 0;
  double sigma = 0.0;
  if (dropped) {
    double hm = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x)
      if (i < J || i >= 2 * J) hm = fmax(hm, fabs(H[i + (long long)n * i]));
    for (int o = 32; o > 0; o >>= 1) hm = fmax(hm, __shfl_xor(hm, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = hm;
    __syncthreads();
    sigma = 2.0 * fmax(fmax(red[0], red[1]), fmax(red[2], red[3])) + 1.0;
  }
  for (int j = blockIdx.y; j < J; j += gridDim.y) {
    const long long c = (long long)n * (J + j);
    for (int i = threadIdx.x; i < J; i += 256) {
      gst(H + i + c, gld(Uh + i + (long long)n * j));
      gst(M + i + c, gld(Um + i + (long long)n * j));
      if (i <= j) {
        gst(H + (J + i) + c, dropped ? (i == j ? sigma : 0.0) : gld(Hpp + i + (long long)J * j));
        gst(M + (J + i) + c, dropped ? (i == j ? 1.0 : 0.0) : gld(Mpp + i + (long long)J * j));
      }
    }
  }
  // rows 2J + i of U -> H[J + j][2J + i]
  const int nb = cdiv(J, SYT);
  for (int q = blockIdx.y; q < nb * nb; q += gridDim.y) {
    const int i0 = (q % nb) * SYT, j0 = (q / nb) * SYT;
    for_tile([&](int r, int c) {
      const bool in = i0 + r < J && j0 + c < J;
      const long long p = (2 * J + i0 + r) + (long long)n * (j0 + c);
      th.v[c][r] = in ? gld(Uh + p) : 0.0;
      tm.v[c][r] = in ? gld(Um + p) : 0.0;
    });
    __syncthreads();
    for_tile([&](int r, int c) {
      if (j0 + r < J && i0 + c < J) {
        const long long p = (J + j0 + r) + (long long)n * (2 * J + i0 + c);
        gst(H + p, th.v[r][c]);
        gst(M + p, tm.v[r][c]);
      }
    });
    __syncthreads();
  }
}

// End of the Rayleigh-Ritz step: E = C with the X rows zeroed next to C in
// SM_C (the coefficients of the next search direction P' = S E = [P W] C_PW),
// P present in the next step, and whether its [X P] Gram blocks are carried:
// while the largest residual of the wanted states is at least CARRY_RES, or
// always with guard columns.
//
// w_dir (the solver): a step on [X W] takes P' = W, E = [0; I].  C_W is square
// there, so W C_W and W span the same space, but the columns of W are
// orthonormal while those of W C_W are nearly dependent (C_W carries the spread
// of H on W): the next step's Schur complement of the P block then had
// eigenvalues down to 6e-9 of its scaled diagonal, and rounding in S^T S and
// S^T H S grew by their reciprocal.  Measured on 36x36x60 with 144 columns, ALBs
// after three iterations against a Householder-orthonormalised form of the same
// iteration: smallest eigenvalue 5.7e-9 -> 5.1e-4, worst element 5e-10 .. 9e-10
// -> 4e-12.
extern "C" __global__ void __launch_bounds__(256)
dg_rr_e(Elem* __restrict__ E, const int* __restrict__ active, int na, int w_dir) {
  __shared__ double red[4];
  const Elem& e = E[active[blockIdx.x]];
  const int J = e.J;
  const int n = (has_p(e) ? 3 : 2) * J;
  const bool keep_w = w_dir && !has_p(e);
  double* Cm = sm(e, SM_C);
  for (int j = blockIdx.y; j < J; j += gridDim.y)
    for (int i = threadIdx.x; i < n; i += 256) {
      const double c = gld(Cm + i + (long long)n * j);
      gst(Cm + i + (long long)n * (J + j), i < J ? 0.0 : !keep_w ? c : i - J == j ? 1.0 : 0.0);
    }
  if (blockIdx.y > 0) return;
  double rmax = 0.0;
  for (int i = threadIdx.x; i < e.jc; i += blockDim.x) rmax = fmax(rmax, e.resid[i]);
  for (int o = 32; o > 0; o >>= 1) rmax = fmax(rmax, __shfl_xor(rmax, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = rmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double r = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    const bool carry = r >= CARRY_RES || e.jc < J;
    e.fl[FL_HASP_NEXT] = 1;
    e.fl[FL_CARRY] = carry ? 2 * J : 0;
  }
}

// P' = W and H P' = H W of such a step (see dg_rr_e): blocks w -> pn, hw -> hpn,
// over what the update product left there.  A pass of its own: as a branch of
// the update kernel it took registers from every product (2306 -> 2370 ms of the
// updates of 200 uneven elements; this pass runs once per solve, 0.2 ms for four
// elements of 36x36x60 with 144 columns).  Work item (element, column).
extern "C" __global__ void __launch_bounds__(256)
dg_keep_w(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix, int na, int w,
          int pn, int hw, int hpn) {
  const int ai = find_elem(prefix, na, blockIdx.x);
  const Elem& e = E[active[ai]];
  const long long c = (long long)(blockIdx.x - prefix[ai]) * e.ld;
  const double *x = bp(e, w) + c, *hx = bp(e, hw) + c;
  double *y = bp(e, pn) + c, *hy = bp(e, hpn) + c;
  for (int i0 = threadIdx.x; i0 < e.ng; i0 += 4 * 256) {
    double a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(i0 + u * 256, e.ng - 1);
      a[u] = gld(x + i);
      b[u] = gld(hx + i);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * 256;
      if (i < e.ng) {
        gst(y + i, a[u]);
        gst(hy + i, b[u]);
      }
    }
  }
}

// Orthonormalised form of the next search direction (blocks without guard
// columns): after dg_sgemm formed A = D^T M D (J x J) for D = E - C (C^T M E)
// with E = C with its X rows zeroed (SM_Z): scaled Cholesky of A; D <- D Dg^-1
// with L^-T kept in SM_L for the final product D L^-T.  If it breaks, P is
// dropped for one iteration.
extern "C" __global__ void __launch_bounds__(SMALL_THREADS)
dg_rr_dchol(Elem* __restrict__ E, const int* __restrict__ active, int na, int single) {
  __shared__ double red[32];
  __shared__ double lds[CH_LDS];
  DevTeam t{red};
  const Elem& e = E[active[blockIdx.x]];
  const int J = e.J;
  const int n = (has_p(e) ? 3 : 2) * J;
  double* A = sm(e, SM_A);
  double* Lm = sm(e, SM_L);
  double* Ez = sm(e, SM_Z);
  double* Cm = sm(e, SM_C);
  double* Dn = Cm + (long long)n * J;
  double* dm = sm(e, SM_V) + 6 * n;
  for (int p = t.tid(); p < J * J; p += t.nt()) {
    int i = p % J, j = p / J;
    if (i > j) A[p] = A[j + (long long)J * i];
  }
  t.sync();
  for (int i = t.tid(); i < J; i += t.nt()) dm[i] = sqrt(fmax(A[i + (long long)J * i], 0.0));
  t.sync();
  int dpos = 1;
  for (int i = 0; i < J; ++i) dpos &= dm[i] > 0.0;
  int pok = 0;
  if (dpos) {
    for (int p = t.tid(); p < J * J; p += t.nt()) {
      int i = p % J, j = p / J;
      A[p] /= dm[i] * dm[j];
    }
    t.sync();
    pok = chol_any(t, A, J, J, CHOL_TOL, lds);
  }
  double rmax = 0.0;
  for (int i = t.tid(); i < e.jc; i += t.nt()) rmax = fmax(rmax, e.resid[i]);
  const bool carry = t.maxv(rmax) >= CARRY_RES || e.jc < J;
  if (pok) {
    tri_inv_t_any(t, A, J, Lm, J, J, lds);                                   // Lm = L^-T
    for (int p = t.tid(); p < n * J; p += t.nt()) Ez[p] /= dm[p / n];
    if (t.tid() == 0) { e.fl[FL_HASP_NEXT] = 1; e.fl[FL_CARRY] = carry ? 2 * J : 0; }
  } else {
    for (int p = t.tid(); p < n * J; p += t.nt()) Dn[p] = 0.0;
    if (t.tid() == 0) { e.fl[FL_HASP_NEXT] = 0; e.fl[FL_P_DROP] += 1; e.fl[FL_CARRY] = carry ? J : 0; }
  }
  t.sync();
}

// End of an iteration: next buffers become current, P presence follows the
// decision of the last Rayleigh-Ritz step.
extern "C" __global__ void dg_advance(Elem* __restrict__ E, const int* __restrict__ active, int na) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < na) {
    const Elem& e = E[active[i]];
    e.fl[FL_HASP] = e.fl[FL_HASP_NEXT];
    e.fl[FL_PAR] ^= 1;
  }
}

// Rows of the restriction box E_K of column j of block `src` into block `dst`
// (rows 0..N_E-1).  Work item (element, column).
extern "C" __global__ void __launch_bounds__(256)
dg_gather_box(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
              int na, int src, int dst) {
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const Elem& e = E[active[ai]];
  int j = b - prefix[ai];
  int b1 = e.hi[0] - e.lo[0], b2 = e.hi[1] - e.lo[1];
  const double* x = bp(e, src) + (long long)j * e.ld;
  double* y = bp(e, dst) + (long long)j * e.ld;
  if (j >= e.jc) {   // guard columns take no part in the ALBs
    for (int r = threadIdx.x; r < e.ne; r += 256) y[r] = 0.0;
    return;
  }
  for (int r = threadIdx.x; r < e.ne; r += 256) {
    int i = r % b1, q = r / b1;
    int jj = q % b2, kk = q / b2;
    y[r] = x[(e.lo[0] + i) + e.n1 * ((e.lo[1] + jj) + e.n2 * (e.lo[2] + kk))];
  }
}

// SVD truncation through the Gram of the restricted unit eigenvectors:
// G = Psi_E^T Psi_E = V S^2 V^T (SM_G, upper); the n_alb largest give
// sigma (descending) and T = V S^-1 / sqrt(dV) (J x n_alb, SM_T), so that
// Psi_E T are the ALBs in the dV sum phi^2 = 1 normalisation.  The n_alb
// largest eigenpairs of G are the lowest of -G, from the Rayleigh-Ritz
// eigensolver (all of it here above order EIG_MAXN), then dg_alb_coeffs.
extern "C" __global__ void __launch_bounds__(SMALL_THREADS)
dg_alb_matrix(Elem* __restrict__ E, const int* __restrict__ active, int na) {
  __shared__ double red[32];
  __shared__ double lds[EIG_LDS];
  DevTeam t{red};
  const Elem& e = E[active[blockIdx.x]];
  const int n = e.J;
  double* G = sm(e, SM_G);
  double* A = sm(e, SM_A);
  double* vec = sm(e, SM_V);
  sym_from_upper(t, G, n, n);
  for (int p = t.tid(); p < n * n; p += t.nt()) A[p] = -G[p];
  t.sync();
  if (n > EIG_MAXN)
    syev_lowest(t, A, n, n, e.nalb, vec + 7 * n, sm(e, SM_Z), n, sm(e, SM_W0), (int*)(vec + 10 * n), lds,
                EIG_LDS);
}

extern "C" __global__ void __launch_bounds__(256)
dg_alb_coeffs(Elem* __restrict__ E, const int* __restrict__ active, int na, double* sigma) {
  const Elem& e = E[active[blockIdx.x]];
  const int n = e.J, na_ = e.nalb;
  const double* Z = sm(e, SM_Z);
  const double* w = sm(e, SM_V) + 7 * n;
  double* Tm = sm(e, SM_T);
  const double isdv = 1.0 / sqrt(e.dv);
  for (int p = threadIdx.x; p < n * na_; p += 256) {
    int i = p % n, c = p / n;
    double s = sqrt(fmax(-w[c], 0.0));
    Tm[p] = s > 0.0 ? Z[i + (long long)n * c] * isdv / s : 0.0;
  }
  for (int c = threadIdx.x; c < na_; c += 256) sigma[e.off_nalb + c] = sqrt(fmax(-w[c], 0.0));
}

// ALB column c of block `src` (rows 0..N_E-1) -> output, sign such that the
// largest-magnitude entry is positive.  Work item (element, ALB).
extern "C" __global__ void __launch_bounds__(256)
dg_pack_albs(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
             int na, int src, double* out) {
  __shared__ double bv[4];
  __shared__ int bi[4];
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const Elem& e = E[active[ai]];
  int c = b - prefix[ai];
  const double* x = bp(e, src) + (long long)c * e.ld;
  double best = -1.0;
  int bidx = 0x7fffffff;
  for (int r = threadIdx.x; r < e.ne; r += 256) {
    double a = fabs(x[r]);
    if (a > best) { best = a; bidx = r; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    double ob = __shfl_xor(best, o, 64);
    int oi = __shfl_xor(bidx, o, 64);
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) { bv[w] = best; bi[w] = bidx; }
  __syncthreads();
  double gb = bv[0];
  int gi = bi[0];
  for (int k = 1; k < 4; ++k)
    if (bv[k] > gb || (bv[k] == gb && bi[k] < gi)) { gb = bv[k]; gi = bi[k]; }
  double sgn = (gi < e.ne && x[gi] < 0.0) ? -1.0 : 1.0;
  double* y = out + e.off_alb + (long long)c * e.ne;
  for (int r = threadIdx.x; r < e.ne; r += 256) y[r] = sgn * x[r];
}

// Eigenpairs to the output: eigvals, eigvecs = X / sqrt(dV) (psi
// normalisation of Eq. localproblem).  Work item (element, column).
extern "C" __global__ void __launch_bounds__(256)
dg_pack_eig(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
            int na, int xs, double* vals, double* vecs) {
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const Elem& e = E[active[ai]];
  int j = b - prefix[ai];
  if (threadIdx.x == 0) vals[e.off_j + j] = e.theta[j];
  if (!vecs) return;
  const double s = 1.0 / sqrt(e.dv);
  const double* x = bp(e, xs) + (long long)j * e.ld;
  double* y = vecs + e.off_ngj + (long long)j * e.ng;
  for (int r = threadIdx.x; r < e.ng; r += 256) y[r] = s * x[r];
}

// Copy a batch-concatenated input (rows per element = N_g, J columns) into
// block `dst` of every element, scaled by `scale`.  Work item (element, column).
extern "C" __global__ void __launch_bounds__(256)
dg_load_block(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
              int na, const double* src, int dst, double scale) {
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const Elem& e = E[active[ai]];
  int j = b - prefix[ai];
  const double* x = src + e.off_ngj + (long long)j * e.ng;
  double* y = bp(e, dst) + (long long)j * e.ld;
  for (int r = threadIdx.x; r < e.ng; r += 256) y[r] = scale * x[r];
}

// Seeded N(0,1) start block, drawn when the caller gives none: entry pairs
// (2q, 2q+1) of column j of batch element e come from Philox4x32-10 (Salmon,
// Moraes, Dror, Shaw, SC 2011) at counter (q, j, e, 0) and key (seed mod
// 2^32, seed div 2^32): its outputs w0..w3 give the 53-bit uniforms
// u1 = (w0 2^21 + w1 >> 11) 2^-53 and u2 from (w2, w3), and the Box-Muller
// transform gives r cos(2 pi u2), r sin(2 pi u2) with r = sqrt(-2 ln(1 - u1)).
__device__ __forceinline__ void philox4x32_10(unsigned x[4], unsigned k0, unsigned k1) {
  for (int r = 0; r < 10; ++r) {
    const unsigned hi0 = __umulhi(0xD2511F53u, x[0]), lo0 = 0xD2511F53u * x[0];
    const unsigned hi1 = __umulhi(0xCD9E8D57u, x[2]), lo1 = 0xCD9E8D57u * x[2];
    const unsigned y0 = hi1 ^ x[1] ^ k0, y2 = hi0 ^ x[3] ^ k1;
    x[0] = y0; x[1] = lo1; x[2] = y2; x[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

__device__ __forceinline__ double uniform53(unsigned hi, unsigned lo) {
  const unsigned long long m = ((unsigned long long)hi << 21) | (unsigned long long)(lo >> 11);
  return (double)m * 0x1p-53;
}

// Work item (element, column j); writes the element's column j of block dst
// or, if out is non-NULL, of the batch array out (layout of X0).
extern "C" __global__ void __launch_bounds__(256)
dg_random_start(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
                int na, unsigned seed_lo, unsigned seed_hi, int dst, double* out) {
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const int elem = active[ai];
  const Elem& e = E[elem];
  int j = b - prefix[ai];
  double* y = out ? out + e.off_ngj + (long long)j * e.ng : bp(e, dst) + (long long)j * e.ld;
  const int nq = (e.ng + 1) / 2;
  for (int q = threadIdx.x; q < nq; q += 256) {
    unsigned x[4] = {(unsigned)q, (unsigned)j, (unsigned)elem, 0u};
    philox4x32_10(x, seed_lo, seed_hi);
    const double u1 = uniform53(x[0], x[1]), u2 = uniform53(x[2], x[3]);
    const double r = sqrt(-2.0 * log1p(-u1));
    double sn, cs;
    sincospi(2.0 * u2, &sn, &cs);
    y[2 * q] = r * cs;
    if (2 * q + 1 < e.ng) y[2 * q + 1] = r * sn;
  }
}

// Any bitwise difference between the projector arrays (gamma, ptr, idx, val)
// and the copies of the ones last laid out sets *flag.
extern "C" __global__ void __launch_bounds__(256)
dg_kb_differs(const double* __restrict__ g, const double* __restrict__ gc, long long np,
              const long long* __restrict__ p, const long long* __restrict__ pc,
              const int* __restrict__ ix, const int* __restrict__ ixc, const double* __restrict__ v,
              const double* __restrict__ vc, long long nnz, int* flag) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long stride = (long long)gridDim.x * 256;
  int d = 0;
  for (long long k = i; k < np; k += stride) d |= __double_as_longlong(g[k]) != __double_as_longlong(gc[k]);
  for (long long k = i; k <= np; k += stride) d |= p[k] != pc[k];
  for (long long k = i; k < nnz; k += stride)
    d |= (ix[k] != ixc[k]) | (__double_as_longlong(v[k]) != __double_as_longlong(vc[k]));
  if (d) atomicOr(flag, 1);
}

// The user slots of one element (one lane).
extern "C" __global__ void dg_bind_user(Elem* e, double* a, double* b, double* c) {
  e->blk[S_U0] = a;
  e->blk[S_U1] = b;
  e->blk[S_U2] = c;
}

// Any non-finite value in a[0..n) sets *flag.
extern "C" __global__ void __launch_bounds__(256)
dg_check_finite(const double* __restrict__ a, long long n, int* flag) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  long long stride = (long long)gridDim.x * 256;
  int bad = 0;
  for (; i < n; i += stride) bad |= !isfinite(a[i]);
  if (bad) atomicOr(flag, 1);
}

}  // namespace dg

namespace dg {
// Batched symmetric eigensolver for tests: matrix b of A (n x n, upper
// triangle read) -> w[b*n ..] ascending, Z[b*n*k ..] first k eigenvectors.
// method 0 up to order SYEV_TINY or above EIG_MAXN: Householder + bisection +
// inverse iteration (lowest k only); method 1: Householder + implicit QL on the whole spectrum.
extern "C" __global__ void __launch_bounds__(SMALL_THREADS)
dg_syev_batch(const double* __restrict__ A, double* w, double* Z, int n, int k, double* work,
              int method) {
  __shared__ double red[32];
  __shared__ double lds[EIG_LDS];
  DevTeam t{red};
  long long b = blockIdx.x;
  double* Aw = work + b * syev_stride(n, k);
  double* U = Aw + (long long)n * n;
  double* vec = U + (long long)n * n;
  copy_mat(t, A + b * n * n, n, Aw, n, n, n);
  sym_from_upper(t, Aw, n, n);
  if (method == 1) {
    syev(t, Aw, n, n, w + b * n, Z + b * n * k, n, k, U, vec);
  } else {
    syev_lowest(t, Aw, n, n, k, w + b * n, Z + b * n * k, n, U, (int*)vec, lds, EIG_LDS);
  }
}

// Method 0 for orders above SYEV_TINY up to EIG_MAXN: the lower triangle of each matrix's copy from
// its upper one, in 32 x 32 tiles through LDS (grid (matrices, tiles)),
// then the tridiagonalisation and the stages of eig_split.h.
constexpr int SYEV_COPY_TILE = 32;
// Orders up to SYEV_TINY stay in dg_syev_batch: six launches against one.
// Measured, 4 matrices of order 1, 3, 4, 5: 47, 55, 58, 61 us in stages; 28, 48,
// 56, 74 in one launch.
constexpr int SYEV_TINY = 4;
extern "C" __global__ void __launch_bounds__(256)
dg_syev_batch_copy(const double* __restrict__ A, int n, int k, double* work) {
  constexpr int TS = SYEV_COPY_TILE;
  __shared__ double tile[TS][TS + 1];
  const int nb = cdiv(n, TS);
  const int q = blockIdx.y, bi = q % nb, bj = q / nb;
  if (bj > bi) return;
  const long long b = blockIdx.x;
  const double* S = A + b * n * n;
  double* Aw = work + b * syev_stride(n, k);
  const int r = threadIdx.x % TS, c0 = threadIdx.x / TS;
#pragma unroll
  for (int c = c0; c < TS; c += 256 / TS) {
    const int row = bj * TS + r, col = bi * TS + c;
    tile[c][r] = (row < n && col < n) ? gld(S + row + (long long)n * col) : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int c = c0; c < TS; c += 256 / TS) {
    const int row = bi * TS + r, col = bj * TS + c;
    if (row < n && col <= row) gst(Aw + row + (long long)n * col, tile[r][c]);
  }
}

}  // namespace dg
