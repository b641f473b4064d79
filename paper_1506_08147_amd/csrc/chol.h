// Cholesky factor and transposed triangular inverse of one symmetric matrix
// by one workgroup of 1024 lanes, in blocks of 16 columns on the matrix cores
// (v_mfma_f64_16x16x4f64; accumulator register r of lane l is entry
// [4 r + l / 16][l % 16], operand lane l is [l % 16][l / 16] of A and
// [l / 16][l % 16] of B).
//
// Column by column these were bound by latency: three barriers and a pass of
// the trailing block through global memory per column.  In blocks of 16 there
// is a sixteenth of both, and the n^3 / 3 flops of each run on the matrix
// cores (0.3 TFLOP/s per compute unit).
#pragma once
#include "eig_split.h"

namespace dg {

constexpr int CH_B = 16;                   // block
// below, column by column: a block always takes its 16 steps.  Measured,
// orthonormalisation of order 1, 4, 8, 12: 70, 84, 85, 87 us in blocks, 61, 79,
// 86, 92 column by column.
constexpr int CH_MINN = 8;
constexpr int CH_MAXN = 832;               // one panel row per lane, panel in LDS
constexpr int CH_LDX = CH_B + 1;           // panel row stride (conflict-free fragment reads)
constexpr int CH_THREADS = 1024;
// panel (or the 16 rows of L of the inverse), diagonal block, its reciprocals, flag
constexpr int CH_PANEL = CH_MAXN * CH_LDX;
constexpr int CH_LDS = CH_PANEL + CH_B * CH_LDX + CH_B + 2;

typedef double ch_acc __attribute__((ext_vector_type(4)));

// Value of lane C of each group of 16 lanes (DPP row_newbcast).
template <int C>
__device__ __forceinline__ double row_bcast(double x) {
  return dpp_mov<0x150 + C>(x);
}

// Columns Q, Q + 1, .. 15 of the update by column C.
template <int C, int Q>
__device__ __forceinline__ void chol16_row(double (&a)[CH_B]) {
  if constexpr (Q < CH_B) {
    a[Q] = fma(-a[C], row_bcast<Q>(a[C]), a[Q]);
    chol16_row<C, Q + 1>(a);
  }
}

// Steps C, C + 1, .. 15 of the Cholesky factor of a 16 x 16 block, row l of it
// in lane l of 16: a[c] becomes L[l][c], rinv[c] its reciprocal diagonal.
template <int C>
__device__ __forceinline__ void chol16(double (&a)[CH_B], double (&rinv)[CH_B], int lane, int kb, double tol,
                                       int& ok) {
  if constexpr (C < CH_B) {
    double p = row_bcast<C>(a[C]);
    if (C < kb && !(p > tol)) ok = 0;
    if (!(p > 0.0)) p = 1.0;               // only after a failed pivot
    const double d = sqrt(p), r = 1.0 / d;
    rinv[C] = r;
    a[C] = lane == C ? d : a[C] * r;
    chol16_row<C, C + 1>(a);
    chol16<C + 1>(a, rinv, lane, kb, tol, ok);
  }
}

// In-place Cholesky of the lower triangle of A (n <= CH_MAXN); 0 if a pivot
// is not above tol (the lower triangle is then partly overwritten).  lds:
// CH_LDS doubles.
template <class T>
__device__ int chol_blocked(T& t, double* A, int lda, int n, double tol, double* lds) {
  double* Xs = lds;                        // panel rows, CH_LDX apart
  double* Ld = lds + CH_PANEL;             // diagonal block, row c at c CH_LDX
  double* rv = Ld + CH_B * CH_LDX;         // reciprocals of its diagonal
  double* okp = rv + CH_B;
  const int tid = t.tid(), lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = t.nt() >> 6;
  const int l16 = lane & 15, g16 = lane >> 4;
  for (int k0 = 0; k0 < n; k0 += CH_B) {
    const int kb = min(CH_B, n - k0), i = k0 + CH_B + tid;
    // panel row of this lane: in flight while wave 0 factors the diagonal block
    double x[CH_B];
#pragma unroll
    for (int c = 0; c < CH_B; ++c) x[c] = i < n ? gld(A + i + (long long)lda * (k0 + c)) : 0.0;
    if (wv == 0) {
      double a[CH_B], rinv[CH_B];
#pragma unroll
      for (int c = 0; c < CH_B; ++c) {
        const bool in = l16 < kb && c < kb;
        a[c] = in && l16 >= c ? gld(A + (k0 + l16) + (long long)lda * (k0 + c)) : (l16 == c ? 1.0 : 0.0);
      }
      int ok = 1;
      chol16<0>(a, rinv, l16, kb, tol, ok);
      if (lane < CH_B) {
#pragma unroll
        for (int c = 0; c < CH_B; ++c) {
          Ld[lane * CH_LDX + c] = a[c];
          if (lane < kb && c <= lane) gst(A + (k0 + lane) + (long long)lda * (k0 + c), a[c]);
        }
      }
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < CH_B; ++c) rv[c] = rinv[c];
        okp[0] = (double)ok;
      }
    }
    t.sync();
    if (okp[0] == 0.0) {                   // the same for every lane
      t.sync();
      return 0;
    }
    // panel: x <- x L^-T, row by row
    if (i < n) {
#pragma unroll
      for (int c = 0; c < CH_B; ++c) {
        double s = x[c];
#pragma unroll
        for (int q = 0; q < c; ++q) s = fma(-x[q], Ld[c * CH_LDX + q], s);
        x[c] = s * rv[c];
      }
#pragma unroll
      for (int c = 0; c < CH_B; ++c) {
        gst(A + i + (long long)lda * (k0 + c), x[c]);
        Xs[tid * CH_LDX + c] = x[c];
      }
    }
    t.sync();
    // trailing block: A22 -= X X^T in tiles [j][i] (lanes along the rows i of a
    // column, contiguous), four row tiles at a time
    const int m = n - k0 - CH_B, nt = m > 0 ? (m + CH_B - 1) / CH_B : 0;
    double* A2 = A + (k0 + CH_B) + (long long)lda * (k0 + CH_B);
    int base = 0;
    for (int J = 0; J < nt; ++J) {
      const int ng = (nt - J + 3) / 4;
      for (int g = (wv - base) & (nw - 1); g < ng; g += nw) {
        const int i0 = CH_B * (J + 4 * g), j0 = CH_B * J;
        ch_acc acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = i0 + CH_B * q + l16, col = j0 + 4 * r + g16;
            acc[q][r] = (row < m && col < m) ? gld(A2 + row + (long long)lda * col) : 0.0;
          }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const int kk = 4 * ks + g16;
          const double fa = -Xs[min(j0 + l16, m - 1) * CH_LDX + kk];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double fb = Xs[min(i0 + CH_B * q + l16, m - 1) * CH_LDX + kk];
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa, fb, acc[q], 0, 0, 0);
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = i0 + CH_B * q + l16, col = j0 + 4 * r + g16;
            if (row < m && col < m) gst(A2 + row + (long long)lda * col, acc[q][r]);
          }
      }
      base += ng;
    }
    t.sync();
  }
  return 1;
}

// Forward substitution along the 16 lanes of a group: step C of
// y_c = (y_c - sum_{q<c} L[c][q] y_q) / L[c][c] for NV independent right-hand
// sides; lane c of a group holds y_c, row c of L in lr and 1 / L[c][c] in ri.
template <int C, int NV>
__device__ __forceinline__ void subst16(double (&y)[NV], const double (&lr)[CH_B], double ri, int l16) {
  if constexpr (C < CH_B) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (l16 == C) y[v] *= ri;
      const double b = row_bcast<C>(y[v]);
      if (l16 > C) y[v] = fma(-lr[C], b, y[v]);
    }
    subst16<C + 1, NV>(y, lr, ri, l16);
  }
}

// Y = L^-T for the lower triangle of L (n <= CH_MAXN), all n x n entries
// written; Y must not alias L.  Column block k of Y (rows up to its own) is
// (I - Y[:, :k] L[k, :k]^T) L_kk^-T: the product on the matrix cores in strips
// of 32 rows per wave with the 16 rows of L in LDS, the substitution by L_kk
// across the lanes that hold the accumulator's columns.  lds: CH_LDS doubles.
template <class T>
__device__ void tri_inv_t_blocked(T& t, const double* L, int ldl, double* Y, int ldy, int n, double* lds) {
  constexpr int LDW = CH_MAXN + 1;         // odd: the 16 rows of a fragment on distinct banks
  static_assert(CH_B * LDW <= CH_PANEL, "rows of L");
  double* Ls = lds;
  const int tid = t.tid(), lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = t.nt() >> 6;
  const int l16 = lane & 15, g16 = lane >> 4;
  const int ns = (n + 31) / 32;
  for (int k0 = 0; k0 < n; k0 += CH_B) {
    const int kb = min(CH_B, n - k0);
    for (int q = tid; q < CH_B * (k0 + CH_B); q += t.nt()) {
      const int c = q & 15, l = q >> 4;
      const bool in = c < kb && l < n && l <= k0 + c;
      Ls[c * LDW + l] = in ? gld(L + (k0 + c) + (long long)ldl * l) : (l == k0 + c ? 1.0 : 0.0);
    }
    t.sync();
    double lr[CH_B];
#pragma unroll
    for (int c = 0; c < CH_B; ++c) lr[c] = Ls[l16 * LDW + k0 + c];
    const double ri = 1.0 / Ls[l16 * LDW + k0 + l16];
    // strips folded over the waves: the first ones have the longest products
    for (int f = 0; f * nw < ns; ++f) {
      const int s = f * nw + ((f & 1) ? nw - 1 - wv : wv);
      if (s >= ns) continue;
      const int r0 = 32 * s;
      double y[8];
#pragma unroll
      for (int v = 0; v < 8; ++v) y[v] = 0.0;
      if (r0 < k0 + CH_B) {
        ch_acc acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
        double f0[4], f1[4], h0[4], h1[4];
        const double* Ya = Y + min(r0 + l16, n - 1);
        const double* Yb = Y + min(r0 + CH_B + l16, n - 1);
        auto fetch = [&](int l0) {
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const long long o = (long long)ldy * (l0 + 4 * ks + g16);
            h0[ks] = gld(Ya + o);
            h1[ks] = gld(Yb + o);
          }
        };
        if (r0 < k0) fetch(r0);
        for (int l0 = r0; l0 < k0; l0 += CH_B) {
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            f0[ks] = h0[ks];
            f1[ks] = h1[ks];
          }
          if (l0 + CH_B < k0) fetch(l0 + CH_B);
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const double fb = -Ls[l16 * LDW + l0 + 4 * ks + g16];
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(f0[ks], fb, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(f1[ks], fb, acc[1], 0, 0, 0);
          }
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          const int row = r0 + CH_B * (v >> 2) + 4 * (v & 3) + g16;
          y[v] = acc[v >> 2][v & 3] + (row == k0 + l16 ? 1.0 : 0.0);
        }
        subst16<0, 8>(y, lr, ri, l16);
      }
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const int row = r0 + CH_B * (v >> 2) + 4 * (v & 3) + g16;
        if (row < n && l16 < kb) gst(Y + row + (long long)ldy * (k0 + l16), y[v]);
      }
    }
    t.sync();
  }
}

// Either form by order.
template <class T>
__device__ __forceinline__ int chol_any(T& t, double* A, int lda, int n, double tol, double* lds) {
  return n >= CH_MINN && n <= CH_MAXN ? chol_blocked(t, A, lda, n, tol, lds) : chol_lower(t, A, lda, n, tol);
}
template <class T>
__device__ __forceinline__ void tri_inv_t_any(T& t, const double* L, int ldl, double* Y, int ldy, int n, double* lds) {
  if (n >= CH_MINN && n <= CH_MAXN) tri_inv_t_blocked(t, L, ldl, Y, ldy, n, lds);
  else tri_inv_lower_t(t, L, ldl, Y, ldy, n, lds, CH_LDS);
}

}  // namespace dg
