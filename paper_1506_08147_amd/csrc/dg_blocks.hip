// Element-local quantities of the DG step built from the ALBs.
//
//   dg_density      rho_K(x) = sum_{j,j'} phi_{K,j}(x) P_{K,j;K,j'} phi_{K,j'}(x)
//                   on the element box: the per-element form of the density
//                   in terms of the diagonal blocks of the density matrix
//                   (Sec. II.A, Eq. newdensity).
//   dg_scatter_box  ALBs (unit basis) into a full-grid block, zero outside E_K
//   dg_nl_block     H_K[j][j'] = sum_p gamma_p <phi_j, b_p> <b_p, phi_j'> over
//                   E_K: the Kleinman-Bylander term of Eq. DGHamiltonian for
//                   K = K' (the coupling to neighbour elements is not formed).
//
// Volume terms of the diagonal block, 1/2 <grad phi, grad phi> + <phi, V phi>
// (Eq. DGHamiltonian, first group), are Gauss quadratures on the element's
// Legendre-Gauss-Lobatto grid with the gradients from differentiation
// matrices (Sec. III, construction of the DG Hamiltonian).  The contractions
// run as strided-batched products (dg_bgemm); the kernels here build their
// small operands:
//   dg_lgl_tables   per axis: LGL weights, differentiation matrix and the
//                   matrix evaluating the trigonometric interpolant of the
//                   extended element's grid at the LGL points
//   dg_box_cols     restriction of full-grid columns to the element box
//   dg_lgl_weights  tensor-product weights w and w * V at the LGL points
#include "common.h"

namespace dg {

constexpr int DEN_ROWS = 64;          // rows of a dg_density workgroup
constexpr int SCATTER_THREADS = 1024;
constexpr int NL_NY = 16;
constexpr int LGL_NY = 32;

// Work item: (element, DEN_ROWS rows of the element box), a wave per 16 rows.
// D = P phi^T for 16 rows of phi by MFMA, DEN_J columns j at a time; D's lane
// layout (j = 4 s + lane / 16, row = lane % 16) is that of phi^T as the second
// operand, so rho = sum_j phi_j D_j is a lane's own products and two exchanges.
// One row per lane with scalar products read phi n / 16 + 1 times behind a serial
// sum.  Measured, 8 elements of 8640 rows, 64 ALBs: 316 -> 31 us.
constexpr int DEN_J = 4;    // blocks of 16 columns j at a time
extern "C" __global__ void __launch_bounds__(256)
dg_density(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
           int na, const double* __restrict__ albs, const double* __restrict__ P,
           double* __restrict__ rho) {
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const Elem& e = E[active[ai]];
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  const int r = (b - prefix[ai]) * DEN_ROWS + (threadIdx.x >> 6) * 16 + l16;
  const int n = e.nalb;
  const long long ne = e.ne;
  const double* phi = albs + e.off_alb + min(r, e.ne - 1);
  const double* Pm = P + e.off_nl;
  double rs = 0.0;
  for (int j0 = 0; j0 < n; j0 += 16 * DEN_J) {
    dbl4 acc[DEN_J];
#pragma unroll
    for (int y = 0; y < DEN_J; ++y) acc[y] = (dbl4){0.0, 0.0, 0.0, 0.0};
    for (int c0 = 0; c0 < n; c0 += 16) {
      double f[4], p[DEN_J][4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int c = c0 + 4 * s + l4, cc = min(c, n - 1);
        f[s] = gld(phi + ne * cc);
#pragma unroll
        for (int y = 0; y < DEN_J; ++y) p[y][s] = gld(Pm + min(j0 + 16 * y + l16, n - 1) + (long long)n * cc);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bool ok = c0 + 4 * s + l4 < n;
        const double fv = ok ? f[s] : 0.0;
#pragma unroll
        for (int y = 0; y < DEN_J; ++y)
          acc[y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ok && j0 + 16 * y + l16 < n ? p[y][s] : 0.0, fv, acc[y], 0,
                                                        0, 0);
      }
    }
#pragma unroll
    for (int y = 0; y < DEN_J; ++y)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int j = j0 + 16 * y + 4 * s + l4;
        const double v = gld(phi + ne * min(j, n - 1));
        rs += j < n ? v * acc[y][s] : 0.0;
      }
  }
  rs += __shfl_xor(rs, 16, 64);
  rs += __shfl_xor(rs, 32, 64);
  if (l4 == 0 && r < e.ne) gst(rho + e.off_ne + r, rs);
}

// Column j of block `dst`: sqrt(dV) phi_j on the element box (ALB j < n_alb),
// zero elsewhere on the grid.  One workgroup per (element, ALB), one pass over
// the grid; a lane's next point is found by carries, not divisions.  Measured,
// 8 x 64 columns of 36x36x60 (of 8 x 128 in two passes before): 161 -> 83 us.
extern "C" __global__ void __launch_bounds__(SCATTER_THREADS)
dg_scatter_box(Elem* __restrict__ E, const int* __restrict__ active, const int* __restrict__ prefix,
               int na, const double* __restrict__ albs, int dst) {
  int b = blockIdx.x;
  int ai = find_elem(prefix, na, b);
  const Elem& e = E[active[ai]];
  int j = b - prefix[ai];
  double* y = bp(e, dst) + (long long)j * e.ld;
  const double s = sqrt(e.dv);
  const double* x = albs + e.off_alb + (long long)j * e.ne;
  const int n1 = e.n1, n2 = e.n2, ng = e.ng;
  const int lo1 = e.lo[0], lo2 = e.lo[1], lo3 = e.lo[2];
  const int b1 = e.hi[0] - lo1, b2 = e.hi[1] - lo2, b3 = e.hi[2] - lo3;
  int q = threadIdx.x / n1, i1 = threadIdx.x - q * n1, i3 = q / n2, i2 = q - i3 * n2;
  const int dq = SCATTER_THREADS / n1, d1 = SCATTER_THREADS - dq * n1, d3 = dq / n2, d2 = dq - d3 * n2;
  for (int i = threadIdx.x; i < ng; i += SCATTER_THREADS) {
    const int k1 = i1 - lo1, k2 = i2 - lo2, k3 = i3 - lo3;
    const bool in = (unsigned)k1 < (unsigned)b1 && (unsigned)k2 < (unsigned)b2 && (unsigned)k3 < (unsigned)b3;
    const double v = gld(x + (in ? k1 + b1 * (k2 + b2 * k3) : 0));
    gst(y + i, in ? s * v : 0.0);
    i1 += d1;
    int c = i1 >= n1;
    i1 -= c ? n1 : 0;
    i2 += d2 + c;
    c = i2 >= n2;
    i2 -= c ? n2 : 0;
    i3 += d3 + c;
  }
}

// H = B^T diag(gamma) B for B = e.proj (n_proj x J, the projections of the
// scattered ALBs), n_alb columns; NL_NY workgroups per element (one spent
// 210 us on 64 x 64 entries of 80 projectors; now 16 us).
extern "C" __global__ void __launch_bounds__(256)
dg_nl_block(Elem* __restrict__ E, const int* __restrict__ active, int na, double* __restrict__ out) {
  const Elem& e = E[active[blockIdx.x]];
  const int n = e.nalb, np = e.n_proj;
  double* H = out + e.off_nl;
  for (int p = blockIdx.y * 256 + threadIdx.x; p < n * n; p += NL_NY * 256) {
    int j = p % n, k = p / n;
    const double *pj = e.proj + (long long)np * j, *pk = e.proj + (long long)np * k;
    double s = 0.0;
    for (int q = 0; q < np; ++q) s += gld(e.gamma + q) * gld(pj + q) * gld(pk + q);
    gst(H + p, s);
  }
}

constexpr int LGL_MAX = 1024;   // LGL points per axis

struct LglTab {
  double* w[3];   // m_d quadrature weights on the element's interval
  double* D[3];   // m_d x m_d differentiation matrix (column-major)
  double* I[3];   // m_d x n_d interpolation matrix (column-major)
  int m[3];
};

// Legendre P_N(x) and P_{N-1}(x) by the three-term recurrence; rk[k] = 1 / (k + 1).
// The quotient is corrected by its remainder, which rounds it as a division
// does: with the product alone the volume blocks of the slab were 6.9e-15 off
// their value in 64 bits, with divisions 6.1e-15.
__device__ inline void legendre_pair(int N, double x, const double* rk, double& pn, double& pn1) {
  double p0 = 1.0, p1 = x;
  if (N == 0) { pn = 1.0; pn1 = 0.0; return; }
  for (int k = 1; k < N; ++k) {
    const double s = (2 * k + 1) * x * p1 - k * p0, q = s * rk[k], p2 = fma(fma(-(k + 1.0), q, s), rk[k], q);
    p0 = p1;
    p1 = p2;
  }
  pn = p1;
  pn1 = p0;
}

// Grid (axis d, LGL_NY) for element ei; each workgroup forms the nodes of its
// axis, a serial chain of m steps per iteration, and a share of the tables
// (one workgroup per axis and always 40 iterations: 447 us at 24 x 24 x 120
// nodes, now 43 us).  LGL nodes on [-1, 1]: the end
// points and the roots of P'_N (N = m - 1), by Newton's method on P'_N with
// P''_N from Legendre's equation, started at the Chebyshev-Lobatto points, to
// a correction below 1e-12 (its square, times at most the reciprocal spacing
// of the nodes, is what is left).
// Weights 2 / (N (N+1) P_N(x_i)^2); differentiation matrix
// D_ij = P_N(x_i) / (P_N(x_j) (x_i - x_j)) off the diagonal, -+N(N+1)/4 at
// the two corners, 0 elsewhere on the diagonal.  The element's interval along
// d is [lo_d h, hi_d h] with h = L_d / n_d; interpolation weight of grid point
// j at x: the periodic Dirichlet kernel (1/n)(1 + 2 sum_{k<n/2} cos(k th)
// + [n even] cos(n th / 2)), th = 2 pi (x - j h) / L_d.
extern "C" __global__ void __launch_bounds__(256)
dg_lgl_tables(const Elem* __restrict__ E, int ei, LglTab t) {
  __shared__ double xs[LGL_MAX], pn[LGL_MAX], rk[LGL_MAX];
  const Elem& e = E[ei];
  const int d = blockIdx.x, m = t.m[d], N = m - 1;
  const int n = d == 0 ? e.n1 : (d == 1 ? e.n2 : e.n3);
  const double L = e.L[d], h = L / n, ell = (e.hi[d] - e.lo[d]) * h, x0 = e.lo[d] * h;
  for (int k = threadIdx.x; k < m; k += 256) rk[k] = 1.0 / (k + 1);
  __syncthreads();
  for (int i = threadIdx.x; i < m; i += 256) {
    double x = i == 0 ? -1.0 : (i == N ? 1.0 : -cos(M_PI * i / N));
    double p, q;
    if (i > 0 && i < N) {
      for (int it = 0; it < 40; ++it) {
        legendre_pair(N, x, rk, p, q);
        double dp = N * (x * p - q) / (x * x - 1.0);
        double d2 = (2.0 * x * dp - N * (N + 1.0) * p) / (1.0 - x * x);
        const double dx = dp / d2;
        x -= dx;
        if (fabs(dx) < 1e-12) break;
      }
    }
    legendre_pair(N, x, rk, p, q);
    xs[i] = x;
    pn[i] = p;
  }
  __syncthreads();
  const double nn = N * (N + 1.0);
  const int t0 = blockIdx.y * 256 + threadIdx.x, ts = LGL_NY * 256;
  for (int i = t0; i < m; i += ts) t.w[d][i] = 0.5 * ell * 2.0 / (nn * pn[i] * pn[i]);
  const double sc = 2.0 / ell;
  for (int p = t0; p < m * m; p += ts) {
    int i = p % m, j = p / m;
    double v;
    if (i != j) v = pn[i] / (pn[j] * (xs[i] - xs[j]));
    else v = i == 0 ? -0.25 * nn : (i == N ? 0.25 * nn : 0.0);
    t.D[d][p] = sc * v;
  }
  const int kmax = (n - 1) / 2;
  for (int p = t0; p < m * n; p += ts) {
    int i = p % m, j = p / m;
    double x = x0 + 0.5 * (xs[i] + 1.0) * ell;
    double th = 2.0 * M_PI * (x - j * h) / L;
    double s = 1.0;
    for (int k = 1; k <= kmax; ++k) s += 2.0 * cos(k * th);
    if (n % 2 == 0) s += cos(0.5 * n * th);
    t.I[d][p] = s / n;
  }
}

// V of elements ei, ei + 1, ... (of one grid) one after another; grid
// (1024 points, elements).
extern "C" __global__ void __launch_bounds__(256)
dg_take_v(const Elem* __restrict__ E, int ei, double* __restrict__ dst) {
  const Elem& e = E[ei + blockIdx.y];
  const double* V = e.V;
  double* y = dst + (long long)blockIdx.y * e.ng;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = blockIdx.x * 1024 + u * 256 + threadIdx.x;
    if (i < e.ng) gst(y + i, gld(V + i));
  }
}

// dst[r + N_E c] = src[flat(r) + N_g c] for the rows r of the element box
// (x fastest), c < J, for blockIdx.z elements of the geometry of element ei
// whose columns follow one another (src stride N_g J, dst stride N_E J).
// Grid (row chunks of 256, J, elements).
extern "C" __global__ void __launch_bounds__(256)
dg_box_cols(const Elem* __restrict__ E, int ei, const double* __restrict__ src, double* __restrict__ dst) {
  const Elem& e = E[ei];
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= e.ne) return;
  const int c = blockIdx.y;
  src += (long long)blockIdx.z * e.ng * e.J;
  dst += (long long)blockIdx.z * e.ne * e.J;
  int b1 = e.hi[0] - e.lo[0], b2 = e.hi[1] - e.lo[1];
  int i = r % b1, q = r / b1;
  int jj = q % b2, kk = q / b2;
  long long flat = (e.lo[0] + i) + (long long)e.n1 * ((e.lo[1] + jj) + (long long)e.n2 * (e.lo[2] + kk));
  dst[r + (long long)e.ne * c] = src[flat + (long long)e.ng * c];
}

// w[q] = w1[i] w2[j] w3[k] and vw[q] = w[q] vL[q] for LGL point q = (i, j, k),
// i fastest; blockIdx.y selects the element (vL, vw stride = LGL points).
extern "C" __global__ void __launch_bounds__(256)
dg_lgl_weights(LglTab t, const double* __restrict__ vL, double* __restrict__ w, double* __restrict__ vw) {
  const int m1 = t.m[0], m2 = t.m[1];
  const long long M = (long long)m1 * m2 * t.m[2];
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= M) return;
  vL += M * blockIdx.y;
  vw += M * blockIdx.y;
  int i = (int)(q % m1);
  long long r = q / m1;
  int j = (int)(r % m2), k = (int)(r / m2);
  double v = t.w[0][i] * t.w[1][j] * t.w[2][k];
  if (blockIdx.y == 0) w[q] = v;
  vw[q] = v * vL[q];
}

}  // namespace dg
