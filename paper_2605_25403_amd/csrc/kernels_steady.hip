// Kernels of the steady Navier-Stokes solver (Newton's method on the
// monolithic P2-P1 system; Section 2.2.1, Newton linearization, with the
// time-derivative term dropped for the steady equations of Section 2.1).
//
// The Newton matrix over x = (U_0, .., U_{d-1}, P) is kept in one SELL-64
// layout ("monolithic"); its values are composed from the blocks the
// row-owner assembly forms on their own patterns (nu K, C(U), N_ce(U), G_c,
// D_c), through a per-entry map (source entry, kind, components). The
// preconditioner's velocity block has a SELL layout of its own. The Krylov
// solver around them (flexible GMRES) uses the generic vector kernels below:
// a SELL product with an axpby, multi-dot products with deterministic
// two-pass reductions, multi-axpys and scalings by device scalars.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "dev_util.hpp"
#include "device.hpp"
#include "steady.hpp"

namespace ipcs {

namespace {

constexpr int SBS = 256;                    // threads per block
constexpr int SCHUNK = SBS * 8;             // rows per block of the reductions

__global__ void __launch_bounds__(SBS)
k_compose(MonoCompose m) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= m.nrows) return;
  const int64_t nu_rows = (int64_t)m.dim * m.n2;
  const bool vrow = r < nu_rows;
  const bool brow = vrow && m.bmask[r % m.n2];
  const int sl = (int)(r >> 6), w = (m.sptr[sl + 1] - m.sptr[sl]) >> 6;
  const int base = m.sptr[sl] + (int)(r & 63);
  for (int k = 0; k < w; ++k) {
    const int e = base + 64 * k;
    const int32_t src = m.src[e];
    const int code = m.code[e];
    const int kind = code & 7, c = (code >> 3) & 3, d = (code >> 5) & 3;
    const int64_t col = m.col[e];
    double pic = 0.0, nwt = 0.0;
    switch (kind) {
      case MONO_UU_DIAG:
        pic = m.nu * m.K[src] + m.C[src];
        nwt = pic + m.N[c * m.dim + d][src];
        break;
      case MONO_UU_OFF: nwt = m.N[c * m.dim + d][src]; break;
      case MONO_G: pic = nwt = m.Gc[c][src]; break;
      case MONO_D: pic = nwt = m.Dc[d][src]; break;
      default: break;   // padding
    }
    const bool bcol = col < nu_rows && m.bmask[col % m.n2];
    if (brow) {
      // boundary velocity row: the increment is zero there (identity row of
      // the Newton matrix); the residual row is zero
      nwt = (col == r && kind != MONO_PAD) ? 1.0 : 0.0;
      pic = 0.0;
    } else if (bcol) {
      nwt = 0.0;   // boundary columns eliminated; the residual keeps them
    }
    if (m.J) m.J[e] = nwt;
    if (m.Pic) m.Pic[e] = pic;
  }
}

// y = beta b + alpha A x over rows [0, nrows) of a SELL-64 FP64 matrix.
__global__ void __launch_bounds__(SBS)
k_sell_axpby(int64_t nrows, const int32_t* sp, const int32_t* col, const double* A,
             const double* x, double alpha, double beta, const double* b, double* y) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrows) return;
  const int sl = (int)(r >> 6), w = (sp[sl + 1] - sp[sl]) >> 6;
  const int base = sp[sl] + (int)(r & 63);
  double s = 0.0;
  for (int k = 0; k < w; k += 4) {
    double a[4], v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kk = k + q < w ? k + q : w - 1;
      const int e = base + 64 * kk;
      a[q] = k + q < w ? A[e] : 0.0;
      v[q] = x[col[e]];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) s += a[q] * v[q];
  }
  y[r] = (beta != 0.0 ? beta * b[r] : 0.0) + alpha * s;
}

// part[j * nblk + blk] = sum over the block's rows of V[j][i] * w[i], j < k
__global__ void __launch_bounds__(SBS)
k_mdot(int64_t n, const double* V, int64_t ldv, const double* w, int k, double* part, int nblk) {
  __shared__ double sh[SBS / 64];
  const int j = blockIdx.y;
  const double* v = V + (int64_t)j * ldv;
  const int64_t i0 = (int64_t)blockIdx.x * SCHUNK;
  double s = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < min<int64_t>(n, i0 + SCHUNK); i += SBS) s += v[i] * w[i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[(int64_t)j * nblk + blockIdx.x] = s;
}

// out[j] = sum over blocks of part[j][.] in block order (one block per j);
// acc != 0 adds the result to out[j] instead of storing it
__global__ void __launch_bounds__(SBS)
k_mdot_fin(const double* part, int nblk, double* out, int acc) {
  __shared__ double sh[SBS / 64];
  const int j = blockIdx.x;
  double s = 0.0;
  for (int b = threadIdx.x; b < nblk; b += SBS) s += part[(int64_t)j * nblk + b];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) out[j] = acc ? out[j] + s : s;
}

// y[i] += sign * sum_{j<k} h[j] V[j][i]
__global__ void __launch_bounds__(SBS)
k_maxpy(int64_t n, const double* V, int64_t ldv, const double* h, int k, double sign, double* y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int j = 0; j < k; ++j) s += h[j] * V[(int64_t)j * ldv + i];
  y[i] += sign * s;
}

// One Gram-Schmidt pass from the partial sums of k_mdot (nblk per vector):
// h[j] = their sum, y -= sum_{j<k} h[j] V[j]; block 0 keeps h in out. nrm (may
// be null) receives the block's partial sum of y^2. Every block adds the
// partials up by itself, a thread per vector: a launch of its own for that
// costs more (48^2 squares: 11 partials of up to 61 vectors).
__global__ void __launch_bounds__(SBS)
k_gs_pass(int64_t n, const double* V, int64_t ldv, const double* part, int nblk, int k, double* out,
          double* y, double* nrm) {
  __shared__ double h[512], sh[SBS / 64];
  for (int j = threadIdx.x; j < k; j += SBS) {
    double s = 0.0;
    for (int b = 0; b < nblk; ++b) s += part[(int64_t)j * nblk + b];
    h[j] = s;
    if (blockIdx.x == 0) out[j] = s;
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double yi = 0.0;
  if (i < n) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int j = 0;
    for (; j + 4 <= k; j += 4)
#pragma unroll
      for (int q = 0; q < 4; ++q) s[q] += h[j + q] * V[(int64_t)(j + q) * ldv + i];
    for (; j < k; ++j) s[0] += h[j] * V[(int64_t)j * ldv + i];
    yi = y[i] - ((s[0] + s[1]) + (s[2] + s[3]));
    y[i] = yi;
  }
  if (nrm) {
    const double q = block_sum(yi * yi, sh);
    if (threadIdx.x == 0) nrm[blockIdx.x] = q;
  }
}

// y /= ||y||, ||y||^2 from nblk partial sums (block 0 keeps it in out)
__global__ void __launch_bounds__(SBS)
k_gs_scale(int64_t n, const double* nrm, int nblk, double* out, double* y) {
  __shared__ double sh[SBS / 64];
  double q = 0.0;
  for (int b = threadIdx.x; b < nblk; b += SBS) q += nrm[b];
  q = block_sum(q, sh);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) out[0] = q;
  if (i < n) y[i] = q > 0.0 ? y[i] / sqrt(q) : 0.0;
}

// y = x / sqrt(*nrm2)
__global__ void __launch_bounds__(SBS)
k_scale_inv_norm(int64_t n, const double* x, const double* nrm2, double* y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double q = *nrm2;
  y[i] = q > 0.0 ? x[i] / sqrt(q) : 0.0;
}

// pressure part of the block-triangular preconditioner: zp = -nu vp / w
// (the lumped pressure mass scaled by 1/nu stands for the Schur complement)
__global__ void __launch_bounds__(SBS)
k_prec_p(int64_t n1, const double* vp, const double* w, double nu, double* zp) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n1) zp[k] = -nu * vp[k] / w[k];
}

// Two Chebyshev steps on D^{-1} M for the consistent pressure mass matrix M
// (eigenvalues in [1/2, (d + 2)/2], Wathen 1987), from x1 = d1 = D^{-1} v / theta:
// d <- a d + b D^{-1} (v - M x), x <- x + d. FIRST forms x1 from v as it gathers;
// the second step writes out = scale x.
template <bool FIRST>
__global__ void __launch_bounds__(SBS)
k_mass_cheb(int64_t n, const int32_t* sp, const int32_t* col, const double* M, const double* dinv,
            const double* v, double itheta, double a, double b, double* x, double* d, double scale,
            double* out) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const int sl = (int)(r >> 6), w = (sp[sl + 1] - sp[sl]) >> 6;
  const int base = sp[sl] + (int)(r & 63);
  double s = 0.0;
  for (int k = 0; k < w; k += 4) {
    double m[4], g[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = base + 64 * (k + q < w ? k + q : w - 1);
      const int c = col[e];
      m[q] = k + q < w ? M[e] : 0.0;
      g[q] = FIRST ? dinv[c] * v[c] * itheta : x[c];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) s += m[q] * g[q];
  }
  const double x0 = FIRST ? dinv[r] * v[r] * itheta : x[r], d0 = FIRST ? x0 : d[r];
  const double dn = a * d0 + b * dinv[r] * (v[r] - s);
  if (FIRST) {
    x[r] = x0 + dn;
    d[r] = dn;
  } else {
    out[r] = scale * (x0 + dn);
  }
}

// heads[c * ldh + i] = v_c[i] - (G_c zp)_i (v_c[i] on the boundary)
// One launch for all components, which share the columns and zp's values; four
// entries' loads go out before the first is used (the launch is one chain of
// dependent loads: 9409 rows are 147 waves, less than one per CU).
__global__ void __launch_bounds__(SBS)
k_prec_rhs(int dim, int64_t n2, const int32_t* sp, const int32_t* col, const double* G0,
           const double* G1, const double* G2, const uint8_t* bmask, const double* v,
           const double* zp, double* heads, int64_t ldh) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n2) return;
  const int sl = (int)(r >> 6), w = (sp[sl + 1] - sp[sl]) >> 6;
  const int base = sp[sl] + (int)(r & 63);
  double s[3] = {0.0, 0.0, 0.0};
  if (!bmask[r])
    for (int k = 0; k < w; k += 4) {
      double g[3][4], z[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool on = k + q < w;
        const int e = base + 64 * (on ? k + q : w - 1);
        z[q] = zp[col[e]];
        g[0][q] = on ? G0[e] : 0.0;
        g[1][q] = on ? G1[e] : 0.0;
        g[2][q] = on && dim == 3 ? G2[e] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += g[c][q] * z[q];
    }
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (c < dim) heads[c * ldh + r] = v[c * n2 + r] - s[c];
}

// heads[c * ldh + i] -= (A z)_(c n2 + i)
// As above, eight entries at a time: the rows are the widest ones here.
__global__ void __launch_bounds__(SBS)
k_prec_resid(int64_t rows, int64_t n2, const int32_t* sp, const int32_t* col, const double* A,
             const double* z, double* heads, int64_t ldh) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const int sl = (int)(r >> 6), w = (sp[sl + 1] - sp[sl]) >> 6;
  const int base = sp[sl] + (int)(r & 63);
  double s = 0.0;
  for (int k = 0; k < w; k += 8) {
    double a[8], v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = base + 64 * (k + q < w ? k + q : w - 1);
      a[q] = k + q < w ? A[e] : 0.0;
      v[q] = z[col[e]];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) s += a[q] * v[q];
  }
  heads[(r / n2) * ldh + r % n2] -= s;
}

// v -= f * (*scal)
__global__ void __launch_bounds__(SBS)
k_sub_scaled(int64_t n, const double* scal, double f, double* v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) v[i] -= f * *scal;
}

__global__ void __launch_bounds__(SBS) k_fill(int64_t n, double v, double* y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = v;
}

__global__ void __launch_bounds__(SBS) k_copy(int64_t n, const double* x, double* y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = x[i];
}

// Jacobi diagonal of a SELL-64 FP64 matrix (1 where the diagonal is zero)
__global__ void __launch_bounds__(SBS)
k_inv_diag(int64_t n, const int32_t* sp, const int32_t* col, const double* A, double* dinv) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const int sl = (int)(r >> 6), w = (sp[sl + 1] - sp[sl]) >> 6;
  const int base = sp[sl] + (int)(r & 63);
  double d = 0.0;
  for (int k = 0; k < w; ++k)
    if (col[base + 64 * k] == r) d += A[base + 64 * k];
  dinv[r] = d != 0.0 ? 1.0 / d : 1.0;
}

inline int grid(int64_t n) { return (int)div_up(n, SBS); }

}  // namespace

void mono_compose(hipStream_t s, const MonoCompose& m) {
  if (m.nrows <= 0) return;
  launch(k_compose, dim3(grid(m.nrows)), dim3(SBS), 0, s, m);
}

void sell_axpby(hipStream_t s, int64_t nrows, const int32_t* sp, const int32_t* col,
                const double* A, const double* x, double alpha, double beta, const double* b,
                double* y) {
  if (nrows <= 0) return;
  launch(k_sell_axpby, dim3(grid(nrows)), dim3(SBS), 0, s, nrows, sp, col, A, x, alpha, beta,
         b, y);
}

int mdot_blocks(int64_t n) { return (int)std::max<int64_t>(1, div_up(n, SCHUNK)); }

void mdot(hipStream_t s, int64_t n, const double* V, int64_t ldv, const double* w, int k,
          double* part, double* out, int acc) {
  if (k <= 0) return;
  const int nb = mdot_blocks(n);
  launch(k_mdot, dim3(nb, k), dim3(SBS), 0, s, n, V, ldv, w, k, part, nb);
  launch(k_mdot_fin, dim3(k), dim3(SBS), 0, s, (const double*)part, nb, out, acc);
}

void maxpy(hipStream_t s, int64_t n, const double* V, int64_t ldv, const double* h, int k,
           double sign, double* y) {
  if (k <= 0 || n <= 0) return;
  launch(k_maxpy, dim3(grid(n)), dim3(SBS), 0, s, n, V, ldv, h, k, sign, y);
}

bool orthonormalize(hipStream_t s, int64_t n, const double* V, int k, double* part, double* h1,
                    double* h2, double* nrm2, double* w) {
  const int nb = mdot_blocks(n), ng = (int)grid(n);
  if (n <= 0 || k <= 0 || k > 512 || nb > kGsParts) return false;
  double* nrm = part + (int64_t)k * nb;
  launch(k_mdot, dim3(nb, k), dim3(SBS), 0, s, n, V, n, (const double*)w, k, part, nb);
  launch(k_gs_pass, dim3(ng), dim3(SBS), 0, s, n, V, n, (const double*)part, nb, k, h1, w,
         (double*)nullptr);
  launch(k_mdot, dim3(nb, k), dim3(SBS), 0, s, n, V, n, (const double*)w, k, part, nb);
  launch(k_gs_pass, dim3(ng), dim3(SBS), 0, s, n, V, n, (const double*)part, nb, k, h2, w, nrm);
  launch(k_gs_scale, dim3(ng), dim3(SBS), 0, s, n, (const double*)nrm, ng, nrm2, w);
  return true;
}

void scale_inv_norm(hipStream_t s, int64_t n, const double* x, const double* nrm2, double* y) {
  launch(k_scale_inv_norm, dim3(grid(n)), dim3(SBS), 0, s, n, x, nrm2, y);
}

void prec_pressure(hipStream_t s, int64_t n1, const double* vp, const double* w, double nu,
                   double* zp) {
  launch(k_prec_p, dim3(grid(n1)), dim3(SBS), 0, s, n1, vp, w, nu, zp);
}

void mass_solve(hipStream_t s, int64_t n, int dim, const int32_t* sp, const int32_t* col,
                const double* M, const double* dinv, const double* v, double scale, double* x,
                double* d, double* out) {
  const double lo = 0.5, hi = 0.5 * (dim + 2), theta = 0.5 * (lo + hi), delta = 0.5 * (hi - lo);
  const double sigma = theta / delta;
  double rho = 1.0 / sigma, rn = 1.0 / (2.0 * sigma - rho);
  launch(k_mass_cheb<true>, dim3(grid(n)), dim3(SBS), 0, s, n, sp, col, M, dinv, v, 1.0 / theta,
         rn * rho, 2.0 * rn / delta, x, d, scale, out);
  rho = rn;
  rn = 1.0 / (2.0 * sigma - rho);
  launch(k_mass_cheb<false>, dim3(grid(n)), dim3(SBS), 0, s, n, sp, col, M, dinv, v, 1.0 / theta,
         rn * rho, 2.0 * rn / delta, x, d, scale, out);
}

void prec_rhs(hipStream_t s, int dim, int64_t n2, const int32_t* sp, const int32_t* col,
              const double* const* G, const uint8_t* bmask, const double* v, const double* zp,
              double* heads, int64_t ldh) {
  launch(k_prec_rhs, dim3(grid(n2)), dim3(SBS), 0, s, dim, n2, sp, col, G[0], G[1],
         dim == 3 ? G[2] : G[0], bmask, v, zp, heads, ldh);
}

void prec_resid(hipStream_t s, int64_t rows, int64_t n2, const int32_t* sp, const int32_t* col,
                const double* A, const double* z, double* heads, int64_t ldh) {
  launch(k_prec_resid, dim3(grid(rows)), dim3(SBS), 0, s, rows, n2, sp, col, A, z, heads, ldh);
}

void sub_scaled(hipStream_t s, int64_t n, const double* scal, double f, double* v) {
  if (n > 0) launch(k_sub_scaled, dim3(grid(n)), dim3(SBS), 0, s, n, scal, f, v);
}

void fill(hipStream_t s, int64_t n, double v, double* y) {
  if (n > 0) launch(k_fill, dim3(grid(n)), dim3(SBS), 0, s, n, v, y);
}

void copy_vec(hipStream_t s, int64_t n, const double* x, double* y) {
  if (n > 0) launch(k_copy, dim3(grid(n)), dim3(SBS), 0, s, n, x, y);
}

void sell_inv_diag(hipStream_t s, int64_t n, const int32_t* sp, const int32_t* col,
                   const double* A, double* dinv) {
  if (n > 0) launch(k_inv_diag, dim3(grid(n)), dim3(SBS), 0, s, n, sp, col, A, dinv);
}

}  // namespace ipcs
