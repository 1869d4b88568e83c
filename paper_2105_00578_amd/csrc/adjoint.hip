// Gradient of a loss l(lambda, V) with respect to the edge weights, through
// the eigenpairs of L_C v = lambda B v (weighted Laplacian of Sec. 3.2).
//
// Raising w_e of edge e = {i, j} changes L_C by (e_i - e_j)(e_i - e_j)^T and,
// for the generalized problem, B = D by e_i e_i^T + e_j e_j^T.  First-order
// perturbation of B-orthonormal eigenpairs (simple eigenvalues) gives, with
// a = V[i,:], b = V[j,:]:
//   eigenvalue terms   g_lam_k [(a_k-b_k)^2 - gen lam_k (a_k^2+b_k^2)]
//   in-block terms     c_kl [(a_k-b_k)(a_l-b_l) - gen lam_k (a_k a_l + b_k b_l)],
//                      c_kl = (g_k . v_l) / (lam_k - lam_l), l != k
//   normalisation      -gen/2 (g_k . v_k)(a_k^2 + b_k^2)
//   out-of-block terms -(mu_ki-mu_kj)(a_k-b_k) + gen lam_k (mu_ki a_k + mu_kj b_k)
// where mu_k solves (L - lam_k B) mu_k = g_k - B V V^T g_k with V^T B mu_k = 0.
// The first three groups are the bilinear forms (a-b)^T M1 (a-b) and
// a^T M2 a + b^T M2 b with small nev x nev matrices built on the host.
//
// The normalized problem L_N y = lambda y has the eigenpairs (lambda, D^1/2 x)
// of the generalized one.  With x = D^-1/2 y, the loss sees y through x and
// through D^1/2, whose entries i and j move by 1/(2 sqrt(d)) when w_e does:
//   dl/dw_e = [generalized gradient with dl/dx = D^1/2 dl/dy]
//             + t_i + t_j,   t_i = sum_k (dl/dy_ik) y_ik / (2 d_i).
//
// mu_k comes from a projected preconditioned conjugate gradient run on all
// columns at once (one Laplacian product per step): iterates stay in the
// B-orthogonal complement of V through z = (I - V V^T B) J r, J the diagonal
// of L - lam_k B inverted; residuals stay orthogonal to V.  The CG blocks are
// n x ld row-major (ld even: 16-byte rows), so the product is the vector-row
// Laplacian kernel with the shift lam_k B and the dots p^T A p fused into its
// epilogue.  The CG scalars (r^T z, alpha, beta, convergence flags) live on
// the device and are computed by one-block reductions in a fixed order; the
// host reads the flags of a batch of steps while the next batch runs.
// Convergence: the relative residual in the preconditioner's norm,
// sqrt(r^T z / f^T J f) <= cg_tol; a converged column no longer moves.
#include <algorithm>
#include <cmath>

#include "kernels.h"

namespace sphx {
namespace {

struct Small {
  double a[kMaxNev * kMaxNev];
};

struct AdjParams {
  int nev;
  int gen;
  double lam[kMaxNev];
};

// Gram partials: out[block][j * nev + k] = sum_i A[i,j] * wgt_i * B[i,k] over
// the block's rows (A, B row-major with row strides lda, ldb).  The 256
// threads form 256 / nev^2 groups, each covering every group-th row of the
// block for all nev^2 pairs (four independent sums per thread keep loads in
// flight); the groups are added in LDS in group order.
__global__ __launch_bounds__(256) void k_small_gram(const double *A, int lda, const double *Bm,
                                                    int ldb, const double *wgt, int64_t n,
                                                    int nev, double *partials,
                                                    int64_t rows_per_block) {
  __shared__ double sh[256];
  const int np = nev * nev;
  const int ng = 256 / np;
  const int t = threadIdx.x;
  const int grp = t / np, pr = t - grp * np;
  const int j = pr / nev, k = pr - j * nev;
  const bool live = grp < ng;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = min(n, r0 + rows_per_block);
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  if (live) {
    int64_t i = r0 + grp;
    const int64_t st = ng;
    for (; i + 3 * st < r1; i += 4 * st) {
      const double a0 = A[i * lda + j], b0 = Bm[i * ldb + k];
      const double a1 = A[(i + st) * lda + j], b1 = Bm[(i + st) * ldb + k];
      const double a2 = A[(i + 2 * st) * lda + j], b2 = Bm[(i + 2 * st) * ldb + k];
      const double a3 = A[(i + 3 * st) * lda + j], b3 = Bm[(i + 3 * st) * ldb + k];
      if (wgt) {
        s0 += a0 * wgt[i] * b0;
        s1 += a1 * wgt[i + st] * b1;
        s2 += a2 * wgt[i + 2 * st] * b2;
        s3 += a3 * wgt[i + 3 * st] * b3;
      } else {
        s0 += a0 * b0;
        s1 += a1 * b1;
        s2 += a2 * b2;
        s3 += a3 * b3;
      }
    }
    for (; i < r1; i += st) s0 += A[i * lda + j] * (wgt ? wgt[i] : 1.0) * Bm[i * ldb + k];
  }
  sh[t] = live ? (s0 + s1) + (s2 + s3) : 0.0;
  __syncthreads();
  if (t < np) {
    double a = 0.0;
    for (int g = 0; g < ng; ++g) a += sh[g * np + t];
    partials[(int64_t)blockIdx.x * kMaxNev * kMaxNev + t] = a;
  }
}

// out[p] = sum over blocks of partials[block][p], p < cnt: one wavefront per
// output, lanes strided over the blocks, then a butterfly (fixed order).
__global__ __launch_bounds__(1024) void k_small_sum(const double *partials, int nblocks,
                                                    int cnt, double *out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int p = wave; p < cnt; p += 16) {
    double a = 0.0;
    for (int b = lane; b < nblocks; b += 64) a += partials[(int64_t)b * kMaxNev * kMaxNev + p];
    for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off);
    if (lane == 0) out[p] = a;
  }
}

// Vp (n x ld) = V (n x nev) with zero padding columns
__global__ void k_pad_cols(const double *V, int nev, double *Vp, int ld, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * ld;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / ld;
    const int c = (int)(e - i * ld);
    Vp[e] = (V && c < nev) ? V[i * nev + c] : 0.0;
  }
}

// r = g - B V (V^T g)  (M = V^T g, nev x nev, device; g stride nev, V and r
// stride ld, padding columns of r zero)
__global__ void k_project_rhs(const double *G, const double *Vp, const double *bd,
                              const double *M, int64_t n, int nev, int ld, double *R) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * ld;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / ld;
    const int k = (int)(e - i * ld);
    if (k >= nev) { R[e] = 0.0; continue; }
    double s = 0.0;
    for (int j = 0; j < nev; ++j) s += Vp[i * ld + j] * M[j * nev + k];
    R[e] = G[i * nev + k] - (bd ? bd[i] : 1.0) * s;
  }
}

// ---- projected CG
//
// A step is four launches: the product (with p^T A p partials per block),
// k_cg_update (alpha, x and r, and the partial sums of the projection),
// k_cg_reduce, and k_cg_direction (the projection, beta and the new p).  At
// the sizes met here (some 10^4 to 10^5 rows of 3..16 columns) a step is bound
// by launches and by its chain of reductions, not by bytes, so every small
// sum is taken where it is used: each block of k_cg_update adds the product's
// partials itself, and each block of k_cg_direction forms beta itself; only
// block 0 writes the state, into the other of two copies.  With z = J r,
// M = V^T B z and G = V^T r, the projected residual z' = z - V M has
// r^T z' = r^T z - sum_j G_jk M_jk, so neither z nor z' is stored.
// Measured on a 256 x 200 grid, 5 columns (51,200 rows): 25 us per step where
// eight kernels with one-block reductions took 63.
struct CgState {
  double rz[kMaxNev], rz0[kMaxNev];
  int done[kMaxNev];
  int iters;       // steps with at least one active column
  int breakdown;   // a column met p^T A p <= 0 before converging
};
// what k_cg_update's alphas tell the state
struct CgAlpha {
  int broke[kMaxNev];
  int any;
};

constexpr int kCgTile = 64;       // rows per tile of k_cg_update
constexpr int kCgBlocks = 1024;   // its blocks, at most
constexpr int kCgParts = 1024;    // product partials a block adds by itself

// sums per block of k_cg_update: M and G (nev x nev each), then r^T z
__host__ __device__ inline int cg_sums(int nev) { return 2 * nev * nev + nev; }

typedef double d2 __attribute__((ext_vector_type(2)));

// 1 / J_ik = d_i - lam_k b_i (d_i where that is not positive)
__device__ __forceinline__ double cg_diag(double d, double b, double lam) {
  const double x = d - lam * b;
  return x > 0.0 ? x : d;
}

// out[c] = sum of column c's product partials (when there are more than
// kCgParts of them), one block per column, fixed order.
__global__ __launch_bounds__(1024) void k_cg_pap(const double *parts, int nparts, double *out) {
  __shared__ double sh[16];
  const double *x = parts + (int64_t)blockIdx.x * kMaxNormBlocks;
  double a = 0.0;
  for (int b = threadIdx.x; b < nparts; b += 1024) a += x[b];
  for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int q = 0; q < 16; ++q) r += sh[q];
    out[(int64_t)blockIdx.x * kMaxNormBlocks] = r;
  }
}

// x += alpha p, r -= alpha A p (pap: the product's partials, sum-major, or
// null for no step), then the block's sums of M, G and r^T z over its tiles,
// stored value-major (value v of block b at sums[v * gridDim.x + b]).  Each
// tile's V, r, z and b are staged in LDS; a thread owns one (j, k) pair of
// every ng-th row of the tile, and the groups are added in order at the end.
// kItems: pairs of a tile per thread, 1 for rows of up to 8 columns, else 2.
template <int kItems>
__global__ __launch_bounds__(256) void k_cg_update(double *MU, double *R, const double *P,
                                                   const double *AP, const double *Vp,
                                                   const double *pap, int nparts,
                                                   const CgState *st, CgAlpha *alpha_out,
                                                   const double *d, const double *bd,
                                                   AdjParams p, int64_t n, int ld, int64_t ntiles,
                                                   double *sums) {
  extern __shared__ d2 cg_lds[];
  __shared__ double al[kMaxNev], wsum[kMaxNev], sb[kCgTile];
  __shared__ double sh[3][256];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int nev = p.nev, h = ld / 2;
  d2 *sV = cg_lds, *sR = sV + kCgTile * h, *sZ = sR + kCgTile * h;
  const double *fV = reinterpret_cast<const double *>(sV);
  const double *fR = reinterpret_cast<const double *>(sR);
  const double *fZ = reinterpret_cast<const double *>(sZ);
  const int np = nev * nev, ng = 256 / np;
  const int grp = t / np, pr = t - grp * np;
  const int j = pr / nev, k = pr - j * nev;
  const bool live = grp < ng;
  double m = 0.0, g = 0.0, rz = 0.0;
  // this thread's column of the state, read ahead of the partials
  const bool col = pap && t < nev;
  const int done0 = col ? st->done[t] : 1;
  const double rz0 = col ? st->rz[t] : 0.0;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t r0 = tile * kCgTile;
    const int rows = (int)min((int64_t)kCgTile, n - r0);
    // all loads of the tile first: the first tile's are in flight while the
    // alphas are formed
    d2 r[kItems], v[kItems], x[kItems], pv[kItems], ap[kItems];
    double di[kItems], bi[kItems];
    int cc[kItems];
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      const int e = t + 256 * u;
      if (e < rows * h) {
        const int row = e / h;
        const int64_t i = r0 + row, q = r0 * h + e;
        cc[u] = 2 * (e - row * h);
        r[u] = reinterpret_cast<const d2 *>(R)[q];
        v[u] = reinterpret_cast<const d2 *>(Vp)[q];
        di[u] = d[i];
        bi[u] = bd ? bd[i] : 1.0;
        if (pap) {
          x[u] = reinterpret_cast<const d2 *>(MU)[q];
          pv[u] = reinterpret_cast<const d2 *>(P)[q];
          ap[u] = reinterpret_cast<const d2 *>(AP)[q];
        }
      }
    }
    if (pap && tile == blockIdx.x) {
      // one wave per column
      for (int c = wave; c < nev; c += 4) {
        const double *q = pap + (int64_t)c * kMaxNormBlocks;
        double a = 0.0;
#pragma unroll 4
        for (int b = lane; b < nparts; b += 64) a += q[b];
        for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off);
        if (lane == 0) wsum[c] = a;
      }
      __syncthreads();
      if (t < kMaxNev) {
        double a = 0.0;
        int broke = 0, any = 0;
        if (!done0) {
          const double q = wsum[t];
          if (q > 0.0) {
            a = rz0 / q;
            any = 1;
          } else {
            broke = 1;
          }
        }
        al[t] = a;
        if (blockIdx.x == 0) {
          alpha_out->broke[t] = broke;
          const unsigned long long who = __ballot(any);
          if (t == 0) alpha_out->any = who ? 1 : 0;
        }
      }
      __syncthreads();
    }
    if (t < rows) sb[t] = bd ? bd[r0 + t] : 1.0;
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      const int e = t + 256 * u;
      if (e < rows * h) {
        const int c = cc[u];
        const int64_t q = r0 * h + e;
        if (pap) {
          const d2 a = {al[c], al[c + 1]};
          reinterpret_cast<d2 *>(MU)[q] = x[u] + a * pv[u];
          r[u] -= a * ap[u];
          reinterpret_cast<d2 *>(R)[q] = r[u];
        }
        sV[e] = v[u];
        sR[e] = r[u];
        // padding columns: r = 0 there
        sZ[e] = d2{r[u][0] / cg_diag(di[u], bi[u], p.lam[c]),
                   c + 1 < nev ? r[u][1] / cg_diag(di[u], bi[u], p.lam[c + 1]) : 0.0};
      }
    }
    __syncthreads();
    if (live) {
#pragma unroll 4
      for (int row = grp; row < rows; row += ng) {
        const double vv = fV[row * ld + j], z = fZ[row * ld + k], rr = fR[row * ld + k];
        m = fma(vv, sb[row] * z, m);
        g = fma(vv, rr, g);
        rz = fma(rr, z, rz);
      }
    }
    __syncthreads();
  }
  sh[0][t] = live ? m : 0.0;
  sh[1][t] = live ? g : 0.0;
  sh[2][t] = live ? rz : 0.0;
  __syncthreads();
  if (t < np) {
    double a = 0.0, b = 0.0, c = 0.0;
#pragma unroll 4
    for (int q = 0; q < ng; ++q) {
      a += sh[0][q * np + t];
      b += sh[1][q * np + t];
      c += sh[2][q * np + t];
    }
    sums[(int64_t)t * gridDim.x + blockIdx.x] = a;
    sums[(int64_t)(np + t) * gridDim.x + blockIdx.x] = b;
    if (t < nev) sums[(int64_t)(2 * np + t) * gridDim.x + blockIdx.x] = c;
  }
}

// red[v] = sum of value v over the nb blocks, one block per value, fixed order
__global__ __launch_bounds__(256) void k_cg_reduce(const double *sums, int nb, double *red) {
  __shared__ double sh[4];
  const double *x = sums + (int64_t)blockIdx.x * nb;
  double a = 0.0;
  for (int b = threadIdx.x; b < nb; b += 256) a += x[b];
  for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) red[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// p = z - V M + beta p, and the state after the step: r^T z', beta and the
// convergence test r^T z' <= tol^2 f^T J f (init: the first preconditioned
// residual, p = z').
__global__ __launch_bounds__(256) void k_cg_direction(double *P, const double *R,
                                                      const double *Vp, const double *red,
                                                      const CgState *st, const CgAlpha *alpha,
                                                      CgState *st_out, const double *d,
                                                      const double *bd, AdjParams p, int64_t n,
                                                      int ld, double tol2, int init) {
  __shared__ double sM[2 * kMaxNev * kMaxNev], beta[kMaxNev];
  const int t = threadIdx.x, nev = p.nev, np = nev * nev, h = ld / 2;
  // a block takes rc rows at a time, one pair of columns per thread; its
  // first elements and the state are read ahead of the small sums
  const int rc = 256 / h, row = t / h, c = 2 * (t - row * h);
  const int64_t i0 = row < rc ? (int64_t)blockIdx.x * rc + row : n;
  d2 r0 = {0.0, 0.0}, q0 = {0.0, 0.0};
  double d0 = 1.0, b0 = 1.0;
  if (i0 < n) {
    r0 = reinterpret_cast<const d2 *>(R)[i0 * h + (c >> 1)];
    if (!init) q0 = reinterpret_cast<const d2 *>(P)[i0 * h + (c >> 1)];
    d0 = d[i0];
    if (bd) b0 = bd[i0];
  }
  const bool col = !init && t < nev;
  const double rz0_old = col ? st->rz0[t] : 0.0, rz_old = col ? st->rz[t] : 1.0;
  const int done_old = col ? st->done[t] | alpha->broke[t] : 0;
  for (int e = t; e < 2 * np; e += 256) sM[e] = red[e];
  double rz = t < nev ? red[2 * np + t] : 0.0;
  __syncthreads();
  if (t < nev) {
#pragma unroll 4
    for (int j = 0; j < nev; ++j) rz = fma(-sM[np + j * nev + t], sM[j * nev + t], rz);
    double rz0, b = 0.0;
    int done;
    if (init) {
      rz0 = rz;
      done = !(rz > 0.0);
    } else {
      rz0 = rz0_old;
      done = done_old || rz <= tol2 * rz0;
      b = done ? 0.0 : rz / rz_old;
    }
    beta[t] = b;
    if (blockIdx.x == 0) {
      st_out->rz[t] = rz;
      st_out->rz0[t] = rz0;
      st_out->done[t] = done;
    }
  } else if (t < kMaxNev) {
    beta[t] = 0.0;
  }
  if (blockIdx.x == 0 && t == 0) {
    int broke = init ? 0 : st->breakdown;
    if (!init)
      for (int c = 0; c < nev; ++c) broke |= alpha->broke[c];
    st_out->breakdown = broke;
    st_out->iters = init ? 0 : st->iters + alpha->any;
  }
  __syncthreads();
  const bool two = c + 1 < nev;
  for (int64_t i = i0; i < n; i += (int64_t)gridDim.x * rc) {
    const int64_t e = i * h + (c >> 1);
    d2 r = r0, q = q0;
    double di = d0, bi = b0;
    if (i != i0) {
      r = reinterpret_cast<const d2 *>(R)[e];
      if (!init) q = reinterpret_cast<const d2 *>(P)[e];
      di = d[i];
      bi = bd ? bd[i] : 1.0;
    }
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
    for (int j = 0; j < nev; ++j) {
      const double v = Vp[i * ld + j];
      s0 = fma(v, sM[j * nev + c], s0);
      if (two) s1 = fma(v, sM[j * nev + c + 1], s1);
    }
    d2 o = {r[0] / cg_diag(di, bi, p.lam[c]) - s0,
            two ? r[1] / cg_diag(di, bi, p.lam[c + 1]) - s1 : 0.0};
    if (!init) {
      o[0] += beta[c] * q[0];
      if (two) o[1] += beta[c + 1] * q[1];
    }
    reinterpret_cast<d2 *>(P)[e] = o;
  }
}

// Edge gradient: one wavefront per row, lanes over its entries.
template <typename IdxT>
__global__ __launch_bounds__(256) void k_edge_grad(int64_t n, const IdxT *rp,
                                                   const int32_t *col, const double *V,
                                                   const double *MU, int ldmu, Small M1,
                                                   Small M2, AdjParams p, int use_mu,
                                                   double *grad) {
  __shared__ double s1[kMaxNev * kMaxNev], s2[kMaxNev * kMaxNev];
  const int nev = p.nev;
  for (int e = threadIdx.x; e < nev * nev; e += blockDim.x) {
    s1[e] = M1.a[e];
    s2[e] = M2.a[e];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x / 64;
  for (int64_t i = (int64_t)blockIdx.x * wpb + threadIdx.x / 64; i < n;
       i += (int64_t)gridDim.x * wpb) {
    double a[kMaxNev], ci[kMaxNev];
    for (int k = 0; k < nev; ++k) {
      a[k] = V[i * nev + k];
      ci[k] = use_mu ? MU[i * ldmu + k] : 0.0;
    }
    for (int64_t q = (int64_t)rp[i] + lane; q < (int64_t)rp[i + 1]; q += 64) {
      int64_t j = col[q];
      double b[kMaxNev], df[kMaxNev];
      for (int k = 0; k < nev; ++k) {
        b[k] = V[j * nev + k];
        df[k] = a[k] - b[k];
      }
      double g1 = 0.0, g2 = 0.0;
      for (int k = 0; k < nev; ++k) {
        double t1 = 0.0, ta = 0.0, tb = 0.0;
        for (int l = 0; l < nev; ++l) {
          t1 += s1[k * nev + l] * df[l];
          ta += s2[k * nev + l] * a[l];
          tb += s2[k * nev + l] * b[l];
        }
        g1 += df[k] * t1;
        g2 += a[k] * ta + b[k] * tb;
      }
      double g3 = 0.0;
      if (use_mu)
        for (int k = 0; k < nev; ++k) {
          double cj = MU[j * ldmu + k];
          g3 -= (ci[k] - cj) * df[k];
          if (p.gen) g3 += p.lam[k] * (ci[k] * a[k] + cj * b[k]);
        }
      grad[q] = g1 - g2 + g3;
    }
  }
}

// normalized problem: X = D^-1/2 Y, GX = D^1/2 GY, t_i = sum_k GY_ik Y_ik / (2 d_i)
__global__ void k_norm_prep(const double *Y, const double *GY, const double *d, int64_t n,
                            int nev, double *X, double *GX, double *t) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double di = d[i];
    const double r = sqrt(di);
    double acc = 0.0;
    for (int k = 0; k < nev; ++k) {
      const double y = Y[i * nev + k];
      X[i * nev + k] = y / r;
      if (GY) {
        const double gy = GY[i * nev + k];
        GX[i * nev + k] = gy * r;
        acc += gy * y;
      }
    }
    t[i] = acc / (2.0 * di);
  }
}

// grad[q] += t_i + t_j for every CSR entry q = (i, j); one wave per row
template <typename IdxT>
__global__ __launch_bounds__(256) void k_add_vertex_terms(int64_t n, const IdxT *rp,
                                                          const int32_t *col, const double *t,
                                                          double *grad) {
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x / 64;
  for (int64_t i = (int64_t)blockIdx.x * wpb + threadIdx.x / 64; i < n;
       i += (int64_t)gridDim.x * wpb) {
    const double ti = t[i];
    for (int64_t q = (int64_t)rp[i] + lane; q < (int64_t)rp[i + 1]; q += 64)
      grad[q] += ti + t[col[q]];
  }
}

constexpr int kSmallBlocks = 1024;
// CG steps between host reads of the flags, at most.  A batch costs some 10 us
// beside its steps; the flags are read one batch behind, so up to two batches
// are run past convergence, at full cost.  The first batches are short (2 steps
// up to step 8, 4 up to step 16: they may be the only ones), and so are all of
// them where a step takes longer than 10 such batches, from kCgLarge values per
// block on.  With 8 steps throughout: 2 M rows, 7 steps needed, 1 column
// 3.10 ms, now 2.69; 9 columns 19.7 ms, now 15.6; 31,680 rows, 2 steps needed,
// 5 columns 0.56 ms, now 0.31.
constexpr int kCgCheck = 8;
constexpr int64_t kCgLarge = 1 << 22;

}  // namespace

size_t adjoint_scratch_bytes(int64_t n, int nev) {
  const int ld = padded_ld(nev, 8);
  size_t blk = align_up(sizeof(double) * n * nev, 256);
  size_t blkp = align_up(sizeof(double) * n * ld, 256);
  // 2 blocks of the normalized transform and t, 5 padded CG blocks (V, mu,
  // r, p, Ap), the product's dot partials, Gram and projection partials
  return 2 * blk + align_up(sizeof(double) * n, 256) + 5 * blkp +
         align_up(sizeof(double) * 2 * kMaxNev * kMaxNormBlocks, 256) +
         align_up(sizeof(double) * kSmallBlocks * kMaxNev * kMaxNev, 256) +
         align_up(sizeof(double) * kCgBlocks * cg_sums(kMaxNev), 256) +
         align_up(sizeof(double) * cg_sums(kMaxNev), 256) +
         align_up(sizeof(double) * kMaxNev * kMaxNev, 256) * 2 +
         align_up(2 * sizeof(CgState), 256) + align_up(sizeof(CgAlpha), 256) + 4096;
}

int eig_backward(sphx_graph *g, const SpmmPlan &plan, int problem, int nev,
                 const double *lam, const double *V, const double *g_vals, const double *gV,
                 double cg_tol, int cg_max_iter, const double *d64, double *grad,
                 void *scratch, void *pinned, hipStream_t s, std::string *err,
                 int *cg_iters, double *cg_relres) {
  const int64_t n = g->n;
  Arena a;
  a.base = static_cast<char *>(scratch);
  size_t blk = (size_t)n * nev;
  if (cg_iters) *cg_iters = 0;
  if (cg_relres) *cg_relres = 0.0;
  if (problem == SPHX_NORMALIZED) {
    double *Xn = a.take<double>(blk);
    double *GXn = a.take<double>(blk);
    double *t = a.take<double>(n);
    hipLaunchKernelGGL(k_norm_prep, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, V, gV, d64,
                       n, nev, Xn, GXn, t);
    int r = eig_backward(g, plan, SPHX_GENERALIZED, nev, lam, Xn, g_vals, gV ? GXn : nullptr,
                         cg_tol, cg_max_iter, d64, grad, a.base + align_up(a.off, 256), pinned, s,
                         err, cg_iters, cg_relres);
    if (r < 0 || !gV) return r;
    unsigned gb = grid_for(n, 4, 1 << 16);
    if (g->rp64)
      hipLaunchKernelGGL((k_add_vertex_terms<int64_t>), dim3(gb), dim3(256), 0, s, n,
                         (const int64_t *)g->rowptr, g->col, (const double *)t, grad);
    else
      hipLaunchKernelGGL((k_add_vertex_terms<int32_t>), dim3(gb), dim3(256), 0, s, n,
                         (const int32_t *)g->rowptr, g->col, (const double *)t, grad);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
      *err = "adjoint kernel failed";
      return SPHX_E_HIP;
    }
    return r;
  }
  const bool gen = problem == SPHX_GENERALIZED;
  const double *bd = gen ? d64 : nullptr;
  const int ld = padded_ld(nev, 8);
  const size_t blkp = (size_t)n * ld;
  double *Vp = a.take<double>(blkp);
  double *MU = a.take<double>(blkp);
  double *Rr = a.take<double>(blkp);
  double *Pp = a.take<double>(blkp);
  double *AP = a.take<double>(blkp);
  double *pap_parts = a.take<double>((size_t)2 * kMaxNev * kMaxNormBlocks);
  double *parts = a.take<double>((size_t)kSmallBlocks * kMaxNev * kMaxNev);
  double *sums = a.take<double>((size_t)kCgBlocks * cg_sums(kMaxNev));
  double *red = a.take<double>(cg_sums(kMaxNev));
  double *Mdev = a.take<double>(kMaxNev * kMaxNev);
  double *Mdev2 = a.take<double>(kMaxNev * kMaxNev);
  CgState *st = a.take<CgState>(2);        // the state before and after a step
  CgAlpha *alpha = a.take<CgAlpha>(1);
  const int64_t rpb = ceil_div(n, kSmallBlocks);
  const int nsb = (int)ceil_div(n, rpb);
  const unsigned gew = grid_for((int64_t)blkp, 256, 4096);
  auto gram_small = [&](const double *A, int lda, const double *B, int ldb, const double *w,
                        double *out) {
    hipLaunchKernelGGL(k_small_gram, dim3(nsb), dim3(256), 0, s, A, lda, B, ldb, w, n, nev,
                       parts, rpb);
    hipLaunchKernelGGL(k_small_sum, dim3(1), dim3(1024), 0, s, (const double *)parts, nsb,
                       nev * nev, out);
  };
  AdjParams prm;
  prm.nev = nev;
  prm.gen = gen ? 1 : 0;
  for (int k = 0; k < kMaxNev; ++k) prm.lam[k] = k < nev ? lam[k] : 0.0;
  Small M1{}, M2{};
  for (int k = 0; k < nev; ++k) {
    double gl = g_vals ? g_vals[k] : 0.0;
    M1.a[k * nev + k] += gl;
    if (gen) M2.a[k * nev + k] += lam[k] * gl;
  }
  int status = SPHX_OK;
  bool use_mu = false;
  if (gV) {
    // G^T V: GtV[j * nev + k] = sum_i g_ij v_ik  -> c_kl = GtV[k][l] / (lam_k - lam_l)
    gram_small(gV, nev, V, nev, nullptr, Mdev);
    double gtv[kMaxNev * kMaxNev];
    if (hipMemcpyAsync(gtv, Mdev, sizeof(double) * nev * nev, hipMemcpyDeviceToHost, s) !=
            hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return SPHX_E_HIP;
    for (int k = 0; k < nev; ++k)
      for (int l = 0; l < nev; ++l) {
        if (l == k) {
          if (gen) M2.a[k * nev + k] += 0.5 * gtv[k * nev + k];
          continue;
        }
        double c = gtv[k * nev + l] / (lam[k] - lam[l]);
        M1.a[k * nev + l] += c;
        if (gen) M2.a[k * nev + l] += lam[k] * c;
      }
    // ---- mu: projected PCG on all columns, scalars on the device
    use_mu = true;
    hipLaunchKernelGGL(k_pad_cols, dim3(gew), dim3(256), 0, s, V, nev, Vp, ld, n);
    // r0 = g - B V (V^T g); mu0 = 0
    gram_small(V, nev, gV, nev, nullptr, Mdev);
    hipLaunchKernelGGL(k_project_rhs, dim3(gew), dim3(256), 0, s, gV, (const double *)Vp, bd,
                       (const double *)Mdev, n, nev, ld, Rr);
    hipLaunchKernelGGL(k_pad_cols, dim3(gew), dim3(256), 0, s, (const double *)nullptr, 0, MU,
                       ld, n);
    const int64_t ntiles = ceil_div(n, kCgTile);
    const unsigned gu = (unsigned)std::min<int64_t>(ntiles, kCgBlocks);
    const size_t lds = 3 * sizeof(double) * kCgTile * ld;
    const unsigned gd = grid_for(n, 256 / (ld / 2), 4096);
    // after the product: np partials of p^T A p (0: the first residual)
    auto step_tail = [&](int np, int cur) {
      auto update = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(gu), dim3(256), lds, s, MU, Rr, (const double *)Pp,
                           (const double *)AP, (const double *)Vp,
                           np ? (const double *)pap_parts : (const double *)nullptr, np,
                           (const CgState *)(st + cur), alpha, d64, bd, prm, n, ld, ntiles,
                           sums);
      };
      if (ld <= 8) update(k_cg_update<1>);
      else update(k_cg_update<2>);
      hipLaunchKernelGGL(k_cg_reduce, dim3(cg_sums(nev)), dim3(256), 0, s, (const double *)sums,
                         (int)gu, red);
      hipLaunchKernelGGL(k_cg_direction, dim3(gd), dim3(256), 0, s, Pp, (const double *)Rr,
                         (const double *)Vp, (const double *)red, (const CgState *)(st + cur),
                         (const CgAlpha *)alpha, st + (np ? 1 - cur : cur), d64, bd, prm, n, ld,
                         cg_tol * cg_tol, np ? 0 : 1);
    };
    EpiShiftDotP<double> ep{AP, ld, nullptr, bd};
    double *lam_dev = Mdev2;   // lam_k on the device for the product's epilogue
    if (hipMemcpyAsync(lam_dev, prm.lam, sizeof(double) * kMaxNev, hipMemcpyHostToDevice, s) !=
        hipSuccess) {
      *err = "adjoint: copy failed";
      return SPHX_E_HIP;
    }
    ep.lam = lam_dev;
    int cur = 0;
    step_tail(0, cur);
    // Batches of up to kCgCheck steps; the state after a batch is copied to pinned
    // memory behind it and read while the next batch runs (steps past the
    // last column's convergence leave x as it is).
    struct Events {
      hipEvent_t e[2] = {nullptr, nullptr};
      ~Events() {
        for (auto x : e)
          if (x) (void)hipEventDestroy(x);
      }
    } evs;
    for (auto &x : evs.e)
      if (hipEventCreateWithFlags(&x, hipEventDisableTiming) != hipSuccess) {
        *err = "adjoint: event creation failed";
        return SPHX_E_HIP;
      }
    static_assert(2 * sizeof(CgState) <= kPinnedSmallBytes, "pinned states");
    CgState *hp = static_cast<CgState *>(pinned);
    CgState hs{};
    const bool large = n * ld >= kCgLarge;
    int it = 0, batches = 0, seen = 0;
    bool all = false;
    while (seen < batches || it < cg_max_iter) {
      if (it < cg_max_iter) {
        const int batch = large || it < 8 ? 2 : (it < 16 ? 4 : kCgCheck);
        const int steps = std::min(batch, cg_max_iter - it);
        for (int q = 0; q < steps; ++q) {
          int np = 0;
          int r = vspmm_shiftdot<double>(g, plan, Pp, ld, nev, ep, pap_parts, &np, s);
          if (r != SPHX_OK) {
            (void)hipStreamSynchronize(s);
            *err = "adjoint CG product failed";
            return r;
          }
          if (np > kCgParts) {
            hipLaunchKernelGGL(k_cg_pap, dim3(nev), dim3(1024), 0, s,
                               (const double *)pap_parts, np, pap_parts);
            np = 1;
          }
          step_tail(np, cur);
          cur = 1 - cur;
        }
        it += steps;
        const int slot = batches & 1;
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(hp + slot, st + cur, sizeof(CgState), hipMemcpyDeviceToHost, s) !=
                hipSuccess ||
            hipEventRecord(evs.e[slot], s) != hipSuccess) {
          *err = "adjoint CG failed";
          return SPHX_E_HIP;
        }
        ++batches;
        if (batches - seen < 2 && it < cg_max_iter) continue;
      }
      if (hipEventSynchronize(evs.e[seen & 1]) != hipSuccess) {
        *err = "adjoint CG failed";
        return SPHX_E_HIP;
      }
      hs = hp[seen & 1];
      ++seen;
      all = true;
      for (int k = 0; k < nev; ++k) all = all && hs.done[k];
      if (all) break;
    }
    double worst = 0.0;
    for (int k = 0; k < nev; ++k)
      if (hs.rz0[k] > 0.0) worst = std::max(worst, std::sqrt(std::max(0.0, hs.rz[k] / hs.rz0[k])));
    if (cg_iters) *cg_iters = hs.iters;
    if (cg_relres) *cg_relres = worst;
    if (!all) status = SPHX_NOT_CONVERGED;
    if (hs.breakdown) {
      *err = "adjoint CG: p^T A p not positive (eigenvalues not separated from the rest)";
      status = SPHX_NOT_CONVERGED;
    }
  }
  unsigned gb = grid_for(n, 4, 1 << 16);
  if (g->rp64)
    hipLaunchKernelGGL((k_edge_grad<int64_t>), dim3(gb), dim3(256), 0, s, n,
                       (const int64_t *)g->rowptr, g->col, V, (const double *)MU, ld, M1, M2,
                       prm, use_mu ? 1 : 0, grad);
  else
    hipLaunchKernelGGL((k_edge_grad<int32_t>), dim3(gb), dim3(256), 0, s, n,
                       (const int32_t *)g->rowptr, g->col, V, (const double *)MU, ld, M1, M2,
                       prm, use_mu ? 1 : 0, grad);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
    *err = "adjoint kernel failed";
    return SPHX_E_HIP;
  }
  return status;
}

}  // namespace sphx
