// Laplacian product y = L_C x of a single column for a CSR graph (Eq. 2 with
// weights), summed per row in difference form y_i = sum_j w_ij (x_i - x_j);
// wider blocks take the vector-row kernels.
//
// Rows are split by degree:
//   rows of the lower degree classes: one lane per row;
//   rows of the highest class below the hubs: one wavefront per row, its lanes
//     striding over the neighbours, combined by a butterfly;
//   hub rows (deg > kHubDeg): kHubChunk-entry chunks, one wavefront each, the
//     partial sums of a row combined by a wavefront in a second kernel.
// All sums are in a fixed order, so results are bitwise reproducible.  The
// lanes of a chunk have 8 entries each, and a row of 16 M neighbours 31,250
// chunks: with the lanes added one after the other and the chunks by one lane
// (as long as hubs began at 16384 neighbours and chunks had 4096 entries, that
// was little beside the gathers) a call on a star of 16 M leaves took 14.1 ms,
// now 1.9, and 25 steps on R-MAT 12 (FP32) 1.26 ms, now 0.79.
//
// Epilogues fused into the product:
//   Store     y = acc
//   Cheb      one step of the Chebyshev iteration for L h = r (Sec. 5.2):
//             out = xs + alpha (xs - prev) + beta s_i (r - L xs), xs = scale x,
//             s_i = 1 or 1/d_i (generalized).
#include "kernels.h"

namespace sphx {
namespace {

template <typename IdxT, typename WT>
struct Csr {
  const IdxT *rp;
  const int32_t *col;
  const WT *w;
};

template <typename T>
__device__ __forceinline__ T fma_t(T a, T b, T c) {
  if constexpr (std::is_same_v<T, float>) return fmaf(a, b, c);
  else return fma(a, b, c);
}

// Sum over entries k0, k0+step, ... < k1 of w_k (xi - x_{col[k]}).
template <typename T, typename IdxT, typename WT>
__device__ __forceinline__ T row_acc(const Csr<IdxT, WT> &A, int64_t k0, int64_t k1, int step,
                                     const T *__restrict__ X, T xi) {
  T acc0 = T(0), acc1 = T(0);
  int64_t k = k0;
  // two independent gathers in flight per iteration
  for (; k + step < k1; k += 2 * step) {
    const T x0 = X[A.col[k]];
    const T x1 = X[A.col[k + step]];
    if constexpr (std::is_same_v<WT, Unit>) {
      acc0 += xi - x0;
      acc1 += xi - x1;
    } else {
      acc0 = fma_t(T(A.w[k]), xi - x0, acc0);
      acc1 = fma_t(T(A.w[k + step]), xi - x1, acc1);
    }
  }
  if (k < k1) {
    const T x0 = X[A.col[k]];
    if constexpr (std::is_same_v<WT, Unit>) acc0 += xi - x0;
    else acc0 = fma_t(T(A.w[k]), xi - x0, acc0);
  }
  return acc0 + acc1;
}

// ------------------------------------------------------------- epilogues
template <typename T>
struct EpiStore {
  T *Y;
  __device__ void operator()(int64_t i, T, T acc) const { Y[i] = acc; }
};

template <typename T>
struct EpiCheb {
  EpiChebP<T> p;
  __device__ void operator()(int64_t i, T xi, T acc) const {
    double xs = p.src_scale * double(xi);
    double pv = p.prev ? p.prev_scale * double(p.prev[i]) : 0.0;
    double si = p.dinv ? p.dinv[i] : 1.0;
    double res = double(p.R[i]) - p.src_scale * double(acc);
    p.OUT[i] = T(xs + p.alpha * (xs - pv) + p.beta * si * res);
  }
};

// ---------------------------------------------------------------- kernels
template <typename T, typename IdxT, typename WT, typename Epi>
__global__ __launch_bounds__(256) void k_spmm_rows(Csr<IdxT, WT> A,
                                                   const int32_t *__restrict__ rows,
                                                   int64_t nrows, const T *__restrict__ X,
                                                   Epi epi) {
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < nrows;
       r += (int64_t)gridDim.x * 256) {
    const int64_t i = rows ? rows[r] : r;
    const T xi = X[i];
    epi(i, xi, row_acc<T>(A, (int64_t)A.rp[i], (int64_t)A.rp[i + 1], 1, X, xi));
  }
}

// Sum over the wavefront, in every lane.
template <typename T>
__device__ __forceinline__ T wave_total(T v) {
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

template <typename T, typename IdxT, typename WT, typename Epi>
__global__ __launch_bounds__(256) void k_spmm_wave(Csr<IdxT, WT> A,
                                                   const int32_t *__restrict__ rows,
                                                   int64_t nrows, const T *__restrict__ X,
                                                   Epi epi) {
  const int lane = threadIdx.x & (kWave - 1);
  for (int64_t r = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave; r < nrows;
       r += (int64_t)gridDim.x * 4) {
    const int64_t i = rows[r];
    const T xi = X[i];
    const T tot = wave_total(
        row_acc<T>(A, (int64_t)A.rp[i] + lane, (int64_t)A.rp[i + 1], kWave, X, xi));
    if (lane == 0) epi(i, xi, tot);
  }
}

// out[q]: the sum of chunk q
template <typename T, typename IdxT, typename WT>
__global__ __launch_bounds__(256) void k_spmm_hub_partial(
    Csr<IdxT, WT> A, const int32_t *__restrict__ hub_chunk_begin, int64_t n_hub,
    const int64_t *__restrict__ k0s, const int32_t *__restrict__ chunk_row,
    const T *__restrict__ X, double *out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t n_chunks = hub_chunk_begin[n_hub];
  for (int64_t q = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave; q < n_chunks;
       q += (int64_t)gridDim.x * 4) {
    const int64_t i = chunk_row[q], k0 = k0s[q];
    const int64_t k1 = min(k0 + kHubChunk, (int64_t)A.rp[i + 1]);
    const T tot = wave_total(row_acc<T>(A, k0 + lane, k1, kWave, X, X[i]));
    if (lane == 0) out[q] = double(tot);
  }
}

// one wavefront per hub, lanes over its chunks
template <typename T, typename Epi>
__global__ __launch_bounds__(256) void k_spmm_hub_combine(
    const int32_t *__restrict__ hub_rows, const int32_t *__restrict__ hub_chunk_begin,
    int64_t n_hub, const double *__restrict__ part, const T *__restrict__ X, Epi epi) {
  const int lane = threadIdx.x & (kWave - 1);
  for (int64_t h = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave; h < n_hub;
       h += (int64_t)gridDim.x * 4) {
    const int64_t i = hub_rows[h];
    T acc = T(0);
#pragma unroll 4
    for (int64_t q = hub_chunk_begin[h] + lane; q < hub_chunk_begin[h + 1]; q += kWave)
      acc += T(part[q]);
    const T tot = wave_total(acc);
    if (lane == 0) epi(i, X[i], tot);
  }
}

// --------------------------------------------------------------- dispatch
constexpr int kRowBlocks = 2048;
constexpr int kWaveBlocks = 1024;
constexpr int kHubBlocks = 64;

template <typename T, typename IdxT, typename WT, typename Epi>
void run_all(const Csr<IdxT, WT> &A, int64_t n, const SpmmPlan &plan, const T *X,
             const Epi &epi, hipStream_t s) {
  if (!plan.binned) {
    hipLaunchKernelGGL((k_spmm_rows<T, IdxT, WT, Epi>), dim3(grid_for(n, 256, kRowBlocks)),
                       dim3(256), 0, s, A, (const int32_t *)nullptr, n, X, epi);
    return;
  }
  // rows of the first kNumBins - 1 classes, whose lists lie one behind the
  // other: one lane per row; the last class: one wavefront per row
  int64_t nshort = 0;
  for (int c = 0; c < kNumBins - 1; ++c) nshort += plan.nrows[c];
  if (nshort > 0)
    hipLaunchKernelGGL((k_spmm_rows<T, IdxT, WT, Epi>), dim3(grid_for(nshort, 256, kRowBlocks)),
                       dim3(256), 0, s, A, plan.rows[0], nshort, X, epi);
  if (plan.nrows[kNumBins - 1] > 0)
    hipLaunchKernelGGL((k_spmm_wave<T, IdxT, WT, Epi>),
                       dim3(grid_for(plan.nrows[kNumBins - 1], 4, kWaveBlocks)), dim3(256), 0,
                       s, A, plan.rows[kNumBins - 1], plan.nrows[kNumBins - 1], X, epi);
  if (plan.n_hub > 0) {
    hipLaunchKernelGGL((k_spmm_hub_partial<T, IdxT, WT>),
                       dim3(grid_for(plan.n_chunks, 4, kWaveBlocks)), dim3(256), 0, s, A,
                       plan.hub_chunk_begin, plan.n_hub, plan.chunk_k0, plan.chunk_row, X,
                       plan.hub_partial);
    hipLaunchKernelGGL((k_spmm_hub_combine<T, Epi>), dim3(grid_for(plan.n_hub, 4, kHubBlocks)),
                       dim3(256), 0, s, plan.hub_rows, plan.hub_chunk_begin, plan.n_hub,
                       (const double *)plan.hub_partial, X, epi);
  }
}

template <typename T, typename Epi>
int dispatch(sphx_graph *g, const SpmmPlan &plan, const T *X, const Epi &epi, hipStream_t s) {
  auto go = [&](auto idx_tag, auto w_tag) {
    using IdxT = decltype(idx_tag);
    using WT = decltype(w_tag);
    Csr<IdxT, WT> A{static_cast<const IdxT *>(g->rowptr), g->col,
                    static_cast<const WT *>(g->w)};
    run_all<T>(A, g->n, plan, X, epi, s);
  };
  if (g->rp64) {
    if (g->wdt == SPHX_UNIT) go(int64_t{}, Unit{});
    else if (g->wdt == SPHX_F32) go(int64_t{}, float{});
    else go(int64_t{}, double{});
  } else {
    if (g->wdt == SPHX_UNIT) go(int32_t{}, Unit{});
    else if (g->wdt == SPHX_F32) go(int32_t{}, float{});
    else go(int32_t{}, double{});
  }
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? SPHX_OK : SPHX_E_HIP;
}

}  // namespace

template <typename T>
int spmm_store(sphx_graph *g, const SpmmPlan &plan, const T *X, T *Y, hipStream_t s) {
  return dispatch(g, plan, X, EpiStore<T>{Y}, s);
}

template <typename T>
int spmm_cheb(sphx_graph *g, const SpmmPlan &plan, const T *X, EpiChebP<T> epi, hipStream_t s) {
  return dispatch(g, plan, X, EpiCheb<T>{epi}, s);
}

template int spmm_store<float>(sphx_graph *, const SpmmPlan &, const float *, float *,
                               hipStream_t);
template int spmm_store<double>(sphx_graph *, const SpmmPlan &, const double *, double *,
                                hipStream_t);
template int spmm_cheb<float>(sphx_graph *, const SpmmPlan &, const float *, EpiChebP<float>,
                              hipStream_t);
template int spmm_cheb<double>(sphx_graph *, const SpmmPlan &, const double *,
                               EpiChebP<double>, hipStream_t);

}  // namespace sphx
