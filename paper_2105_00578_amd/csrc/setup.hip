// Graph validation, degrees and the degree-binned row plan of the Laplacian
// product.  Degrees are the diagonal of L_C (Eq. 2, weighted); the regular /
// irregular classification is max degree / average degree <= 10 (Sec. 6.1).
#include <algorithm>

#include "fixed.h"
#include "kernels.h"

namespace sphx {
namespace {

enum : int {
  F_BAD_GRAPH = 1,
  F_SELF_LOOP = 2,
  F_NOT_SYM = 4,
  F_BAD_WEIGHT = 8,
};

// One wavefront per row; lanes stride over the row's entries.
template <typename IdxT, typename WT>
__global__ __launch_bounds__(256) void k_validate(int64_t n, int64_t nnz,
                                                  const IdxT *rp, const int32_t *col,
                                                  const WT *w, const int32_t *vwgt,
                                                  int *flags) {
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x / 64;
  int f = 0;
  for (int64_t i = (int64_t)blockIdx.x * wpb + threadIdx.x / 64; i < n;
       i += (int64_t)gridDim.x * wpb) {
    int64_t b = rp[i], e = rp[i + 1];
    if (lane == 0) {
      if (e < b || b < 0 || e > nnz) f |= F_BAD_GRAPH;
      if (i == 0 && b != 0) f |= F_BAD_GRAPH;
      if (i == n - 1 && e != nnz) f |= F_BAD_GRAPH;
      if (vwgt && vwgt[i] < 1) f |= F_BAD_WEIGHT;
    }
    if (e < b || b < 0 || e > nnz) continue;
    for (int64_t k = b + lane; k < e; k += 64) {
      int64_t j = col[k];
      if (j < 0 || j >= n) { f |= F_BAD_GRAPH; continue; }
      if (j == i) f |= F_SELF_LOOP;
      if (k > b && col[k - 1] >= col[k]) f |= F_BAD_GRAPH;
      if constexpr (!std::is_same_v<WT, Unit>) {
        WT wk = w[k];
        if (!(wk > WT(0)) || !(wk < WT(INFINITY))) f |= F_BAD_WEIGHT;
      }
      // symmetric partner (i in row j), binary search over row j, whose
      // bounds are checked first (a malformed row_ptr must not send the
      // search outside col[0..nnz))
      int64_t lo = rp[j], hi = rp[j + 1] - 1;
      if (lo < 0 || hi + 1 < lo || hi + 1 > nnz) { f |= F_BAD_GRAPH; continue; }
      bool found = false;
      int64_t kk = -1;
      while (lo <= hi) {
        int64_t mid = (lo + hi) >> 1;
        int64_t cm = col[mid];
        if (cm == i) { found = true; kk = mid; break; }
        if (cm < i) lo = mid + 1; else hi = mid - 1;
      }
      if (!found) f |= F_NOT_SYM;
      else if constexpr (!std::is_same_v<WT, Unit>) {
        if (!(w[kk] == w[k])) f |= F_NOT_SYM;
      }
    }
  }
  if (f) atomicOr(flags, f);
}

// Block statistics of the rows' neighbour counts and weighted degrees ->
// stats[block][4]: max and min count, max and min weighted degree.
__device__ void block_degree_stats(double mx, double mn, double wmx, double wmn,
                                   double *stats) {
  __shared__ double sh[4][4];
  for (int off = 32; off >= 1; off >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, off));
    mn = fmin(mn, __shfl_xor(mn, off));
    wmx = fmax(wmx, __shfl_xor(wmx, off));
    wmn = fmin(wmn, __shfl_xor(wmn, off));
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sh[wave][0] = mx;
    sh[wave][1] = mn;
    sh[wave][2] = wmx;
    sh[wave][3] = wmn;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    const int q = threadIdx.x;
    double a = sh[0][q];
    for (int w = 1; w < 4; ++w) a = (q & 1) ? fmin(a, sh[w][q]) : fmax(a, sh[w][q]);
    stats[blockIdx.x * 4 + q] = a;
  }
}

// Degrees of weighted graphs.  The weighted degree is the exact sum of the
// row's weights rounded once to FP64 (128-bit fixed point, see fixed.h), so it
// does not depend on any summation order.  Four lanes per row, their sums
// added by the first; rows above kDegLong entries are listed and summed by the
// whole block with a tree in LDS.  The row loop is uniform over the block.
// One wavefront per row, with 64 lane sums added by one lane, left the memory
// idle: 27-point mesh of 512,000 rows, FP64 weights: 620 -> 41 us.
constexpr int kDegLanes = 4;
constexpr int kDegLong = 256;

template <typename IdxT, typename WT>
__global__ __launch_bounds__(256) void k_degrees(int64_t n, const IdxT *rp,
                                                 const WT *w, int e0, double *d64,
                                                 float *d32, double *stats) {
  constexpr int R = 256 / kDegLanes;
  __shared__ unsigned long long plo[256], phi[256];
  __shared__ int64_t longs[R];
  __shared__ int nlong;
  const int t = threadIdx.x, gl = t & (kDegLanes - 1);
  double mx = 0.0, mn = 1e300, wmx = 0.0, wmn = 1e300;
  auto put = [&](int64_t i, int64_t d, const U128 &tot) {
    const double s = fixed_to_double(tot, e0);
    d64[i] = s;
    if (d32) d32[i] = float(s);
    mx = fmax(mx, double(d));
    mn = fmin(mn, double(d));
    wmx = fmax(wmx, s);
    wmn = fmin(wmn, s);
  };
  auto sum = [&](int64_t b, int64_t e, int step) {
    U128 acc{0, 0};
#pragma unroll 4
    for (int64_t k = b; k < e; k += step) {
      unsigned long long lo, hi;
      fixed_of(w[k], e0, lo, hi);
      add128(acc, lo, hi);
    }
    return acc;
  };
  if (t == 0) nlong = 0;
  for (int64_t r0 = (int64_t)blockIdx.x * R; r0 < n; r0 += (int64_t)gridDim.x * R) {
    const int64_t i = r0 + t / kDegLanes;
    const int64_t b = i < n ? rp[i] : 0, e = i < n ? rp[i + 1] : 0;
    const bool small = e - b <= kDegLong;
    const U128 acc = small ? sum(b + gl, e, kDegLanes) : U128{0, 0};
    plo[t] = acc.lo;
    phi[t] = acc.hi;
    __syncthreads();
    if (gl == 0 && i < n) {
      if (small) {
        U128 tot = acc;
        for (int q = 1; q < kDegLanes; ++q) add128(tot, plo[t + q], phi[t + q]);
        put(i, e - b, tot);
      } else {
        longs[atomicAdd(&nlong, 1)] = i;
      }
    }
    __syncthreads();
    const int nl = nlong;
    for (int l = 0; l < nl; ++l) {
      const int64_t il = longs[l];
      const int64_t bl = rp[il], el = rp[il + 1];
      const U128 a = sum(bl + t, el, 256);
      plo[t] = a.lo;
      phi[t] = a.hi;
      __syncthreads();
      for (int h = 128; h >= 1; h >>= 1) {
        if (t < h) {
          U128 x{plo[t], phi[t]};
          add128(x, plo[t + h], phi[t + h]);
          plo[t] = x.lo;
          phi[t] = x.hi;
        }
        __syncthreads();
      }
      if (t == 0) put(il, el - bl, U128{plo[0], phi[0]});
      __syncthreads();
    }
    if (t == 0) nlong = 0;
    __syncthreads();
  }
  block_degree_stats(mx, mn, wmx, wmn, stats);
}

// Unit weights: the degree is the row length; one thread per row.  d64 and
// d32 may be null (statistics only).
template <typename IdxT>
__global__ __launch_bounds__(256) void k_degrees_unit(int64_t n, const IdxT *rp, double *d64,
                                                      float *d32, double *stats) {
  double mx = 0.0, mn = 1e300;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double s = double(rp[i + 1] - rp[i]);
    if (d64) d64[i] = s;
    if (d32) d32[i] = float(s);
    mx = fmax(mx, s);
    mn = fmin(mn, s);
  }
  block_degree_stats(mx, mn, mx, mn, stats);
}

// edge-weight range (for the exact cut), block partials
template <typename WT>
__global__ __launch_bounds__(256) void k_wrange(int64_t nnz, const WT *w, double *stats) {
  double mx = 0.0, mn = 1e300;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz;
       k += (int64_t)gridDim.x * blockDim.x) {
    double v = double(w[k]);
    mx = fmax(mx, v);
    mn = fmin(mn, v);
  }
  __shared__ double s0[4], s1[4];
  for (int off = 32; off >= 1; off >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, off));
    mn = fmin(mn, __shfl_xor(mn, off));
  }
  if ((threadIdx.x & 63) == 0) {
    s0[threadIdx.x >> 6] = mx;
    s1[threadIdx.x >> 6] = mn;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    stats[blockIdx.x * 2] = fmax(fmax(s0[0], s0[1]), fmax(s0[2], s0[3]));
    stats[blockIdx.x * 2 + 1] = fmin(fmin(s1[0], s1[1]), fmin(s1[2], s1[3]));
  }
}

// Deterministic row binning into kNumBins + 1 classes (the last = hubs).
constexpr int kBinRows = 1024;   // rows per block
constexpr int kNumCls = kNumBins + 1;

template <typename IdxT>
__device__ __forceinline__ int row_class(const IdxT *rp, int64_t i) {
  const int64_t d = rp[i + 1] - rp[i];
  int c = 0;
  while (c < kNumBins && d > bin_max_deg(c)) ++c;
  return c;
}

template <typename IdxT>
__global__ __launch_bounds__(256) void k_bin_count(int64_t n, const IdxT *rp, int *counts) {
  __shared__ int c[kNumCls];
  if (threadIdx.x < kNumCls) c[threadIdx.x] = 0;
  __syncthreads();
  int64_t r0 = (int64_t)blockIdx.x * kBinRows;
  for (int t = threadIdx.x; t < kBinRows; t += blockDim.x) {
    int64_t i = r0 + t;
    if (i < n) atomicAdd(&c[row_class(rp, i)], 1);
  }
  __syncthreads();
  if (threadIdx.x < kNumCls) counts[blockIdx.x * kNumCls + threadIdx.x] = c[threadIdx.x];
}

// Exclusive scan of the per-block counts into positions of one packed list
// (class 0 rows first, then class 1, ...); totals[c] = rows of class c.  One
// block: thread t adds the counts of a run of blocks per class, a scan over
// the threads in LDS, then each thread writes its run's positions.
__global__ __launch_bounds__(1024) void k_bin_scan(int nblocks, int *counts, int *totals) {
  __shared__ int sh[kNumCls][1024];
  const int t = threadIdx.x;
  const int per = (nblocks + 1023) / 1024;
  const int b0 = min(nblocks, t * per), b1 = min(nblocks, b0 + per);
  int own[kNumCls] = {};
  for (int b = b0; b < b1; ++b)
    for (int c = 0; c < kNumCls; ++c) own[c] += counts[b * kNumCls + c];
  for (int c = 0; c < kNumCls; ++c) sh[c][t] = own[c];
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    int x[kNumCls];
    for (int c = 0; c < kNumCls; ++c) x[c] = t >= off ? sh[c][t - off] : 0;
    __syncthreads();
    for (int c = 0; c < kNumCls; ++c) sh[c][t] += x[c];
    __syncthreads();
  }
  int base = 0;
  for (int c = 0; c < kNumCls; ++c) {
    const int tot = sh[c][1023];
    if (t == 0) totals[c] = tot;
    int acc = base + sh[c][t] - own[c];
    for (int b = b0; b < b1; ++b) {
      const int v = counts[b * kNumCls + c];
      counts[b * kNumCls + c] = acc;
      acc += v;
    }
    base += tot;
  }
}

// Chunk table of the hub rows (one block): begin[h] is hub h's first chunk
// (begin[nh] the number of chunks), k0 and row a chunk's first entry and its row.
template <typename IdxT>
__global__ __launch_bounds__(1024) void k_hub_table(const IdxT *rp, const int32_t *hubs, int nh,
                                                    int32_t *begin, int64_t *k0, int32_t *row) {
  __shared__ int sh[1024];
  const int t = threadIdx.x;
  int base = 0;
  for (int h0 = 0; h0 < nh; h0 += 1024) {
    const int h = h0 + t;
    int64_t b = 0, e = 0;
    if (h < nh) {
      b = rp[hubs[h]];
      e = rp[hubs[h] + 1];
    }
    const int cnt = (int)((e - b + kHubChunk - 1) / kHubChunk);
    sh[t] = cnt;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const int x = t >= off ? sh[t - off] : 0;
      __syncthreads();
      sh[t] += x;
      __syncthreads();
    }
    const int at = base + sh[t] - cnt;
    if (h < nh) {
      begin[h] = at;
      for (int q = 0; q < cnt; ++q) {
        k0[at + q] = b + (int64_t)q * kHubChunk;
        row[at + q] = hubs[h];
      }
    }
    base += sh[1023];
    __syncthreads();
  }
  if (t == 0) begin[nh] = base;
}

template <typename IdxT>
__global__ __launch_bounds__(256) void k_bin_scatter(int64_t n, const IdxT *rp,
                                                     const int *offsets, int32_t *packed) {
  // each thread owns kBinRows/256 consecutive rows; ranks via a block scan
  __shared__ int cnt[kNumCls][256];
  const int per = kBinRows / 256;
  int64_t r0 = (int64_t)blockIdx.x * kBinRows + (int64_t)threadIdx.x * per;
  int local[kNumCls] = {};
  for (int t = 0; t < per; ++t) {
    int64_t i = r0 + t;
    if (i < n) local[row_class(rp, i)]++;
  }
  for (int c = 0; c < kNumCls; ++c) cnt[c][threadIdx.x] = local[c];
  __syncthreads();
  if (threadIdx.x < kNumCls) {
    int c = threadIdx.x, acc = 0;
    for (int t = 0; t < 256; ++t) {
      int v = cnt[c][t];
      cnt[c][t] = acc;
      acc += v;
    }
  }
  __syncthreads();
  int pos[kNumCls];
  for (int c = 0; c < kNumCls; ++c) pos[c] = offsets[blockIdx.x * kNumCls + c] + cnt[c][threadIdx.x];
  for (int t = 0; t < per; ++t) {
    int64_t i = r0 + t;
    if (i < n) {
      int c = row_class(rp, i);
      packed[pos[c]++] = (int32_t)i;
    }
  }
}

template <typename F>
void with_types(sphx_graph *g, F &&f) {
  if (g->rp64) {
    if (g->wdt == SPHX_UNIT) f(int64_t{}, Unit{});
    else if (g->wdt == SPHX_F32) f(int64_t{}, float{});
    else f(int64_t{}, double{});
  } else {
    if (g->wdt == SPHX_UNIT) f(int32_t{}, Unit{});
    else if (g->wdt == SPHX_F32) f(int32_t{}, float{});
    else f(int32_t{}, double{});
  }
}

}  // namespace

int validate_graph(sphx_graph *g, hipStream_t s, int32_t *flags_dev, int *flags_host) {
  SPHX_HIP(g->h, hipMemsetAsync(flags_dev, 0, sizeof(int), s));
  unsigned gb = grid_for(g->n, 4, 1 << 16);
  with_types(g, [&](auto it, auto wt) {
    using IdxT = decltype(it);
    using WT = decltype(wt);
    hipLaunchKernelGGL((k_validate<IdxT, WT>), dim3(gb), dim3(256), 0, s, g->n, g->nnz,
                       (const IdxT *)g->rowptr, g->col, (const WT *)g->w, g->vwgt,
                       (int *)flags_dev);
  });
  SPHX_HIP(g->h, hipGetLastError());
  SPHX_HIP(g->h, hipMemcpyAsync(flags_host, flags_dev, sizeof(int), hipMemcpyDeviceToHost, s));
  SPHX_HIP(g->h, hipStreamSynchronize(s));
  int f = *flags_host;
  if (f & F_BAD_GRAPH) return set_err(g->h, SPHX_E_BAD_GRAPH,
      "CSR arrays malformed: row_ptr not monotone / not [0..nnz], column out of range, "
      "or columns not strictly increasing within a row");
  if (f & F_SELF_LOOP) return set_err(g->h, SPHX_E_SELF_LOOP, "graph has a self-loop");
  if (f & F_BAD_WEIGHT) return set_err(g->h, SPHX_E_BAD_WEIGHT,
      "edge weight not finite and > 0, or vertex weight < 1");
  if (f & F_NOT_SYM) return set_err(g->h, SPHX_E_NOT_SYMMETRIC,
      "pattern or weights not symmetric");
  return SPHX_OK;
}

constexpr int kDegBlocks = 1024;

int weight_range(sphx_graph *g, void *scratch, void *pinned, hipStream_t s) {
  if (g->wdt == SPHX_UNIT || known(g->wrange_valid)) return SPHX_OK;
  double *stats = static_cast<double *>(scratch);
  double *host = static_cast<double *>(pinned);
  const unsigned gw = grid_for(g->nnz, 256, kWrangeBlocks);
  if (g->wdt == SPHX_F32)
    hipLaunchKernelGGL((k_wrange<float>), dim3(gw), dim3(256), 0, s, g->nnz,
                       (const float *)g->w, stats);
  else
    hipLaunchKernelGGL((k_wrange<double>), dim3(gw), dim3(256), 0, s, g->nnz,
                       (const double *)g->w, stats);
  SPHX_HIP(g->h, hipGetLastError());
  SPHX_HIP(g->h, hipMemcpyAsync(host, stats, sizeof(double) * 2 * gw,
                                hipMemcpyDeviceToHost, s));
  SPHX_HIP(g->h, hipStreamSynchronize(s));
  double a = 0, b = 1e300;
  for (unsigned q = 0; q < gw; ++q) {
    a = std::max(a, host[q * 2]);
    b = std::min(b, host[q * 2 + 1]);
  }
  int ea, eb;
  std::frexp(a, &ea);
  std::frexp(b, &eb);
  if (g->nnz > 0 && ea - eb > 40)
    return set_err(g->h, SPHX_E_BAD_WEIGHT,
                   "edge weights span more than a factor 2^40 (exact sums unsupported)");
  g->wmax = a;
  g->wmin = b;
  publish(g->wrange_valid);
  return SPHX_OK;
}

int compute_degrees(sphx_graph *g, double *d64, float *d32, void *scratch,
                    DegreeStats *out, void *pinned, hipStream_t s) {
  double *stats = static_cast<double *>(scratch);
  double *host = static_cast<double *>(pinned);
  // edge-weight range: e0 of the exact degree sums and of the exact cut
  SPHX_TRY(weight_range(g, scratch, pinned, s));
  int e0 = 0;
  if (g->wdt == SPHX_F32) e0 = fixed_exponent<float>(g->wmin);
  if (g->wdt == SPHX_F64) e0 = fixed_exponent<double>(g->wmin);
  unsigned gb = grid_for(g->n, 256 / kDegLanes, kDegBlocks);
  if (g->wdt == SPHX_UNIT) {
    gb = grid_for(g->n, 256, kDegBlocks);
    if (g->rp64)
      hipLaunchKernelGGL((k_degrees_unit<int64_t>), dim3(gb), dim3(256), 0, s, g->n,
                         (const int64_t *)g->rowptr, d64, d32, stats);
    else
      hipLaunchKernelGGL((k_degrees_unit<int32_t>), dim3(gb), dim3(256), 0, s, g->n,
                         (const int32_t *)g->rowptr, d64, d32, stats);
  } else {
    with_types(g, [&](auto it, auto wt) {
      using IdxT = decltype(it);
      using WT = decltype(wt);
      if constexpr (!std::is_same_v<WT, Unit>)
        hipLaunchKernelGGL((k_degrees<IdxT, WT>), dim3(gb), dim3(256), 0, s, g->n,
                           (const IdxT *)g->rowptr, (const WT *)g->w, e0, d64, d32, stats);
    });
  }
  SPHX_HIP(g->h, hipGetLastError());
  SPHX_HIP(g->h, hipMemcpyAsync(host, stats, sizeof(double) * 4 * gb,
                                hipMemcpyDeviceToHost, s));
  SPHX_HIP(g->h, hipStreamSynchronize(s));
  double mx = 0, mn = 1e300, wmx = 0, wmn = 1e300;
  for (unsigned b = 0; b < gb; ++b) {
    mx = std::max(mx, host[b * 4 + 0]);
    mn = std::min(mn, host[b * 4 + 1]);
    wmx = std::max(wmx, host[b * 4 + 2]);
    wmn = std::min(wmn, host[b * 4 + 3]);
  }
  out->max_deg = (int64_t)mx;
  out->min_deg = (int64_t)mn;
  out->sum_deg = g->nnz;
  out->max_wdeg = wmx;
  out->min_wdeg = wmn;
  if (!known(g->stats_valid)) {
    g->max_deg = out->max_deg;
    g->min_deg = out->min_deg;
    g->sum_deg = out->sum_deg;
    publish(g->stats_valid);
  }
  return SPHX_OK;
}

int pattern_stats(sphx_graph *g, void *scratch, DegreeStats *out, void *pinned, hipStream_t s) {
  SPHX_TRY(weight_range(g, scratch, pinned, s));
  if (!known(g->stats_valid)) {
    sphx_graph u = *g;        // the same pattern with unit weights
    u.wdt = SPHX_UNIT;
    u.stats_valid = 0;
    SPHX_TRY(compute_degrees(&u, nullptr, nullptr, scratch, out, pinned, s));
    g->max_deg = u.max_deg;
    g->min_deg = u.min_deg;
    g->sum_deg = u.sum_deg;
    publish(g->stats_valid);
  }
  out->max_deg = g->max_deg;
  out->min_deg = g->min_deg;
  out->sum_deg = g->sum_deg;
  out->max_wdeg = double(g->max_deg);
  out->min_wdeg = double(g->min_deg);
  return SPHX_OK;
}

namespace {

// Column offsets from the row as int16; *overflow is set when some offset does
// not fit (the offsets are then not used).  A block takes 256 rows: each
// thread notes its row at its entries in LDS, then the block goes over the
// run of entries with coalesced loads and stores (one thread per row
// throughout: 33 instead of 25 us on a 2 M-row 7-point grid).
__global__ __launch_bounds__(256) void k_delta16(int64_t n, const int32_t *__restrict__ rp,
                                                 const int32_t *__restrict__ col, int16_t *d,
                                                 int *overflow) {
  __shared__ uint8_t own[256 * kUnbinnedMaxDeg];
  int f = 0;
  for (int64_t r0 = (int64_t)blockIdx.x * 256; r0 < n; r0 += (int64_t)gridDim.x * 256) {
    const int64_t i = r0 + threadIdx.x, r1 = min(n, r0 + 256);
    const int64_t k0 = rp[r0], k1 = rp[r1];
    if (i < n) {
      const int b = (int)(rp[i] - k0), e = (int)(rp[i + 1] - k0);
      for (int k = b; k < e; ++k) own[k] = (uint8_t)threadIdx.x;
    }
    __syncthreads();
    for (int64_t k = k0 + threadIdx.x; k < k1; k += 256) {
      const int64_t o = (int64_t)col[k] - (r0 + own[k - k0]);
      const bool fits = o >= -32767 && o <= 32767;
      d[k] = (int16_t)(fits ? o : 0);
      f |= fits ? 0 : 1;
    }
    __syncthreads();
  }
  if (f) atomicOr(overflow, 1);
}

__global__ void k_fill_int(int *x, int cnt, int v) {
  for (int i = threadIdx.x; i < cnt; i += blockDim.x) x[i] = v;
}

}  // namespace

namespace {

// ---- degree order: rows by floor(log2 degree), descending, ties in
// increasing id (a stable bucket sort), so that the frequently gathered rows
// of high degree share cache lines
constexpr int kOrdCls = 32;
constexpr int kOrdRows = 1024;   // rows per counting block

template <typename IdxT>
__device__ __forceinline__ int ord_class(const IdxT *rp, int64_t i) {
  const int64_t d = (int64_t)rp[i + 1] - (int64_t)rp[i];
  int lg = 0;
  for (int64_t x = d; x > 1; x >>= 1) ++lg;
  return kOrdCls - 1 - min(lg, kOrdCls - 1);
}

template <typename IdxT>
__global__ __launch_bounds__(256) void k_ord_count(int64_t n, const IdxT *rp, int *counts) {
  __shared__ int c[kOrdCls];
  if (threadIdx.x < kOrdCls) c[threadIdx.x] = 0;
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * kOrdRows;
  for (int t = threadIdx.x; t < kOrdRows; t += blockDim.x) {
    const int64_t i = r0 + t;
    if (i < n) atomicAdd(&c[ord_class(rp, i)], 1);
  }
  __syncthreads();
  if (threadIdx.x < kOrdCls) counts[blockIdx.x * kOrdCls + threadIdx.x] = c[threadIdx.x];
}

// counts[b][c] -> start of block b's class-c rows in the new order (class 0
// first): one thread per class scans the blocks, then thread 0 adds the
// class offsets
__global__ __launch_bounds__(64) void k_ord_scan(int nblocks, int *counts) {
  __shared__ long long tot[kOrdCls];
  const int c = threadIdx.x;
  if (c < kOrdCls) {
    long long acc = 0;
    for (int b = 0; b < nblocks; ++b) {
      const int v = counts[b * kOrdCls + c];
      counts[b * kOrdCls + c] = (int)acc;
      acc += v;
    }
    tot[c] = acc;
  }
  __syncthreads();
  if (c < kOrdCls) {
    long long base = 0;
    for (int q = 0; q < c; ++q) base += tot[q];
    for (int b = 0; b < nblocks; ++b) counts[b * kOrdCls + c] += (int)base;
  }
}

// perm[new] = old
template <typename IdxT>
__global__ __launch_bounds__(256) void k_ord_scatter(int64_t n, const IdxT *rp,
                                                     const int *offsets, int32_t *perm) {
  __shared__ int cnt[kOrdCls][256];
  const int per = kOrdRows / 256;
  const int64_t r0 = (int64_t)blockIdx.x * kOrdRows + (int64_t)threadIdx.x * per;
  int local[kOrdCls];
  for (int c = 0; c < kOrdCls; ++c) local[c] = 0;
  for (int t = 0; t < per; ++t) {
    const int64_t i = r0 + t;
    if (i < n) local[ord_class(rp, i)]++;
  }
  for (int c = 0; c < kOrdCls; ++c) cnt[c][threadIdx.x] = local[c];
  __syncthreads();
  if (threadIdx.x < kOrdCls) {
    const int c = threadIdx.x;
    int acc = 0;
    for (int t = 0; t < 256; ++t) {
      const int v = cnt[c][t];
      cnt[c][t] = acc;
      acc += v;
    }
  }
  __syncthreads();
  int pos[kOrdCls];
  for (int c = 0; c < kOrdCls; ++c)
    pos[c] = offsets[blockIdx.x * kOrdCls + c] + cnt[c][threadIdx.x];
  for (int t = 0; t < per; ++t) {
    const int64_t i = r0 + t;
    if (i < n) perm[pos[ord_class(rp, i)]++] = (int32_t)i;
  }
}

template <typename IdxT>
__global__ __launch_bounds__(256) void k_ord_degrees(int64_t n, const IdxT *rp,
                                                     const int32_t *perm, int32_t *inv,
                                                     long long *deg_new) {
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n;
       p += (int64_t)gridDim.x * 256) {
    const int64_t o = perm[p];
    inv[o] = (int32_t)p;
    deg_new[p] = (long long)rp[o + 1] - (long long)rp[o];
  }
}

// exclusive scan of deg_new into the new row pointers: block sums, a scan of
// the block sums (one block), then each block's local scan plus its offset
constexpr int kScanRows = 1024;

__global__ __launch_bounds__(256) void k_scan_sums(int64_t n, const long long *x,
                                                   long long *bsum) {
  __shared__ long long sh[4];
  const int64_t r0 = (int64_t)blockIdx.x * kScanRows;
  long long acc = 0;
  for (int t = threadIdx.x; t < kScanRows; t += 256) {
    const int64_t i = r0 + t;
    if (i < n) acc += x[i];
  }
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

__global__ __launch_bounds__(64) void k_scan_bsums(int nb, long long *bsum) {
  if (threadIdx.x == 0) {
    long long acc = 0;
    for (int b = 0; b < nb; ++b) {
      const long long v = bsum[b];
      bsum[b] = acc;
      acc += v;
    }
  }
}

template <typename IdxT>
__global__ __launch_bounds__(256) void k_scan_rows(int64_t n, const long long *x,
                                                   const long long *bsum, IdxT *out) {
  __shared__ long long sh[kScanRows];
  const int64_t r0 = (int64_t)blockIdx.x * kScanRows;
  for (int t = threadIdx.x; t < kScanRows; t += 256) {
    const int64_t i = r0 + t;
    sh[t] = i < n ? x[i] : 0;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    long long acc = bsum[blockIdx.x];
    for (int t = 0; t < kScanRows; ++t) {
      const long long v = sh[t];
      sh[t] = acc;
      acc += v;
    }
    if (r0 + kScanRows >= n) out[n] = (IdxT)acc;   // the last block writes the total
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kScanRows; t += 256) {
    const int64_t i = r0 + t;
    if (i < n) out[i] = (IdxT)sh[t];
  }
}

// new row p = old row perm[p], columns renamed by inv: one wavefront per row
template <typename IdxT, typename WT>
__global__ __launch_bounds__(256) void k_ord_rows(int64_t n, const IdxT *rp, const int32_t *col,
                                                  const WT *w, const int32_t *perm,
                                                  const int32_t *inv, const IdxT *rp_new,
                                                  int32_t *col_new, WT *w_new) {
  const int lane = threadIdx.x & 63;
  for (int64_t p = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6; p < n;
       p += ((int64_t)gridDim.x * 256) >> 6) {
    const int64_t o = perm[p];
    const int64_t k0 = rp[o], d = (int64_t)rp[o + 1] - k0, q0 = rp_new[p];
    for (int64_t k = lane; k < d; k += 64) {
      col_new[q0 + k] = inv[col[k0 + k]];
      if constexpr (!std::is_same_v<WT, Unit>) w_new[q0 + k] = w[k0 + k];
    }
  }
}

}  // namespace

size_t degree_order_bytes(const sphx_graph *g) {
  const int64_t n = g->n;
  const int64_t nb = ceil_div(n, kOrdRows);
  const size_t ib = g->rp64 ? 8 : 4;
  const size_t wb = g->wdt == SPHX_F64 ? 8 : (g->wdt == SPHX_F32 ? 4 : 0);
  size_t b = 0;
  b += align_up(sizeof(int32_t) * n, 256) * 2;                 // perm, inv
  b += align_up(ib * (n + 1), 256);                            // row pointers
  b += align_up(sizeof(int32_t) * g->nnz, 256);                // columns
  b += align_up(wb * g->nnz, 256);                             // weights
  b += align_up(sizeof(long long) * n, 256);                   // new degrees
  b += align_up(sizeof(int) * nb * kOrdCls, 256);              // class counts
  b += align_up(sizeof(long long) * ceil_div(n, kScanRows), 256);
  return b + 1024;
}

int build_degree_order(sphx_graph *g, void *scratch, sphx_graph *out, int32_t **perm_out,
                       int32_t **inv_out, hipStream_t s) {
  const int64_t n = g->n;
  const int64_t nb = ceil_div(n, kOrdRows);
  const size_t wb = g->wdt == SPHX_F64 ? 8 : (g->wdt == SPHX_F32 ? 4 : 0);
  Arena a;
  a.base = static_cast<char *>(scratch);
  int32_t *perm = a.take<int32_t>(n);
  int32_t *inv = a.take<int32_t>(n);
  char *rpn = a.take<char>((g->rp64 ? 8 : 4) * (n + 1));
  int32_t *coln = a.take<int32_t>(g->nnz);
  char *wn = a.take<char>(wb * g->nnz);
  long long *degn = a.take<long long>(n);
  int *counts = a.take<int>(nb * kOrdCls);
  long long *bsum = a.take<long long>(ceil_div(n, kScanRows));
  const unsigned gs = (unsigned)ceil_div(n, kScanRows);
  auto go = [&](auto idx_tag, auto w_tag) {
    using IdxT = decltype(idx_tag);
    using WT = decltype(w_tag);
    const IdxT *rp = static_cast<const IdxT *>(g->rowptr);
    hipLaunchKernelGGL((k_ord_count<IdxT>), dim3((unsigned)nb), dim3(256), 0, s, n, rp, counts);
    hipLaunchKernelGGL(k_ord_scan, dim3(1), dim3(64), 0, s, (int)nb, counts);
    hipLaunchKernelGGL((k_ord_scatter<IdxT>), dim3((unsigned)nb), dim3(256), 0, s, n, rp,
                       (const int *)counts, perm);
    hipLaunchKernelGGL((k_ord_degrees<IdxT>), dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, n,
                       rp, (const int32_t *)perm, inv, degn);
    hipLaunchKernelGGL(k_scan_sums, dim3(gs), dim3(256), 0, s, n, (const long long *)degn, bsum);
    hipLaunchKernelGGL(k_scan_bsums, dim3(1), dim3(64), 0, s, (int)gs, bsum);
    hipLaunchKernelGGL((k_scan_rows<IdxT>), dim3(gs), dim3(256), 0, s, n,
                       (const long long *)degn, (const long long *)bsum, (IdxT *)rpn);
    hipLaunchKernelGGL((k_ord_rows<IdxT, WT>), dim3(grid_for(n, 4, 8192)), dim3(256), 0, s, n,
                       rp, g->col, static_cast<const WT *>(g->w), (const int32_t *)perm,
                       (const int32_t *)inv, (const IdxT *)rpn, coln, (WT *)wn);
  };
  with_types(g, go);
  SPHX_HIP(g->h, hipGetLastError());
  *out = *g;
  out->rowptr = rpn;
  out->col = coln;
  out->w = wb ? wn : nullptr;
  out->vwgt = nullptr;
  out->stats_valid = 0;
  out->offsets16 = 0;
  *perm_out = perm;
  *inv_out = inv;
  return SPHX_OK;
}

// the int16 column offsets are kept for unit-weight graphs with 32-bit row
// pointers that are (or may be, before their degrees are known) unbinned
static bool may_compress(const sphx_graph *g) {
  return g->wdt == SPHX_UNIT && !g->rp64 && (!known(g->stats_valid) || g->max_deg <= kUnbinnedMaxDeg);
}

size_t plan_bytes(sphx_graph *g) {
  int64_t n = g->n;
  int64_t nb = ceil_div(n, kBinRows);
  int64_t max_hub = g->nnz / kHubDeg + 1;
  int64_t max_chunks = g->nnz / kHubChunk + max_hub + 1;
  size_t b = 0;
  b += align_up(sizeof(int32_t) * n, 256);              // packed class lists
  b += align_up(sizeof(int32_t) * (max_hub + 1), 256);  // hub chunk begin
  b += align_up(sizeof(int64_t) * max_chunks, 256) +    // chunks: first entries
       align_up(sizeof(int32_t) * max_chunks, 256);     // and rows
  b += align_up(sizeof(double) * max_chunks * kMaxNev, 256);
  b += align_up(sizeof(int) * (nb * kNumCls + kNumCls), 256);
  if (may_compress(g)) b += align_up(sizeof(int16_t) * g->nnz, 256) + 256;
  return b + 4096;
}

int build_plan(sphx_graph *g, Arena &ws, SpmmPlan *plan, const DegreeStats &st,
               void *pinned, hipStream_t s, bool offsets) {
  *plan = SpmmPlan{};
  int64_t n = g->n;
  int64_t nb = ceil_div(n, kBinRows);
  int64_t max_hub = g->nnz / kHubDeg + 1;
  int64_t max_chunks = g->nnz / kHubChunk + max_hub + 1;
  int32_t *packed = ws.take<int32_t>(n);
  int32_t *hcb = ws.take<int32_t>(max_hub + 1);
  int64_t *k0 = ws.take<int64_t>(max_chunks);
  int32_t *krow = ws.take<int32_t>(max_chunks);
  double *hp = ws.take<double>(max_chunks * kMaxNev);
  int *counts = ws.take<int>(nb * kNumCls + kNumCls);
  if (st.max_deg <= kUnbinnedMaxDeg) {   // natural order, one group size
    plan->group = st.max_deg <= bin_max_deg(0) ? bin_group(0) : bin_group(1);
    int fits = known(g->offsets16);
    if (offsets && may_compress(g) && g->nnz > 0 && fits != 2) {
      int16_t *d = ws.take<int16_t>(g->nnz);
      int *flag = ws.take<int>(4);
      hipLaunchKernelGGL(k_fill_int, dim3(1), dim3(64), 0, s, flag, 4, 0);
      hipLaunchKernelGGL(k_delta16, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, n,
                         (const int32_t *)g->rowptr, g->col, d, flag);
      SPHX_HIP(g->h, hipGetLastError());
      if (fits == 0) {           // whether the pattern's offsets fit is known after this
        int *hf = static_cast<int *>(pinned);
        SPHX_HIP(g->h, hipMemcpyAsync(hf, flag, sizeof(int), hipMemcpyDeviceToHost, s));
        SPHX_HIP(g->h, hipStreamSynchronize(s));
        fits = hf[0] == 0 ? 1 : 2;
        publish(g->offsets16, fits);
      }
      if (fits == 1) plan->dcol = d;
    }
    return SPHX_OK;
  }
  plan->binned = true;
  int *totals = counts + nb * kNumCls;
  if (g->rp64) {
    hipLaunchKernelGGL((k_bin_count<int64_t>), dim3(nb), dim3(256), 0, s, n,
                       (const int64_t *)g->rowptr, counts);
    hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, s, (int)nb, counts, totals);
    hipLaunchKernelGGL((k_bin_scatter<int64_t>), dim3(nb), dim3(256), 0, s, n,
                       (const int64_t *)g->rowptr, counts, packed);
  } else {
    hipLaunchKernelGGL((k_bin_count<int32_t>), dim3(nb), dim3(256), 0, s, n,
                       (const int32_t *)g->rowptr, counts);
    hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, s, (int)nb, counts, totals);
    hipLaunchKernelGGL((k_bin_scatter<int32_t>), dim3(nb), dim3(256), 0, s, n,
                       (const int32_t *)g->rowptr, counts, packed);
  }
  SPHX_HIP(g->h, hipGetLastError());
  int *th = static_cast<int *>(pinned);
  SPHX_HIP(g->h, hipMemcpyAsync(th, totals, sizeof(int) * kNumCls, hipMemcpyDeviceToHost, s));
  SPHX_HIP(g->h, hipStreamSynchronize(s));
  int64_t base = 0;
  for (int c = 0; c < kNumBins; ++c) {
    plan->rows[c] = packed + base;
    plan->nrows[c] = th[c];
    base += th[c];
  }
  const int32_t *l2 = packed + base;
  plan->hub_rows = l2;
  plan->n_hub = th[kNumBins];
  plan->hub_chunk_begin = hcb;
  plan->chunk_k0 = k0;
  plan->chunk_row = krow;
  plan->hub_partial = hp;
  if (plan->n_hub > 0) {
    plan->n_chunks = max_chunks;
    if (g->rp64)
      hipLaunchKernelGGL((k_hub_table<int64_t>), dim3(1), dim3(1024), 0, s,
                         (const int64_t *)g->rowptr, l2, (int)plan->n_hub, hcb, k0, krow);
    else
      hipLaunchKernelGGL((k_hub_table<int32_t>), dim3(1), dim3(1024), 0, s,
                         (const int32_t *)g->rowptr, l2, (int)plan->n_hub, hcb, k0, krow);
    SPHX_HIP(g->h, hipGetLastError());
  }
  return SPHX_OK;
}

}  // namespace sphx
