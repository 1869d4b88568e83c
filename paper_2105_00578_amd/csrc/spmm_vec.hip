// Laplacian block product Y = L_C X over row-major blocks of at least two
// columns (Eq. 2 with weights, difference form y_i = sum_j w_ij (x_i - x_j)).
//
// A row of ld values is read as NV vectors of E values: vector v starts at
// value v E, the last one at ld - E, so that a width that is no multiple of E
// makes the last two overlap (the shared values are computed twice, to the
// same bits) and nothing outside the row is touched.  Vectors are only aligned
// to their elements.  The caller's blocks have exactly their columns; so have
// the solver's (block_ld) and the polynomials' (compact_ld) where every row has
// at most 12 neighbours (but for 5 and 6 FP32 columns of the solver's, which
// are padded), elsewhere the solver's rows are whole 16-byte vectors and the
// polynomials' an even number of values; the adjoint's are always padded.
// Short rows are handled one thread per row: the thread keeps x_i and the
// NV-vector accumulator in registers and gathers each neighbour row with NV
// vector loads (adjacent threads take adjacent rows, so on mesh-like graphs the
// gathers of a wavefront are contiguous).  Blocks of rows are mapped so that
// each of the 8 XCDs (hardware places consecutive workgroups round robin on
// them) works on one contiguous eighth of the rows, which keeps the gathered
// neighbours of a mesh in that XCD's L2.  Longer rows of power-law graphs use
// groups of 4, 16 or 64 lanes (lanes over the neighbours, butterfly reduction
// in a fixed order), hub rows fixed-size chunks combined in a second pass.  All
// sums are in a fixed order, so results are bitwise reproducible.
//
// Epilogues (whole rows): Store, Residual (r = acc - b_i theta_c x_i, output r
// or the Jacobi step r / d_i, FP64 norm partials of ||r||^2_{B^-1} and
// ||x||^2_B per column c < m), and one Chebyshev step of the iteration for
// L h = r (Sec. 5.2).
#include <hip/hip_ext.h>

#include <algorithm>

#include "kernels.h"

namespace sphx {
namespace {

// Row vectors of VB bytes: 16 (float4 / double2), or 8 (float2) for the FP32
// widths that with_vectors names.
template <typename T, int VB> struct Vec;
template <> struct Vec<float, 16> {
  typedef float type __attribute__((ext_vector_type(4)));
  typedef type mem __attribute__((aligned(4)));
  static constexpr int E = 4;
};
template <> struct Vec<float, 8> {
  typedef float type __attribute__((ext_vector_type(2)));
  typedef type mem __attribute__((aligned(4)));
  static constexpr int E = 2;
};
template <> struct Vec<double, 16> {
  typedef double type __attribute__((ext_vector_type(2)));
  typedef type mem __attribute__((aligned(8)));
  static constexpr int E = 2;
};

// The row of ld values at p, and its store; `last` = ld - E.
template <typename T, int VB, int NV>
__device__ __forceinline__ void load_row(const T *__restrict__ p, int last,
                                         typename Vec<T, VB>::type (&x)[NV]) {
  using M = typename Vec<T, VB>::mem;
  constexpr int E = Vec<T, VB>::E;
#pragma unroll
  for (int v = 0; v < NV - 1; ++v) x[v] = *reinterpret_cast<const M *>(p + v * E);
  x[NV - 1] = *reinterpret_cast<const M *>(p + last);
}
template <typename T, int VB, int NV>
__device__ __forceinline__ void store_row(T *p, int last,
                                          const typename Vec<T, VB>::type (&x)[NV]) {
  using M = typename Vec<T, VB>::mem;
  constexpr int E = Vec<T, VB>::E;
#pragma unroll
  for (int v = 0; v < NV - 1; ++v) *reinterpret_cast<M *>(p + v * E) = x[v];
  *reinterpret_cast<M *>(p + last) = x[NV - 1];
}

// Unit weights with the column indices stored as int16 offsets from the row
// (graphs whose every neighbour lies within 32767 rows: two bytes per entry
// instead of four in the index stream).
struct UnitD16 {};
template <typename WT>
constexpr bool kUnitW = std::is_same_v<WT, Unit> || std::is_same_v<WT, UnitD16>;
template <typename WT> struct ColOf { using type = int32_t; };
template <> struct ColOf<UnitD16> { using type = int16_t; };

template <typename IdxT, typename WT>
struct Csr {
  const IdxT *rp;
  const typename ColOf<WT>::type *col;
  const WT *w;
  // neighbour of row i stored at entry k, and the entry's weight
  __device__ __forceinline__ int64_t nbr(int64_t i, int64_t k) const {
    if constexpr (std::is_same_v<WT, UnitD16>) return i + (int64_t)col[k];
    else return (int64_t)col[k];
  }
  __device__ __forceinline__ WT wk(int64_t k) const { return w[k]; }
};

// The same entries read from an LDS copy of a contiguous run of them
// (entries k0 ..; staged by the row-chunk kernel below).
template <typename WT>
struct LdsCsr {
  using CT = typename ColOf<WT>::type;
  using WS = std::conditional_t<kUnitW<WT>, float, WT>;
  const CT *col;
  const WS *w;
  int64_t k0;
  __device__ __forceinline__ int64_t nbr(int64_t i, int64_t k) const {
    if constexpr (std::is_same_v<WT, UnitD16>) return i + (int64_t)col[k - k0];
    else return (int64_t)col[k - k0];
  }
  __device__ __forceinline__ WS wk(int64_t k) const { return w[k - k0]; }
};

// Block id remap: XCD x = b % 8 receives a contiguous range of block ids.
__device__ __forceinline__ int64_t xcd_remap(int64_t b, int64_t nb) {
  const int64_t q = nb / 8, r = nb % 8;
  const int64_t x = b % 8, pos = b / 8;
  return x * q + (x < r ? x : r) + pos;
}

// acc = sum over entries k0, k0 + step, ... < k1 of w_k (x_i - x_col[k]).
// U independent partial sums (U gathers in flight per lane), combined in a
// fixed order.
// kWhole: the vectors of a neighbour row are loaded one behind the other.  Left
// to itself the compiler loads the first vectors of all U rows and then the last
// ones, whose address it forms later; where the neighbours of 64 lanes are
// anywhere (binned plans), U x 64 lines of 128 bytes are the whole of a compute
// unit's L1, and the last vectors are fetched from L2 again: store product of 5
// FP32 columns on R-MAT 22 1347 us, with whole rows 1094; R-MAT 17 37.4 and 30.4.
// On meshes the lines stay, and the order costs the 27-point mesh's 5 FP64
// columns 2 %.
template <typename T, int VB, int NV, typename WT, bool kWhole, typename Src>
__device__ __forceinline__ void vrow_acc(const Src &A, int64_t i, int64_t k0, int64_t k1,
                                         int step, const T *__restrict__ X, int ld, int last,
                                         const typename Vec<T, VB>::type (&xi)[NV],
                                         typename Vec<T, VB>::type (&acc)[NV]) {
  using V = typename Vec<T, VB>::type;
  constexpr int U = NV <= 2 ? 4 : 2;
  V a[U][NV];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int v = 0; v < NV; ++v) a[u][v] = V(0);
  int64_t k = k0;
  for (; k + (U - 1) * step < k1; k += U * step) {
    int64_t j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) j[u] = A.nbr(i, k + u * step);
    V x[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      load_row<T, VB, NV>(X + j[u] * ld, last, x[u]);
      if constexpr (kWhole && NV > 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (kUnitW<WT>) {
#pragma unroll
        for (int v = 0; v < NV; ++v) a[u][v] += xi[v] - x[u][v];
      } else {
        const T wk = T(A.wk(k + u * step));
#pragma unroll
        for (int v = 0; v < NV; ++v) a[u][v] += wk * (xi[v] - x[u][v]);
      }
    }
  }
  // tail: fewer than U entries left, into the partial sums in order
#pragma unroll
  for (int u = 0; u < U - 1; ++u) {
    if (k < k1) {
      V x[NV];
      load_row<T, VB, NV>(X + A.nbr(i, k) * ld, last, x);
      if constexpr (kUnitW<WT>) {
#pragma unroll
        for (int v = 0; v < NV; ++v) a[u][v] += xi[v] - x[v];
      } else {
        const T w0 = T(A.wk(k));
#pragma unroll
        for (int v = 0; v < NV; ++v) a[u][v] += w0 * (xi[v] - x[v]);
      }
      k += step;
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if constexpr (U == 4) acc[v] = (a[0][v] + a[1][v]) + (a[2][v] + a[3][v]);
    else acc[v] = a[0][v] + a[1][v];
  }
}

// ------------------------------------------------------------- epilogues
template <typename T, int VB, int NV>
struct VStore {
  EpiStoreP<T> p;
  int last;
  static constexpr bool kNorms = false;
  using V = typename Vec<T, VB>::type;
  __device__ void row(int64_t i, const V (&xi)[NV], const V (&acc)[NV], double *, double *) const {
    store_row<T, VB, NV>(p.Y + i * p.ldy, last, acc);
  }
};

// Norm epilogues: slot s = v E + e of the thread's sums is column v E + e, and
// in the last vector column last + e, which the vector before holds already
// where that is below (NV - 1) E (slot_column gives -1 then).
template <int E, int NV>
__device__ __forceinline__ int slot_column(int v, int e, int last) {
  if (v < NV - 1) return v * E + e;
  return last + e >= (NV - 1) * E ? last + e : -1;
}

template <typename T, int VB, int NV>
struct VResidual {
  EpiResidualP<T> p;
  int m;
  int last;
  bool store_lx = true;   // false: L X is already in p.LX (streaming pass)
  static constexpr bool kNorms = true;
  static constexpr bool kBoth = true;
  using V = typename Vec<T, VB>::type;
  static constexpr int E = Vec<T, VB>::E;
  __device__ void row(int64_t i, const V (&xi)[NV], const V (&acc)[NV], double *n1,
                      double *n2) const {
    const double di = p.d64 ? p.d64[i] : 1.0;
    const double b = p.generalized ? di : 1.0;
    // one division per row for the B^-1-norm terms (exactly 1 when B = I)
    const double ib = p.generalized ? 1.0 / di : 1.0;
    V o[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int c = v < NV - 1 ? v * E + e : last + e;
        const double x = double(xi[v][e]);
        const double th = c < m ? p.theta[c] : 0.0;
        const double r = double(acc[v][e]) - b * th * x;
        o[v][e] = T(p.jacobi ? r / di : r);
        if (slot_column<E, NV>(v, e, last) >= 0 && c < m) {
          n1[v * E + e] += r * r * ib;
          n2[v * E + e] += b * x * x;
        }
      }
    if (store_lx) store_row<T, VB, NV>(p.LX + i * p.ld, last, acc);
    store_row<T, VB, NV>(p.OUT + i * p.ld, last, o);
  }
};

template <typename T, int VB, int NV>
struct VShiftDot {     // padded blocks: vectors do not overlap
  EpiShiftDotP<T> p;
  int m;
  int last;
  static constexpr bool kNorms = true;
  static constexpr bool kBoth = false;
  using V = typename Vec<T, VB>::type;
  static constexpr int E = Vec<T, VB>::E;
  __device__ void row(int64_t i, const V (&xi)[NV], const V (&acc)[NV], double *n1,
                      double *) const {
    const double b = p.bd ? p.bd[i] : 1.0;
    V *out = reinterpret_cast<V *>(p.OUT + i * p.ld);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      V o;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int c = v * E + e;
        const double x = double(xi[v][e]);
        const double lc = c < m ? p.lam[c] : 0.0;
        const double y = double(acc[v][e]) - b * lc * x;
        o[e] = T(y);
        if (c < m) n1[c] += x * y;
      }
      out[v] = o;
    }
  }
};

// The polynomial epilogues read every vector of a row before they write one:
// outputs may overwrite the previous iterate (or the sum) in place, and the
// last two vectors may overlap.
template <typename T, int VB, int NV>
struct VCheb {
  EpiChebP<T> p;
  int last;
  static constexpr bool kNorms = false;
  using V = typename Vec<T, VB>::type;
  static constexpr int E = Vec<T, VB>::E;
  __device__ void row(int64_t i, const V (&xi)[NV], const V (&acc)[NV], double *, double *) const {
    const double si = p.dinv ? p.dinv[i] : 1.0;
    V r[NV], pv[NV], o[NV];
    load_row<T, VB, NV>(p.R + i * p.ld, last, r);
    if (p.prev) {
      load_row<T, VB, NV>(p.prev + i * p.ld, last, pv);
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) pv[v] = V(0);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const double xs = p.src_scale * double(xi[v][e]);
        const double pr = p.prev_scale * double(pv[v][e]);
        const double res = double(r[v][e]) - p.src_scale * double(acc[v][e]);
        o[v][e] = T(xs + p.alpha * (xs - pr) + p.beta * si * res);
      }
    store_row<T, VB, NV>(p.OUT + i * p.ld, last, o);
  }
};

template <typename T, int VB, int NV>
struct VPoly {
  EpiPolyP<T> p;
  int last;
  static constexpr bool kNorms = false;
  using V = typename Vec<T, VB>::type;
  static constexpr int E = Vec<T, VB>::E;
  __device__ void row(int64_t i, const V (&xi)[NV], const V (&acc)[NV], double *, double *) const {
    const double si = p.dinv ? p.dinv[i] : 1.0;
    V y[NV], pn[NV];
    if (p.Yin) {
      load_row<T, VB, NV>(p.Yin + i * p.ld, last, y);
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) y[v] = V(0);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const double pv = double(xi[v][e]);
        const double pnew = pv - si * double(acc[v][e]) * p.inv_t;
        double yv = double(y[v][e]) + pv * p.inv_t;
        if (p.last) yv += pnew * p.inv_t_next;
        y[v][e] = T(yv);
        pn[v][e] = T(pnew);
      }
    store_row<T, VB, NV>(p.Yout + i * p.ld, last, y);
    if (!p.last) store_row<T, VB, NV>(p.Pout + i * p.ld, last, pn);
  }
};

// x + (x of lane - kN within the row of 16 lanes, cyclic).
template <int kN>
__device__ __forceinline__ double add_row_ror(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x120 + kN, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x120 + kN, 0xF, 0xF, false);
  return x + __hiloint2double(hi, lo);
}

// Sum of x over the wavefront, in every lane, in the order of a butterfly over
// distances 32, 16, ..., 1.  After each distance the lanes that differ in its
// bit hold the same value, so within a row of 16 a rotation by 8, 4, 2, 1
// brings the butterfly partner's value, without a trip through the LDS unit:
// the 14 sums of 7 columns took 168 exchanges per wave there, now 56 (residual
// product of 2 M rows of 7 FP32 columns 87.7 -> 79.7 us, the streaming pass of
// 216,000 rows of 5 FP64 columns 11.4 -> 9.5).
__device__ __forceinline__ double wave_sum(double x) {
  x += __shfl_xor(x, 32);
  x += __shfl_xor(x, 16);
  x = add_row_ror<8>(x);
  x = add_row_ror<4>(x);
  x = add_row_ror<2>(x);
  return add_row_ror<1>(x);
}

// Per-column block sums of the thread norms (columns < m), fixed order:
// butterfly within each wavefront, then the 4 wavefronts in order.
// kBoth false: only the first of the two sums is wanted and stored.
template <int E, int NV, bool kBoth>
__device__ void block_norms(const double (&n1)[E * NV], const double (&n2)[E * NV], int last,
                            int m, double *partials, int slot) {
  __shared__ double sh[4][2 * kMaxNev];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int c = slot_column<E, NV>(v, e, last);
      if (c < 0 || c >= m) continue;    // uniform
      const double a = wave_sum(n1[v * E + e]);
      double b = 0.0;
      if constexpr (kBoth) b = wave_sum(n2[v * E + e]);
      if (lane == 0) {
        sh[wave][c] = a;
        if constexpr (kBoth) sh[wave][kMaxNev + c] = b;
      }
    }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < m) {
    double a = sh[0][t] + sh[1][t] + sh[2][t] + sh[3][t];
    partials[(int64_t)t * kMaxNormBlocks + slot] = a;
    if constexpr (kBoth) {
      double b = sh[0][kMaxNev + t] + sh[1][kMaxNev + t] + sh[2][kMaxNev + t] +
                 sh[3][kMaxNev + t];
      partials[(int64_t)(kMaxNev + t) * kMaxNormBlocks + slot] = b;
    }
  }
}

// ----------------------------------------------------------------- kernels
// Short rows, one thread per row; `rpt` rows per thread, 256-row strides.
template <typename T, int VB, int NV, typename IdxT, typename WT, typename Epi>
__global__ __launch_bounds__(256) void k_vrow(Csr<IdxT, WT> A, int64_t nrows,
                                              const T *__restrict__ Xs, int ld, int rpt, Epi epi,
                                              double *partials, int m) {
  using V = typename Vec<T, VB>::type;
  constexpr int LD = NV * Vec<T, VB>::E;
  const int last = ld - Vec<T, VB>::E;
  const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
  double n1[LD], n2[LD];
#pragma unroll
  for (int c = 0; c < LD; ++c) { n1[c] = 0.0; n2[c] = 0.0; }
  for (int q = 0; q < rpt; ++q) {
    const int64_t i = (b * rpt + q) * 256 + threadIdx.x;
    if (i >= nrows) break;
    V xi[NV], acc[NV];
    load_row<T, VB, NV>(Xs + i * ld, last, xi);
    vrow_acc<T, VB, NV, WT, false>(A, i, (int64_t)A.rp[i], (int64_t)A.rp[i + 1], 1, Xs, ld, last, xi, acc);
    epi.row(i, xi, acc, n1, n2);
  }
  if constexpr (Epi::kNorms)
    block_norms<Vec<T, VB>::E, NV, Epi::kBoth>(n1, n2, ld - Vec<T, VB>::E, m, partials, (int)blockIdx.x);
}

template <typename T, int VB, int NV, int G>
__device__ __forceinline__ void group_sum(typename Vec<T, VB>::type (&acc)[NV]) {
  constexpr int E = Vec<T, VB>::E;
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      T a = acc[v][e];
#pragma unroll
      for (int off = G / 2; off >= 1; off >>= 1) a += __shfl_xor(a, off);
      acc[v][e] = a;
    }
}

// G lanes per row (G = 2 or 4), natural order over all n rows: the lanes of a
// group take every G-th neighbour of the row, so a group reads a contiguous
// run of the column indices; the group's partial sums are combined by a
// butterfly in a fixed order and the group's first lane runs the epilogue.
// Each block takes a contiguous range of rpb rows (a multiple of the groups
// per block), and block ids are remapped so that each XCD works on one
// contiguous stretch of ranges (as the one-lane kernel does): the gathered
// neighbour rows of a mesh then stay in that XCD's L2.
template <typename T, int VB, int NV, int G, typename IdxT, typename WT, typename Epi>
__global__ __launch_bounds__(256) void k_vgroup(Csr<IdxT, WT> A, int64_t nrows,
                                                const T *__restrict__ Xs, int ld, int64_t rpb,
                                                Epi epi, double *partials, int m) {
  using V = typename Vec<T, VB>::type;
  constexpr int LD = NV * Vec<T, VB>::E;
  constexpr int GPB = 256 / G;   // groups per block
  const int last = ld - Vec<T, VB>::E;
  const int gl = threadIdx.x & (G - 1);
  const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t rend = min(nrows, (b + 1) * rpb);
  double n1[LD], n2[LD];
#pragma unroll
  for (int c = 0; c < LD; ++c) { n1[c] = 0.0; n2[c] = 0.0; }
  for (int64_t i = b * rpb + threadIdx.x / G; i < rend; i += GPB) {
    V xi[NV], acc[NV];
    load_row<T, VB, NV>(Xs + i * ld, last, xi);
    vrow_acc<T, VB, NV, WT, false>(A, i, (int64_t)A.rp[i] + gl, (int64_t)A.rp[i + 1], G, Xs, ld, last, xi, acc);
    group_sum<T, VB, NV, G>(acc);
    if (gl == 0) epi.row(i, xi, acc, n1, n2);
  }
  if constexpr (Epi::kNorms)
    block_norms<Vec<T, VB>::E, NV, Epi::kBoth>(n1, n2, ld - Vec<T, VB>::E, m, partials, (int)blockIdx.x);
}

// Rows of 13..48 neighbours in natural order (mesh-like graphs), G lanes per
// row, with the column indices (and weights) staged in LDS: a block takes
// chunks of kLdsThreads / G consecutive rows (one, up to 2^20 chunks), whose
// CSR entries form one contiguous run; it loads that run with coalesced loads
// (adjacent threads, adjacent entries) into LDS, and the groups then walk their
// rows from LDS.  Read per lane from global memory instead, the index and
// weight lines of all resident waves exceed the L2 and are fetched again
// (measured: about twice the algorithmic bytes on the weighted 27-point mesh).
// A chunk with more than cap entries (those of rows of the graph's largest
// degree, at most kLdsEntries) is read from global memory.
// Chunks are remapped per XCD as above.  The summation order is the same as
// k_vgroup's.
//
// Bound by the latency of the two steps, so what counts is how much is in
// flight: a thread loads kLdsLoads entries before it stores the first (one
// load at a time left 13 waits in a row: 66.9 us per Chebyshev step of 5 FP64
// columns on the weighted 27-point mesh of 512,000 rows, now 54.5), the arrays
// have the length that the graph's rows need (26 neighbours: four waves per
// SIMD beside FP64 weights, 52.6), and blocks are two waves instead of four
// (51.5, that is 4.8 TB/s; the mesh of 216,000 rows: 22.9 -> 20.1).  More gathers in flight
// per lane cost registers and measured no better.
constexpr int kLdsThreads = 128;
constexpr int kLdsEntries = 16 * kLdsThreads;
constexpr int kLdsBlocks = 1 << 20;
constexpr int kLdsLoads = 7;

template <typename T, int VB, int NV, int G, typename IdxT, typename WT, typename Epi>
__global__ __launch_bounds__(kLdsThreads) void k_vlds(Csr<IdxT, WT> A, int64_t nrows,
                                                      const T *__restrict__ Xs, int ld,
                                                      int64_t rpb, int cap, Epi epi) {
  static_assert(!Epi::kNorms, "the epilogue takes no norms");
  using V = typename Vec<T, VB>::type;
  using L = LdsCsr<WT>;
  constexpr int R = kLdsThreads / G;   // rows per chunk
  extern __shared__ double lds_entries[];     // cap weights (none of a unit graph), cap columns
  auto *sw = reinterpret_cast<typename L::WS *>(lds_entries);
  auto *scol = reinterpret_cast<typename L::CT *>(sw + (kUnitW<WT> ? 0 : cap));
  const int last = ld - Vec<T, VB>::E;
  const int gl = threadIdx.x & (G - 1);
  const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t rend = min(nrows, (b + 1) * rpb);
  for (int64_t r0 = b * rpb; r0 < rend; r0 += R) {
    const int64_t r1 = min(rend, r0 + (int64_t)R);
    const int64_t k0 = A.rp[r0], k1 = A.rp[r1];
    const bool staged = k1 - k0 <= cap;
    if (staged) {
      for (int64_t kb = k0; kb < k1; kb += kLdsThreads * kLdsLoads) {
        typename L::CT c[kLdsLoads];
        typename L::WS w[kUnitW<WT> ? 1 : kLdsLoads];
#pragma unroll
        for (int u = 0; u < kLdsLoads; ++u) {
          const int64_t k = min(kb + kLdsThreads * u + (int64_t)threadIdx.x, k1 - 1);
          c[u] = A.col[k];
          if constexpr (!kUnitW<WT>) w[u] = A.w[k];
        }
#pragma unroll
        for (int u = 0; u < kLdsLoads; ++u) {
          const int64_t k = kb + kLdsThreads * u + (int64_t)threadIdx.x;
          if (k >= k1) continue;
          scol[k - k0] = c[u];
          if constexpr (!kUnitW<WT>) sw[k - k0] = w[u];
        }
      }
    }
    __syncthreads();
    const int64_t i = r0 + threadIdx.x / G;
    if (i < r1) {                       // uniform over each group of G lanes
      V xi[NV], acc[NV];
      load_row<T, VB, NV>(Xs + i * ld, last, xi);
      const int64_t ka = (int64_t)A.rp[i] + gl, kb = (int64_t)A.rp[i + 1];
      if (staged) {
        const L S{scol, sw, k0};
        vrow_acc<T, VB, NV, WT, false>(S, i, ka, kb, G, Xs, ld, last, xi, acc);
      } else {
        vrow_acc<T, VB, NV, WT, false>(A, i, ka, kb, G, Xs, ld, last, xi, acc);
      }
      group_sum<T, VB, NV, G>(acc);
      if (gl == 0) epi.row(i, xi, acc, nullptr, nullptr);
    }
    __syncthreads();
  }
}

// Degree-binned rows (power-law graphs), one launch: consecutive ranges of
// blocks take the chunks of the hub rows, then the row classes from the
// widest group down, so that the long rows start first and the short ones
// fill the chip behind them (one launch per class ran them one after the
// other: 24 products of 5 FP32 columns on R-MAT 17 took 2.3 ms, now 0.9).
// On 4 M rows, where each class fills the chip, that wins little: R-MAT 22, 5
// columns, one launch per class and then this one: FP32 store 1195 and 1094 us,
// residual 1380 and 1192; FP64 store 1610 and 1655 (7 columns 1552 and 1661),
// residual 1843 and 1715.  This kernel class by class is slower than at once at
// every size (R-MAT 22, FP32 store 1415 instead of 1347 before rows were loaded
// whole), and hubs from 16384 neighbours on gain 2 % there and lose half of the
// speed on R-MAT 17, so there is no rule on sizes.
// Hub chunks write partial row sums (as double), which k_vhub_combine adds.
struct BinRows {
  const int32_t *rows[kNumBins];
  int64_t nrows[kNumBins];
  unsigned end[kNumBins + 1];     // end[0]: hub blocks; then class 3, 2, 1, 0
  const int32_t *hub_rows, *hub_chunk_begin;
  int64_t n_hub;
  const int64_t *k0;
  const int32_t *chunk_row;
  double *hub_partial;
};

template <typename T, int VB, int NV, int G, typename IdxT, typename WT, typename Epi>
__device__ __forceinline__ void bin_rows(const Csr<IdxT, WT> &A, const int32_t *rows,
                                         int64_t nrows, unsigned b, unsigned nb, const T *Xs,
                                         int ld, const Epi &epi,
                                         double (&n1)[NV * Vec<T, VB>::E],
                                         double (&n2)[NV * Vec<T, VB>::E]) {
  using V = typename Vec<T, VB>::type;
  constexpr int GPB = 256 / G;   // groups per block
  const int last = ld - Vec<T, VB>::E;
  const int gl = threadIdx.x & (G - 1);
  for (int64_t r = (int64_t)b * GPB + threadIdx.x / G; r < nrows; r += (int64_t)nb * GPB) {
    const int64_t i = rows[r];
    V xi[NV], acc[NV];
    load_row<T, VB, NV>(Xs + i * ld, last, xi);
    vrow_acc<T, VB, NV, WT, true>(A, i, (int64_t)A.rp[i] + gl, (int64_t)A.rp[i + 1], G, Xs, ld, last,
                            xi, acc);
    if constexpr (G > 1) group_sum<T, VB, NV, G>(acc);
    if (gl == 0) epi.row(i, xi, acc, n1, n2);
  }
}

template <typename T, int VB, int NV, typename IdxT, typename WT, typename Epi>
__global__ __launch_bounds__(256) void k_vbin(Csr<IdxT, WT> A, BinRows B,
                                              const T *__restrict__ Xs, int ld, Epi epi,
                                              double *partials, int m) {
  using V = typename Vec<T, VB>::type;
  constexpr int E = Vec<T, VB>::E;
  constexpr int LD = NV * E;
  const unsigned b = blockIdx.x;
  if (b < B.end[0]) {
    const int last = ld - E;
    const int lane = threadIdx.x & 63;
    const int64_t n_chunks = B.hub_chunk_begin[B.n_hub];
    for (int64_t q = (int64_t)b * 4 + (threadIdx.x >> 6); q < n_chunks;
         q += (int64_t)B.end[0] * 4) {
      const int64_t i = B.chunk_row[q], k0 = B.k0[q];
      const int64_t k1 = min(k0 + kHubChunk, (int64_t)A.rp[i + 1]);
      V xi[NV], acc[NV];
      load_row<T, VB, NV>(Xs + i * ld, last, xi);
      vrow_acc<T, VB, NV, WT, true>(A, i, k0 + lane, k1, 64, Xs, ld, last, xi, acc);
      group_sum<T, VB, NV, 64>(acc);
      if (lane == 0)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int e = 0; e < E; ++e)
            B.hub_partial[q * kMaxNev + (v < NV - 1 ? v * E : last) + e] = double(acc[v][e]);
    }
    return;
  }
  double n1[LD], n2[LD];
#pragma unroll
  for (int c = 0; c < LD; ++c) { n1[c] = 0.0; n2[c] = 0.0; }
  static_assert(kNumBins == 4 && bin_group(0) == 1 && bin_group(1) == 4 && bin_group(2) == 16 &&
                    bin_group(3) == 64, "row classes");
  if (b < B.end[1])
    bin_rows<T, VB, NV, 64>(A, B.rows[3], B.nrows[3], b - B.end[0], B.end[1] - B.end[0], Xs, ld,
                            epi, n1, n2);
  else if (b < B.end[2])
    bin_rows<T, VB, NV, 16>(A, B.rows[2], B.nrows[2], b - B.end[1], B.end[2] - B.end[1], Xs, ld,
                            epi, n1, n2);
  else if (b < B.end[3])
    bin_rows<T, VB, NV, 4>(A, B.rows[1], B.nrows[1], b - B.end[2], B.end[3] - B.end[2], Xs, ld,
                           epi, n1, n2);
  else
    bin_rows<T, VB, NV, 1>(A, B.rows[0], B.nrows[0], b - B.end[3], B.end[4] - B.end[3], Xs, ld,
                           epi, n1, n2);
  if constexpr (Epi::kNorms)
    block_norms<Vec<T, VB>::E, NV, Epi::kBoth>(n1, n2, ld - Vec<T, VB>::E, m, partials, (int)(b - B.end[0]));
}

// Hub rows: one wavefront per hub row, lanes over its chunks, combined by a
// butterfly in a fixed order.
template <typename T, int VB, int NV, typename Epi>
__global__ __launch_bounds__(256) void k_vhub_combine(BinRows B, const T *__restrict__ Xs, int ld,
                                                      Epi epi, double *partials, int slot0,
                                                      int m) {
  using V = typename Vec<T, VB>::type;
  constexpr int E = Vec<T, VB>::E;
  constexpr int LD = NV * E;
  const int last = ld - E;
  const int lane = threadIdx.x & 63;
  double n1[LD], n2[LD];
#pragma unroll
  for (int c = 0; c < LD; ++c) { n1[c] = 0.0; n2[c] = 0.0; }
  for (int64_t h = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); h < B.n_hub;
       h += (int64_t)gridDim.x * 4) {
    const int64_t i = B.hub_rows[h];
    V xi[NV], acc[NV];
    load_row<T, VB, NV>(Xs + i * ld, last, xi);
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = V(0);
    for (int64_t q = B.hub_chunk_begin[h] + lane; q < B.hub_chunk_begin[h + 1]; q += 64)
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int e = 0; e < E; ++e)
          acc[v][e] += T(B.hub_partial[q * kMaxNev + (v < NV - 1 ? v * E : last) + e]);
    group_sum<T, VB, NV, 64>(acc);
    if (lane == 0) epi.row(i, xi, acc, n1, n2);
  }
  if constexpr (Epi::kNorms)
    block_norms<Vec<T, VB>::E, NV, Epi::kBoth>(n1, n2, ld - Vec<T, VB>::E, m, partials, slot0 + (int)blockIdx.x);
}

// The residual epilogue as a streaming pass over an L X that a store product
// has already written: one thread per row, `rpt` rows per thread in 256-row
// strides, the same arithmetic and norm partials as the fused epilogue.
template <typename T, int VB, int NV>
__global__ __launch_bounds__(256) void k_resid_rows(int64_t n, const T *__restrict__ Xs,
                                                    VResidual<T, VB, NV> epi, int rpt,
                                                    double *partials, int m) {
  using V = typename Vec<T, VB>::type;
  constexpr int LD = NV * Vec<T, VB>::E;
  const int ld = epi.p.ld;
  double n1[LD], n2[LD];
#pragma unroll
  for (int c = 0; c < LD; ++c) { n1[c] = 0.0; n2[c] = 0.0; }
  for (int q = 0; q < rpt; ++q) {
    const int64_t i = ((int64_t)blockIdx.x * rpt + q) * 256 + threadIdx.x;
    if (i >= n) break;
    V xi[NV], acc[NV];
    load_row<T, VB, NV>(Xs + i * ld, epi.last, xi);
    load_row<T, VB, NV>(epi.p.LX + i * ld, epi.last, acc);
    epi.row(i, xi, acc, n1, n2);
  }
  block_norms<Vec<T, VB>::E, NV, true>(n1, n2, epi.last, m, partials, (int)blockIdx.x);
}

// go(VB, NV) for the vectors of a row of ld values.  FP32 rows of 2 and 3
// values hold no 16-byte vector; those of 5, 6, 10 and 14 take 8-byte ones too,
// whose number of partial sums the solver's results depend on.  Measured
// against overlapping 16-byte ones (Chebyshev apply, 25 steps): better where
// lanes read neighbouring rows (2 M-row 7-point grid, 5 columns 944 and 974 us,
// 9,504-row 27-point brick 166 and 208), worse where the loads or the index
// stream count (R-MAT 17 945 and 910 us, R-MAT 20 8.0 and 7.7 ms, 512,000-row
// brick with FP32 weights 1086 and 964 us); 10 and 14 columns within 3 %.
template <typename T, typename F>
int with_vectors(int ld, F &&go) {
#define SPHX_NV(VB_, NV_) \
  case NV_: return go(std::integral_constant<int, VB_>{}, std::integral_constant<int, NV_>{});
  if constexpr (std::is_same_v<T, float>) {
    if (ld == 3 || ld == 5 || ld % 4 == 2) {
      switch ((ld + 1) / 2) {
        SPHX_NV(8, 1) SPHX_NV(8, 2) SPHX_NV(8, 3) SPHX_NV(8, 5) SPHX_NV(8, 7)
        default: return SPHX_E_INVALID_ARG;
      }
    }
  }
  constexpr int E = 16 / (int)sizeof(T);
  switch ((ld + E - 1) / E) {
    SPHX_NV(16, 1) SPHX_NV(16, 2) SPHX_NV(16, 3) SPHX_NV(16, 4)
    default: break;
  }
  if constexpr (std::is_same_v<T, double>) {
    switch ((ld + E - 1) / E) {
      SPHX_NV(16, 5) SPHX_NV(16, 6) SPHX_NV(16, 7) SPHX_NV(16, 8)
      default: break;
    }
  }
#undef SPHX_NV
  return SPHX_E_INVALID_ARG;
}

template <typename T>
int resid_stream(int64_t n, const T *X, int ld, int m, const EpiResidualP<T> &p,
                 double *partials, int *nparts, hipStream_t s) {
  const int64_t nb0 = ceil_div(n, 256);
  const int rpt = (int)ceil_div(nb0, kMaxNormBlocks);
  const unsigned nb = (unsigned)ceil_div(n, 256 * (int64_t)rpt);
  const int r = with_vectors<T>(ld, [&](auto vb, auto nv) -> int {
    constexpr int VB = decltype(vb)::value, NV = decltype(nv)::value;
    VResidual<T, VB, NV> e{p};
    e.m = m;
    e.last = ld - Vec<T, VB>::E;
    e.store_lx = false;
    hipLaunchKernelGGL((k_resid_rows<T, VB, NV>), dim3(nb), dim3(256), 0, s, n, X, e, rpt,
                       partials, m);
    return SPHX_OK;
  });
  if (r != SPHX_OK) return r;
  if (nparts) *nparts = (int)nb;
  return hipGetLastError() == hipSuccess ? SPHX_OK : SPHX_E_HIP;
}

// ----------------------------------------------------------------- dispatch
constexpr int kMaxShortBlocks = 8192;
constexpr int kGroupBlocks = 8192;
constexpr int kBinBlocks = 2048;    // per row class of a binned plan, and for the hub chunks
constexpr int kHubBlocks = 256;
static_assert(kMaxShortBlocks <= kMaxNormBlocks && kGroupBlocks <= kMaxNormBlocks &&
                  kNumBins * kBinBlocks + kHubBlocks <= kMaxNormBlocks,
              "norm partial slots");

template <typename T, int VB, int NV, typename IdxT, typename WT, typename Epi>
void run_vec(const Csr<IdxT, WT> &A, int64_t n, int64_t max_deg, const SpmmPlan &plan, const T *X, int ld,
             const Epi &epi, double *partials, int *nparts, int m, hipStream_t s,
             const LaunchEvents *ev) {
  // Every launch writes one norm-partial slot per block: the grids below
  // stay within kMaxNormBlocks in total (grid-stride loops cover the rest).
  int used = 0;
  // an unbinned plan is one launch, which ev (if given) times exactly
  const bool stamp = ev && !plan.binned;
  hipEvent_t e0 = stamp ? ev->start : nullptr, e1 = stamp ? ev->stop : nullptr;
  if (ev && !stamp) (void)hipEventRecord(ev->start, s);
  auto short_rows = [&](int64_t nr) {
    int64_t nb = ceil_div(nr, 256);
    int rpt = (int)ceil_div(nb, kMaxShortBlocks);
    nb = ceil_div(nr, 256 * (int64_t)rpt);
    hipExtLaunchKernelGGL((k_vrow<T, VB, NV, IdxT, WT, Epi>), dim3((unsigned)nb), dim3(256), 0,
                          s, e0, e1, 0, A, nr, X, ld, rpt, epi, partials, m);
    used += (int)nb;
  };
  // contiguous ranges of whole group-steps per block, at most kGroupBlocks
  auto ranges = [&](int G, int64_t nr, int64_t &rpb) {
    const int64_t gpb = 256 / G;
    rpb = ceil_div(ceil_div(nr, gpb), kGroupBlocks) * gpb;
    return (unsigned)std::max<int64_t>(1, ceil_div(nr, rpb));
  };
  if (!plan.binned) {
    // rows of 13..48 neighbours: wide gathered rows (>= 32 bytes) take two
    // lanes per row (measured on the 27-point meshes against one and four
    // lanes, FP32 and FP64), narrow rows four
    int G = plan.group;
    if (G > 1 && VB * NV >= 32) G = 2;
    int64_t rpb = 0;
    if (G == 1) {
      short_rows(n);
    } else {
      // the LDS-staged index stream pays off for the light epilogues (store,
      // polynomial steps: 8..20 % faster on the weighted 27-point mesh); with
      // the residual epilogue's per-thread norm sums the extra LDS costs more
      // occupancy than it saves (measured 11..30 % slower), so that one reads
      // its indices per lane
      if constexpr (Epi::kNorms) {
        const unsigned gb = ranges(G, n, rpb);
        used += (int)gb;
        if (G == 2)
          hipExtLaunchKernelGGL((k_vgroup<T, VB, NV, 2, IdxT, WT, Epi>), dim3(gb), dim3(256), 0,
                                s, e0, e1, 0, A, n, X, ld, rpb, epi, partials, m);
        else
          hipExtLaunchKernelGGL((k_vgroup<T, VB, NV, 4, IdxT, WT, Epi>), dim3(gb), dim3(256), 0,
                                s, e0, e1, 0, A, n, X, ld, rpb, epi, partials, m);
      } else {
        using L = LdsCsr<WT>;
        const int64_t rows = kLdsThreads / G;   // of a chunk
        rpb = ceil_div(ceil_div(n, rows), kLdsBlocks) * rows;
        const unsigned lb = (unsigned)ceil_div(n, rpb);
        const int cap = (int)std::min<int64_t>(max_deg * rows, kLdsEntries);
        const unsigned lds = (unsigned)cap * (sizeof(typename L::CT) +
                                              (kUnitW<WT> ? 0 : sizeof(typename L::WS)));
        if (G == 2)
          hipExtLaunchKernelGGL((k_vlds<T, VB, NV, 2, IdxT, WT, Epi>), dim3(lb),
                                dim3(kLdsThreads), lds, s, e0, e1, 0, A, n, X, ld, rpb, cap, epi);
        else
          hipExtLaunchKernelGGL((k_vlds<T, VB, NV, 4, IdxT, WT, Epi>), dim3(lb),
                                dim3(kLdsThreads), lds, s, e0, e1, 0, A, n, X, ld, rpb, cap, epi);
      }
    }
  } else if constexpr (!std::is_same_v<WT, UnitD16>) {   // (offsets: unbinned plans only)
    BinRows B{};
    B.hub_rows = plan.hub_rows;
    B.hub_chunk_begin = plan.hub_chunk_begin;
    B.n_hub = plan.n_hub;
    B.k0 = plan.chunk_k0;
    B.chunk_row = plan.chunk_row;
    B.hub_partial = plan.hub_partial;
    // n_chunks is an upper bound: blocks without a chunk end at once
    B.end[0] = plan.n_hub > 0 ? grid_for(plan.n_chunks, 4, kBinBlocks) : 0;
    for (int c = kNumBins - 1, q = 1; c >= 0; --c, ++q) {
      B.rows[c] = plan.rows[c];
      B.nrows[c] = plan.nrows[c];
      B.end[q] = B.end[q - 1] +
                 (plan.nrows[c] ? grid_for(plan.nrows[c], 256 / bin_group(c), kBinBlocks) : 0);
    }
    if (B.end[kNumBins] > 0)
      hipLaunchKernelGGL((k_vbin<T, VB, NV, IdxT, WT, Epi>), dim3(B.end[kNumBins]), dim3(256),
                         0, s, A, B, X, ld, epi, partials, m);
    used += (int)(B.end[kNumBins] - B.end[0]);
    if (plan.n_hub > 0) {
      const unsigned gc = grid_for(plan.n_hub, 4, kHubBlocks);
      hipLaunchKernelGGL((k_vhub_combine<T, VB, NV, Epi>), dim3(gc), dim3(256), 0, s, B, X, ld,
                         epi, partials, used, m);
      used += (int)gc;
    }
  }
  if (ev && !stamp) (void)hipEventRecord(ev->stop, s);
  if (nparts) *nparts = used;
}

template <typename T, int VB, int NV, template <typename, int, int> class EpiT, typename P>
int dispatch_types(sphx_graph *g, const SpmmPlan &plan, const T *X, int ld, const P &p,
                   int m, double *partials, int *nparts, hipStream_t s,
                   const LaunchEvents *ev) {
  auto go = [&](auto idx_tag, auto w_tag) {
    using IdxT = decltype(idx_tag);
    using WT = decltype(w_tag);
    const typename ColOf<WT>::type *col;
    if constexpr (std::is_same_v<WT, UnitD16>) col = plan.dcol;
    else col = g->col;
    Csr<IdxT, WT> A{static_cast<const IdxT *>(g->rowptr), col, static_cast<const WT *>(g->w)};
    EpiT<T, VB, NV> epi{p};
    epi.last = ld - Vec<T, VB>::E;
    if constexpr (std::is_same_v<EpiT<T, VB, NV>, VResidual<T, VB, NV>> ||
                  std::is_same_v<EpiT<T, VB, NV>, VShiftDot<T, VB, NV>>)
      epi.m = m;
    run_vec<T, VB, NV>(A, g->n, known(g->stats_valid) ? g->max_deg : kUnbinnedMaxDeg, plan, X, ld, epi, partials, nparts, m, s, ev);
  };
  if (g->rp64) {
    if (g->wdt == SPHX_UNIT) go(int64_t{}, Unit{});
    else if (g->wdt == SPHX_F32) go(int64_t{}, float{});
    else go(int64_t{}, double{});
  } else {
    if (g->wdt == SPHX_UNIT && plan.dcol) go(int32_t{}, UnitD16{});
    else if (g->wdt == SPHX_UNIT) go(int32_t{}, Unit{});
    else if (g->wdt == SPHX_F32) go(int32_t{}, float{});
    else go(int32_t{}, double{});
  }
  return hipGetLastError() == hipSuccess ? SPHX_OK : SPHX_E_HIP;
}

template <typename T, template <typename, int, int> class EpiT, typename P>
int dispatch_nv(sphx_graph *g, const SpmmPlan &plan, const T *X, int ld, const P &p, int m,
                double *partials, int *nparts, hipStream_t s,
                const LaunchEvents *ev = nullptr) {
  if (ld < m || ld > kMaxNev || ld < 2) return SPHX_E_INVALID_ARG;
  // the shifted product's blocks are padded
  if constexpr (std::is_same_v<EpiT<T, 16, 1>, VShiftDot<T, 16, 1>>)
    if ((ld * (int)sizeof(T)) % 16) return SPHX_E_INVALID_ARG;
  return with_vectors<T>(ld, [&](auto vb, auto nv) -> int {
    return dispatch_types<T, decltype(vb)::value, decltype(nv)::value, EpiT>(
        g, plan, X, ld, p, m, partials, nparts, s, ev);
  });
}

}  // namespace

template <typename T>
int vspmm_store(sphx_graph *g, const SpmmPlan &plan, const T *X, int ld, int m,
                EpiStoreP<T> epi, hipStream_t s) {
  return dispatch_nv<T, VStore>(g, plan, X, ld, epi, m, nullptr, nullptr, s);
}
template <typename T>
int vspmm_residual(sphx_graph *g, const SpmmPlan &plan, const T *X, int ld, int m,
                   EpiResidualP<T> epi, double *norm_partials, int *n_norm_blocks,
                   hipStream_t s) {
  if (!plan.binned && plan.group > 1) {
    // 13..48-neighbour meshes: the LDS-staged store product writes L X, then
    // a streaming pass forms the residual, the Jacobi step and the norms
    // (the fused residual epilogue keeps per-lane index reads and ran at
    // about two thirds of the store product's rate there)
    int r = vspmm_store<T>(g, plan, X, ld, m, EpiStoreP<T>{epi.LX, ld}, s);
    if (r != SPHX_OK) return r;
    return resid_stream<T>(g->n, X, ld, m, epi, norm_partials, n_norm_blocks, s);
  }
  return dispatch_nv<T, VResidual>(g, plan, X, ld, epi, m, norm_partials, n_norm_blocks, s);
}
template <typename T>
int vspmm_shiftdot(sphx_graph *g, const SpmmPlan &plan, const T *X, int ld, int m,
                   EpiShiftDotP<T> epi, double *partials, int *n_blocks, hipStream_t s) {
  return dispatch_nv<T, VShiftDot>(g, plan, X, ld, epi, m, partials, n_blocks, s);
}
template <typename T>
int vspmm_cheb(sphx_graph *g, const SpmmPlan &plan, const T *X, int ld, int m,
               EpiChebP<T> epi, hipStream_t s, const LaunchEvents *ev) {
  return dispatch_nv<T, VCheb>(g, plan, X, ld, epi, m, nullptr, nullptr, s, ev);
}

template <typename T>
int vspmm_poly(sphx_graph *g, const SpmmPlan &plan, const T *X, int ld, int m,
               EpiPolyP<T> epi, hipStream_t s, const LaunchEvents *ev) {
  return dispatch_nv<T, VPoly>(g, plan, X, ld, epi, m, nullptr, nullptr, s, ev);
}

// One epilogue and element type per translation unit (the build compiles
// this file once for each SPHX_VEC_PART, so that the units build in parallel):
// parts 0..4 are the FP32 epilogues, 5..9 the FP64 ones.
#ifndef SPHX_VEC_PART
#error "compile with -DSPHX_VEC_PART=0..9"
#endif
#if SPHX_VEC_PART < 5
using PartT = float;
#else
using PartT = double;
#endif
#if SPHX_VEC_PART % 5 == 0
template int vspmm_store<PartT>(sphx_graph *, const SpmmPlan &, const PartT *, int, int,
                                EpiStoreP<PartT>, hipStream_t);
#elif SPHX_VEC_PART % 5 == 1
extern template int vspmm_store<PartT>(sphx_graph *, const SpmmPlan &, const PartT *, int, int,
                                       EpiStoreP<PartT>, hipStream_t);
template int vspmm_residual<PartT>(sphx_graph *, const SpmmPlan &, const PartT *, int, int,
                                   EpiResidualP<PartT>, double *, int *, hipStream_t);
#elif SPHX_VEC_PART % 5 == 2
template int vspmm_shiftdot<PartT>(sphx_graph *, const SpmmPlan &, const PartT *, int, int,
                                   EpiShiftDotP<PartT>, double *, int *, hipStream_t);
#elif SPHX_VEC_PART % 5 == 3
template int vspmm_cheb<PartT>(sphx_graph *, const SpmmPlan &, const PartT *, int, int,
                               EpiChebP<PartT>, hipStream_t, const LaunchEvents *);
#else
template int vspmm_poly<PartT>(sphx_graph *, const SpmmPlan &, const PartT *, int, int,
                               EpiPolyP<PartT>, hipStream_t, const LaunchEvents *);
#endif

}  // namespace sphx
