// Dense block kernels of LOBPCG (Algorithm 1): initial blocks, Gram matrices
// on FP64 matrix cores, Rayleigh-Ritz in one workgroup, the fused block
// update, the convergence check, and final normalisation.
//
// Blocks are row-major n x ld (ld >= m; columns m..ld-1 are padding).  The
// Rayleigh-Ritz basis is
// S = [X, H_a, P_a] where a lists the active (unconverged) columns.
#include <cmath>

#include "kernels.h"

namespace sphx {
namespace {

// ------------------------------------------------------------ random init
// Counter-based normal draws: splitmix64 (Steele, Lea, Flood 2014) of the
// element counter gives two uniforms, Box-Muller turns them into N(0, 1).
__device__ __forceinline__ uint64_t splitmix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Element (i, c) draws from the counter i * m + c, independent of the padding.
template <typename T>
__global__ void k_init_random(T *X, int64_t n, int m, int ld, uint64_t seed) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * ld;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / ld;
    const int c = (int)(e - i * ld);
    if (c >= m) {
      X[e] = T(0);
      continue;
    }
    const uint64_t ctr = (uint64_t)(i * m + c);
    uint64_t a = splitmix64(seed ^ splitmix64(2 * ctr));
    uint64_t b = splitmix64(seed ^ splitmix64(2 * ctr + 1));
    double u1 = (double)((a >> 11) + 1) * 0x1.0p-53;   // (0, 1]
    double u2 = (double)(b >> 11) * 0x1.0p-53;         // [0, 1)
    X[e] = T(sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
  }
}

// Sec. 6.2.1: column 0 is the constant vector; column j >= 1 is the indicator
// of index block j-1 of d blocks [floor(b n / d), floor((b+1) n / d)).
template <typename T>
__global__ void k_init_piecewise(T *X, int64_t n, int m, int ld) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * ld;
       e += (int64_t)gridDim.x * blockDim.x) {
    int64_t i = e / ld;
    int c = (int)(e - i * ld);
    T v = T(0);
    if (c == 0) v = T(1);
    else if (c < m) {
      int64_t b = c - 1;
      int64_t lo = b * n / m, hi = (b + 1) * n / m;
      v = (i >= lo && i < hi) ? T(1) : T(0);
    }
    X[e] = v;
  }
}

// ------------------------------------------------------------------ Gram
typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kCh = 64;   // rows per LDS chunk

struct GramDev {
  int64_t n;
  int m, ld, w;
  int offH, offP;           // column offsets of the H and P parts in S
  int use_h, use_p;
  int inv[kMaxNev];         // inverse active map: column -> position or -1
  const double *bdiag;
};

// Source s of the basis: 0 X, 1 LX, 2 H, 3 LH, 4 P, 5 LP.  Even sources
// feed S, odd ones L S.  Column c of source s lands at S column
// off[s/2] + pos, pos = c (X) or the active position of c (H, P).
template <typename T>
struct GramSrc {
  const T *p[6];
};

constexpr int kPre = (kCh * kMaxNev + 255) / 256;   // staged values per thread and source

// Tiles: NT x NT tiles of 16 columns cover the padded width W = 16 NT; the
// upper ones (NT (NT + 1) / 2 per matrix) are formed.  kCompact (NT = 2,
// w <= 24): two tiles per matrix instead -- T1 = columns 0..15 against
// 0..15, and T2 = columns w-16..w-1 (rows) against 16..w-1 followed by
// 0..w-17 (columns), whose entries give the pairs with a column >= 16 (the
// ones against 0..w-17 by symmetry, stored transposed); one tile per wave.
template <typename T, int NT, bool kCompact = false>
__global__ __launch_bounds__(256) void k_gram(GramDev a, GramSrc<T> src,
                                              int64_t rows_per_block, double *partials) {
  static_assert(!kCompact || NT == 2, "compact tiles are for two-tile widths");
  constexpr int W = 16 * NT;
  constexpr int WP = W + 1;
  constexpr int NTILES = kCompact ? 4 : NT * (NT + 1);   // tiles of both matrices
  constexpr int TPW = (NTILES + 3) / 4;
  __shared__ double sS[kCh * WP];
  __shared__ double sL[kCh * WP];
  __shared__ double sb[kCh];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = t >> 6;
  const int m = a.m;
  const int ld = a.ld;
  for (int e = t; e < kCh * WP; e += blockDim.x) {
    sS[e] = 0.0;
    sL[e] = 0.0;
  }
  // tile ownership, and the S columns of this lane's tile row / column
  const int i16 = lane & 15;
  const int k4 = lane >> 4;
  const int wc = a.w - 16;      // compact: T2 row offset, and the width of its two column runs
  int tmat[TPW], tti[TPW], ttj[TPW], tci[TPW], tcj[TPW];
  d4 acc[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    int tt = wave + 4 * q;
    tmat[q] = -1;
    tti[q] = ttj[q] = 0;
    if (tt < NTILES) {
      if (kCompact) {
        tmat[q] = tt >> 1;
        tti[q] = tt & 1;          // 0: T1, 1: T2
      } else {
        int mat = tt / (NT * (NT + 1) / 2);
        int r = tt % (NT * (NT + 1) / 2);
        int ti = 0;
        while (r >= NT - ti) { r -= NT - ti; ++ti; }
        tmat[q] = mat;
        tti[q] = ti;
        ttj[q] = ti + r;
      }
    }
    if (kCompact) {
      const bool t2 = tti[q] == 1;
      tci[q] = t2 ? wc + i16 : i16;
      // T2 columns: 16..w-1, then 0..w-17, then a zero padding column
      tcj[q] = !t2 ? i16 : (i16 < wc ? 16 + i16 : (i16 < 2 * wc ? i16 - wc : W - 1));
    } else {
      tci[q] = tti[q] * 16 + i16;
      tcj[q] = ttj[q] * 16 + i16;
    }
    acc[q] = d4{0.0, 0.0, 0.0, 0.0};
  }
  // per staged slot: destination (row, S column) or -1
  const bool use[6] = {true, true, a.use_h != 0, a.use_h != 0, a.use_p != 0, a.use_p != 0};
  const int offs[3] = {0, a.offH, a.offP};
  int dst[3][kPre];
#pragma unroll
  for (int r = 0; r < kPre; ++r) {
    int e = t + 256 * r;
    int row = e / ld, c = e - row * ld;
    bool in = e < kCh * ld && c < m;
    dst[0][r] = in ? row * WP + c : -1;
    int pos = (in && a.inv[c] >= 0) ? a.inv[c] : -1;
    dst[1][r] = pos >= 0 ? row * WP + offs[1] + pos : -1;
    dst[2][r] = pos >= 0 ? row * WP + offs[2] + pos : -1;
  }
  const int64_t rb = (int64_t)blockIdx.x * rows_per_block;
  const int64_t re = min(a.n, rb + rows_per_block);
  T st[6][kPre];
  auto fetch = [&](int64_t r0) {
    const int64_t base = r0 * ld;
    const int64_t lim = (re - r0) * ld;   // valid elements of this chunk
#pragma unroll
    for (int s = 0; s < 6; ++s) {
#pragma unroll
      for (int r = 0; r < kPre; ++r) {
        int e = t + 256 * r;
        st[s][r] = (use[s] && dst[s >> 1][r] >= 0 && e < lim) ? src.p[s][base + e] : T(0);
      }
    }
  };
  __syncthreads();
  if (rb < re) fetch(rb);
  for (int64_t r0 = rb; r0 < re; r0 += kCh) {
    // stage the fetched chunk into LDS
#pragma unroll
    for (int s = 0; s < 6; ++s) {
      if (!use[s]) continue;
      double *dstm = (s & 1) ? sL : sS;
#pragma unroll
      for (int r = 0; r < kPre; ++r) {
        int d = dst[s >> 1][r];
        if (d >= 0) dstm[d] = double(st[s][r]);
      }
    }
    if (t < kCh) {
      int64_t gr = r0 + t;
      sb[t] = gr < re ? (a.bdiag ? a.bdiag[gr] : 1.0) : 0.0;
    }
    __syncthreads();
    // the next chunk's loads overlap the products below
    if (r0 + kCh < re) fetch(r0 + kCh);
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      if (tmat[q] < 0) continue;
      const int ci = tci[q];
      const int cj = tcj[q];
      if (tmat[q] == 0) {
#pragma unroll 4
        for (int kk = 0; kk < kCh; kk += 4) {
          int k = kk + k4;
          double av = sS[k * WP + ci];
          double bv = sL[k * WP + cj];
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[q], 0, 0, 0);
        }
      } else {
#pragma unroll 4
        for (int kk = 0; kk < kCh; kk += 4) {
          int k = kk + k4;
          double av = sS[k * WP + ci];
          double bv = sS[k * WP + cj] * sb[k];
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[q], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
  // D layout of the 16x16x4 FP64 product: accumulator register r of a lane
  // holds row 4*r + lane/16, column lane%16.
  double *out = partials + (int64_t)blockIdx.x * 2 * W * W;
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    if (tmat[q] < 0) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (kCompact && tti[q] == 1) {
        // T2 entry (row R, column C): the upper entry (R, C) for C >= 16,
        // R <= C; the upper entry (C, R) for C < w-16, R >= 16 (pairs with
        // both below 16 come from T1); nothing for the padding column
        const int R = wc + 4 * r + k4, C = tcj[q];
        int gi = -1, gj = -1;
        if (C >= 16 && C < a.w && R <= C) { gi = R; gj = C; }
        if (C < wc && R >= 16) { gi = C; gj = R; }
        if (gi >= 0) out[(int64_t)tmat[q] * W * W + gi * W + gj] = acc[q][r];
      } else {
        int gi = (kCompact ? 0 : tti[q] * 16) + 4 * r + k4;
        int gj = (kCompact ? 0 : ttj[q] * 16) + i16;
        out[(int64_t)tmat[q] * W * W + gi * W + gj] = acc[q][r];
      }
    }
  }
}

// Sum the block partials of upper tiles in block order: each block takes 16
// entries, 16 thread groups sum interleaved subsets of the partial blocks,
// and the 16 subset sums are added in a fixed order.
__global__ __launch_bounds__(256) void k_gram_reduce(const double *partials, int nblocks,
                                                     int NT, int w, double *out) {
  const int W = 16 * NT;
  const int E = 2 * W * W;
  const int t = threadIdx.x;
  const int e = blockIdx.x * 16 + (t & 15);
  const int sub = t >> 4;
  __shared__ double sh[256];
  double s0 = 0.0, s1 = 0.0;
  if (e < E) {
    int ij = e % (W * W);
    int i = ij / W, j = ij - i * W;
    if (i <= j && j < w) {
      int b = sub;
#pragma unroll 8
      for (; b + 16 < nblocks; b += 32) {
        s0 += partials[(int64_t)b * E + e];
        s1 += partials[(int64_t)(b + 16) * E + e];
      }
      if (b < nblocks) s0 += partials[(int64_t)b * E + e];
    }
  }
  sh[t] = s0 + s1;
  __syncthreads();
  if (t < 16 && e < E) {
    double tot = 0.0;
    for (int u = 0; u < 16; ++u) tot += sh[u * 16 + t];
    int mat = e / (W * W);
    int ij = e - mat * W * W;
    int i = ij / W, j = ij - i * W;
    out[mat * kMaxW * kMaxW + i * kMaxW + j] = tot;
  }
}

// --------------------------------------------------------- Rayleigh-Ritz
constexpr int LDA = kMaxW + 1;
static_assert(kMaxW < 64, "Rayleigh-Ritz pivot search: one candidate per lane of a wave");

// Cyclic Jacobi eigensolver (round-robin parallel ordering) on a k x k
// symmetric matrix.  For odd k the matrix carries one zero row and column k
// (its pairs never rotate), so that every pair of a round has two rows; kk is
// the even order.  The pairs (p, q), p < q, of one round are disjoint, so
// A <- R^T A R splits into independent 2 x 2 blocks (pair I's rows, pair J's
// columns).  In every wave, lane I computes the angle of pair I from the
// matrix of the previous round; each thread then takes one block, fetches
// the angles of I and J from those lanes, rotates its rows with I's angle,
// then its columns with J's (a row pass followed by a column pass; a pair
// that does not rotate has c = 1, s = 0, which leaves its entries exactly as
// they are); V <- V R likewise by blocks.  Before each sweep every pair is
// tested once: the sweeps stop when no pair would rotate.
//
// A round is bound by instruction issue (one or two waves work; a wave issues
// at most one FP64 operation per 4 cycles) and by its chain of LDS trips, so
// index work is kept out of it: the matrices are stored in the order of the
// round, pair I in rows and columns 2 I (p) and 2 I + 1 (q), so a thread's
// block is two aligned 16-byte reads at a fixed address, and each entry is
// written to its place in the next round's order, in the other buffer
// (JTab: per round and pair, the next byte offsets of its two rows and its two
// columns; one barrier per round).  Threads past the last block repeat block
// 0 of their kind, writing the same values, so that the loads need no branch.
// Measured, k_rr in all (rank 11 / 15 / 21 / 27, pencils of random H and P
// columns): 32.5 / 48.1 / 88.5 / 152 us, with the index arithmetic and 8-byte
// reads in the round 52.5 / 77.5 / 125 / 221 us.  The angles fetched through
// LDS instead of lane shuffles: 36.8 / 54.7 / 106 / 167 us.
constexpr int JLD = kMaxW + 2;            // row stride of the ordered matrices
constexpr int kJBuf = kMaxW * JLD;        // doubles of one of them
// [A, V, A', V']: the buffers alternate by round
constexpr int kJWork = 4 * kJBuf;

struct JTab {
  // low half: the pair's first (p) row or column, high half: the second (q)
  uint32_t row[kMaxW - 1][kMaxW / 2], col[kMaxW - 1][kMaxW / 2];
};
static_assert(kMaxW * JLD * 8 < 65536, "row byte offsets fit 16 bits");

// place of index i in the order of round 0 (pair 0 is (0, kk - 1), pair t is
// (t, kk - 1 - t)); the index at place 2 t is t, at 2 t + 1 it is kk - 1 - t
__device__ __forceinline__ int jacobi_place(int i, int kk) {
  return 2 * i < kk ? 2 * i : 2 * (kk - 1 - i) + 1;
}

// pair and slot, as one place, of index i in round r: kk - 1 meets r; any
// other index is r + t or r - t modulo kk - 1 and meets the other one
__device__ __forceinline__ int jacobi_place_at(int i, int r, int kk) {
  const int q = kk - 1;
  if (i == q) return 1;                   // pair 0, the larger index
  int d = i - r;
  d = d < 0 ? d + q : d;
  const int t = 2 * d < q ? d : q - d;
  if (t == 0) return 0;
  int j = 2 * d < q ? r - t : r + t;      // the partner
  j = j < 0 ? j + q : (j >= q ? j - q : j);
  return 2 * t + (i > j ? 1 : 0);
}

// rotations stop once an off-diagonal entry is at rounding level (a few ulps
// of ||A||), or negligible next to both diagonal entries:
// |a_pq| > 2e-16 sqrt(|a_pp a_qq|), compared in squares
__device__ __forceinline__ bool jacobi_rotates(double apq, double app, double aqq,
                                               double abs_floor) {
  return (fabs(apq) > abs_floor) & (apq * apq > 4e-32 * fabs(app * aqq));
}

// 1/x and 1/sqrt(x) from the hardware estimates and two Newton steps each
// (quadratic convergence from the estimate's error to a few ulps)
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  for (int i = 0; i < 2; ++i) {
    const double h = fma(-0.5 * x * y, y, 0.5);   // (1 - x y^2) / 2
    y = fma(y, h, y);
  }
  return y;
}

// Rotation (c, s) that annihilates a_pq (Rutishauser's form: the tangent
// t = sgn(th) / (|th| + sqrt(th^2 + 1)), th = (a_qq - a_pp) / (2 a_pq), the
// smaller root; c = 1 / sqrt(1 + t^2), s = t c); (1, 0) if the pair does not
// rotate.  th is clamped at 1e150 (then t ~ 1 / (2 th) underflows to a
// negligible rotation either way).
__device__ __forceinline__ void jacobi_rotation(double app, double aqq, double apq, bool rot,
                                                double &c, double &s) {
  const double h = rot ? 2.0 * apq : 1.0;
  double th = (aqq - app) * recip(h);
  th = fmin(fmax(th, -1e150), 1e150);
  const double q = fma(th, th, 1.0);
  const double den = fma(q, rsqrt_nr(q), fabs(th));
  const double tt = (th >= 0 ? 1.0 : -1.0) * recip(den);
  const double cc = rsqrt_nr(fma(tt, tt, 1.0));
  c = rot ? cc : 1.0;
  s = rot ? tt * cc : 0.0;
}

constexpr int kJacobiThreads = 256;
// blocks per thread and round: 2 (kMaxW / 2)^2 over kJacobiThreads threads
constexpr int kJacobiItems = (2 * (kMaxW / 2) * (kMaxW / 2) + kJacobiThreads - 1) / kJacobiThreads;

// The rounds' table for order kk, by threads first .. first + cnt - 1.
__device__ __forceinline__ void jacobi_table(JTab *tab, int kk, int first, int cnt) {
  const int id = (int)threadIdx.x - first;
  if (id < 0 || id >= cnt) return;
  uint16_t *row = reinterpret_cast<uint16_t *>(tab->row);
  uint16_t *col = reinterpret_cast<uint16_t *>(tab->col);
  for (int e = id; e < (kk - 1) * kk; e += cnt) {
    const int r = e / kk, i = e - r * kk;
    const int at = r * kMaxW + jacobi_place_at(i, r, kk);
    const int to = jacobi_place_at(i, r + 1 == kk - 1 ? 0 : r + 1, kk);
    row[at] = (uint16_t)(to * JLD * 8);
    col[at] = (uint16_t)(to * 8);
  }
}

typedef double d2 __attribute__((ext_vector_type(2)));

// The sweeps over work = [A, V, A', V'] (A and V in the order of round 0);
// returns the offset (0 or 2 kJBuf) of the final A, in the same order.
template <int kItems>
__device__ __forceinline__ int jacobi_sweeps(double *work, const JTab *tab, int k,
                                             double abs_floor, int *flags) {
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int kk = k + (k & 1);
  const int npair = kk / 2;              // <= kMaxW / 2 < 64: one pair per lane
  const int nblk = npair * npair;
  const int nwork = 2 * nblk;
  const int la = lane < npair ? 2 * lane * (JLD + 1) : 0;   // this lane's diagonal block
  // this thread's blocks: pair indices (V: rows 2 I and 2 I + 1 of V) and kind
  int bI[kItems], bJ[kItems], src[kItems];
  bool bV[kItems];
#pragma unroll
  for (int u = 0; u < kItems; ++u) {
    const int e = t + u * kJacobiThreads;
    bV[u] = e >= nblk;
    const int b = e < nblk ? e : (e < nwork ? e - nblk : 0);
    bI[u] = b / npair;
    bJ[u] = b - bI[u] * npair;
    src[u] = (bV[u] ? kJBuf : 0) + 2 * bI[u] * JLD + 2 * bJ[u];
  }
  int cur = 0;                           // offset of this round's A, V
  for (int sweep = 0; sweep < 40; ++sweep) {
    // flags cycle through three words: the one tested now was cleared two
    // sweeps ago, and read by every thread before the barriers of the last
    // sweep, when it is cleared again
    int *rot = flags + sweep % 3;
    if (t == 0) flags[(sweep + 1) % 3] = 0;
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      if (bV[u]) continue;
      const int I = bI[u], J = bJ[u];
      const double *a = work + cur + src[u];
      const double *dI = work + cur + 2 * I * (JLD + 1), *dJ = work + cur + 2 * J * (JLD + 1);
      // indices: place 2 I holds I, 2 I + 1 holds kk - 1 - I
      const int i0 = I, i1 = kk - 1 - I, j0 = J, j1 = kk - 1 - J;
      const double di0 = dI[0], di1 = dI[JLD + 1], dj0 = dJ[0], dj1 = dJ[JLD + 1];
      const bool any = ((i0 < j0) & jacobi_rotates(a[0], di0, dj0, abs_floor)) |
                       ((i0 < j1) & jacobi_rotates(a[1], di0, dj1, abs_floor)) |
                       ((i1 < j0) & jacobi_rotates(a[JLD], di1, dj0, abs_floor)) |
                       ((i1 < j1) & jacobi_rotates(a[JLD + 1], di1, dj1, abs_floor));
      if (any) *rot = 1;
    }
    __syncthreads();
    if (*rot == 0) break;
    for (int r = 0; r < kk - 1; ++r) {
      const int nxt = 2 * kJBuf - cur;
      if (wave * 64 < nwork) {           // the same for a whole wave
        const d2 ad = *reinterpret_cast<const d2 *>(work + cur + la);
        const double aqq = work[cur + la + JLD + 1];
        d2 x0[kItems], x1[kItems];
        uint32_t tr[kItems], tc[kItems];
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
          x0[u] = *reinterpret_cast<const d2 *>(work + cur + src[u]);
          x1[u] = *reinterpret_cast<const d2 *>(work + cur + src[u] + JLD);
          tr[u] = tab->row[r][bI[u]];
          tc[u] = tab->col[r][bJ[u]];
        }
        const bool rr = (lane < npair) & jacobi_rotates(ad[1], ad[0], aqq, abs_floor);
        double c, s;
        jacobi_rotation(ad[0], aqq, ad[1], rr, c, s);
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
          if (u * kJacobiThreads >= nwork) break;     // uniform
          const double cI0 = __shfl(c, bI[u]), sI0 = __shfl(s, bI[u]);
          const double cJ = __shfl(c, bJ[u]), sJ = __shfl(s, bJ[u]);
          const double cI = bV[u] ? 1.0 : cI0, sI = bV[u] ? 0.0 : sI0;
          const double a00 = x0[u][0], a01 = x0[u][1], a10 = x1[u][0], a11 = x1[u][1];
          const double b00 = fma(cI, a00, -(sI * a10)), b10 = fma(sI, a00, cI * a10);
          const double b01 = fma(cI, a01, -(sI * a11)), b11 = fma(sI, a01, cI * a11);
          // byte offsets (V: its rows stay)
          const uint32_t v0 = (uint32_t)(2 * bI[u] * JLD * 8);
          const uint32_t r0 = bV[u] ? v0 : tr[u] & 0xffffu;
          const uint32_t r1 = bV[u] ? v0 + JLD * 8 : tr[u] >> 16;
          const uint32_t c0 = tc[u] & 0xffffu, c1 = tc[u] >> 16;
          char *o = reinterpret_cast<char *>(work + nxt + (bV[u] ? kJBuf : 0));
          *reinterpret_cast<double *>(o + (r0 + c0)) = fma(cJ, b00, -(sJ * b01));
          *reinterpret_cast<double *>(o + (r0 + c1)) = fma(sJ, b00, cJ * b01);
          *reinterpret_cast<double *>(o + (r1 + c0)) = fma(cJ, b10, -(sJ * b11));
          *reinterpret_cast<double *>(o + (r1 + c1)) = fma(sJ, b10, cJ * b11);
        }
      }
      __syncthreads();
      cur = nxt;
    }
  }
  return cur;
}

// Eigenpairs of the k x k matrix A (LDS, stride LDA): lam[i], and V(i, c) at
// (returned pointer)[i * JLD + jacobi_place(c, kk)], kk = k + (k & 1).  A may
// not overlap work; tab is that of order kk.  Every thread of the block calls
// this, and the caller's writes of A and tab need a barrier before.  Ends with
// a barrier.
__device__ __forceinline__ const double *jacobi_eig(const double *A, double *work,
                                                    const JTab *tab, int k, double *lam,
                                                    int *flags) {
  __shared__ double anorm;
  const int t = threadIdx.x;
  const int kk = k + (k & 1);
  if (t < 64) {
    double s = 0.0;
    for (int e = t; e < k * k; e += 64) {
      int i = e / k, j = e - i * k;
      s = fma(A[i * LDA + j], A[i * LDA + j], s);
    }
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (t == 0) anorm = sqrt(s);
  } else {
    const int tx = t & 15, ty = (t - 64) >> 4;      // 12 rows of 16 threads
    for (int i = ty; i < kk; i += (kJacobiThreads - 64) / 16)
      for (int j = tx; j < kk; j += 16) {
        const int pj = jacobi_place(j, kk);
        work[jacobi_place(i, kk) * JLD + pj] = (i == k || j == k) ? 0.0 : A[i * LDA + j];
        work[kJBuf + i * JLD + pj] = (i == j) ? 1.0 : 0.0;
      }
  }
  if (t < 3) flags[t] = 0;
  __syncthreads();
  int cur = 0;
  if (k >= 2) {
    const double abs_floor = 4e-16 * anorm + 1e-300;
    // blocks per thread: one up to kk = 22 (the pencils of 7 vectors), two up
    // to kk = 32, else kJacobiItems
    const int nwork = kk * kk / 2;
    if (nwork <= kJacobiThreads) cur = jacobi_sweeps<1>(work, tab, k, abs_floor, flags);
    else if (nwork <= 2 * kJacobiThreads) cur = jacobi_sweeps<2>(work, tab, k, abs_floor, flags);
    else cur = jacobi_sweeps<kJacobiItems>(work, tab, k, abs_floor, flags);
  }
  if (t < k) lam[t] = work[cur + jacobi_place(t, kk) * (JLD + 1)];
  __syncthreads();
  return work + cur + kJBuf;
}

// Rayleigh-Ritz (Algorithm 1, RR(S, nev)) on the reduced Gram matrices.
//
// The columns of S are scaled to unit B-norm (Gs = D G_B D, As = D G_A D with
// D = diag(G_B)^-1/2).  A pivoted Cholesky factorisation of Gs picks, at each
// step, the column with the largest remaining Schur-complement diagonal and
// stops when that is at most drop_tol: the k chosen columns span the others
// up to the tolerance (those are dropped as linearly dependent), and
// Gs(piv, piv) = L L^T.  The rows of W = L^-1 are formed along with the
// columns of L: row k is W[k][c] = -(1 / l_kk) sum_j L[k][j] W[j][c] for
// c < k and 1 / l_kk for c = k.  With C = W^T, S(:, piv) C is B-orthonormal
// and the projected matrix A' = W As(piv, piv) W^T is diagonalised by cyclic
// Jacobi; the m smallest Ritz pairs give Y = D P W^T Z.  If fewer than m
// columns survive, the P block is dropped and the step retried once.
//
// The kernel is one workgroup and bound by latency and issue, so the
// factorisation runs in one wave without barriers, lane i holding row i: a
// step is the pivot search, one pass over the columns of L formed so far
// (left-looking: both sums take the broadcast entry L[p][q]; the terms are
// subtracted in the order of the steps) and one write of a column of L and a
// row of W.
constexpr int kRRThreads = kJacobiThreads;

// Maximum of x over the wave, in every lane: within each row of 16 lanes by
// DPP moves (swap of neighbours, of pairs, then the half-row and row mirrors,
// each pairing every lane with one holding the other half's largest so far),
// then across the four rows by lane reads.
template <int kCtrl>
__device__ __forceinline__ unsigned dpp_max(unsigned x) {
  const unsigned y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, 0xF, 0xF, false);
  return x > y ? x : y;
}
__device__ __forceinline__ unsigned wave_max(unsigned x) {
  x = dpp_max<0xB1>(x);    // quad_perm(1, 0, 3, 2)
  x = dpp_max<0x4E>(x);    // quad_perm(2, 3, 0, 1)
  x = dpp_max<0x141>(x);   // row_half_mirror
  x = dpp_max<0x140>(x);   // row_mirror
  unsigned b = (unsigned)__builtin_amdgcn_readlane((int)x, 0);
#pragma unroll
  for (int r = 1; r < 4; ++r) {
    const unsigned y = (unsigned)__builtin_amdgcn_readlane((int)x, 16 * r);
    b = b > y ? b : y;
  }
  return b;
}

// Lane of the largest positive d of the wave (the lowest lane on ties), in
// every lane, or -1.  Positive doubles order as their bits, so the high words
// decide unless several lanes share the largest one.
__device__ __forceinline__ int wave_pivot(double d) {
  const bool pos = d > 0.0;
  const unsigned hi = pos ? (unsigned)__double2hiint(d) : 0u;
  const unsigned lo = pos ? (unsigned)__double2loint(d) : 0u;
  const unsigned mh = wave_max(hi);
  unsigned long long who = __ballot(pos && hi == mh);
  if (who == 0ull) return -1;
  if (who & (who - 1)) {                       // uniform: more than one lane
    const unsigned ml = wave_max(hi == mh ? lo : 0u);
    who = __ballot(pos && hi == mh && lo == ml);
  }
  return __ffsll((long long)who) - 1;
}

// value of lane p (the same p in every lane)
__device__ __forceinline__ double lane_value(double v, int p) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), p),
                          __builtin_amdgcn_readlane(__double2loint(v), p));
}

__global__ __launch_bounds__(kRRThreads) void k_rr(const double *__restrict__ gram, RRArgs a,
                                                   double *Y, double *theta, DevStatus *st) {
  constexpr int MS = kMaxW * LDA;
  __shared__ __align__(16) double Msh[kJWork + 2 * MS];
  __shared__ JTab tab;
  // M1 and M2 share the rotations' buffers, which are filled from M3
  static_assert(MS <= kJBuf, "M1 and M2 fit the first two buffers");
  double *M1 = Msh, *M2 = Msh + kJBuf, *M3 = Msh + kJWork, *Wi = Msh + kJWork + MS;
  __shared__ double sc[kMaxW], lam[kMaxW];
  __shared__ int piv[kMaxW], ipiv[kMaxW], perm[kMaxW];
  __shared__ int flags[3], rank;
  const int t = threadIdx.x;
  const int w = a.w, m = a.m;
  const double *GA = gram;
  const double *GB = gram + kMaxW * kMaxW;
  int restarted = 0;
  for (int attempt = 0; attempt < 2; ++attempt) {
    const int wl = attempt == 0 ? w : a.p_begin;   // drop P on retry
    // M1 = Gs, M3 = As, M2 = the columns of L (column q in row q of M2);
    // after the factorisation M1, M2 and M3 take As(piv, piv),
    // As(piv, piv) W^T and A' in turn
    const int tx = t & 15, ty = t >> 4;
    for (int i = ty; i < wl; i += 16)
      for (int j = tx; j < wl; j += 16) {
        int lo = i < j ? i : j, hi = i < j ? j : i;
        M1[i * LDA + j] = GB[lo * kMaxW + hi];
        M3[i * LDA + j] = GA[lo * kMaxW + hi];
      }
    for (int e = t; e < (wl + 7) / 8 * 8 * LDA; e += blockDim.x) M2[e] = Wi[e] = 0.0;
    __syncthreads();
    if (t < kMaxW) {
      double g = (t < wl) ? M1[t * LDA + t] : 0.0;
      sc[t] = (t < wl && g > 0.0) ? 1.0 / sqrt(g) : 0.0;
      ipiv[t] = -1;
    }
    __syncthreads();
    for (int i = ty; i < wl; i += 16)
      for (int j = tx; j < wl; j += 16) {
        double sij = sc[i] * sc[j];
        M1[i * LDA + j] *= sij;
        M3[i * LDA + j] *= sij;
      }
    __syncthreads();
    if (t < 64) {
      // ---- pivoted Cholesky of Gs: lane i holds row i (lanes past the
      // matrix, and rows already chosen, hold d = 0 and never are a pivot)
      const int i = t < wl ? t : 0;
      double d = t < wl ? M1[i * LDA + i] : 0.0;
      bool open = t < wl;
      int k = 0;
      for (; k < wl; ++k) {
        const int p = wave_pivot(d);
        if (p < 0) break;
        const double pval = lane_value(d, p);
        if (!(pval > a.drop_tol)) break;
        const double rd = 1.0 / sqrt(pval);
        // s = Gs[p][i] - sum_q L[p][q] L[i][q], v = sum_q L[p][q] W[q][i]
        double s = M1[p * LDA + i], v = 0.0;
        const double *lp = M2 + p, *lq = M2 + i, *wq = Wi + i;
        // (rows k .. of M2 and Wi are zero, so whole groups of 8 are taken)
        for (int q = 0; q < k; q += 8, lp += 8 * LDA, lq += 8 * LDA, wq += 8 * LDA) {
          double b[8], l[8], x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            b[u] = lp[u * LDA];
            l[u] = lq[u * LDA];
            x[u] = wq[u * LDA];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            s = fma(-b[u], l[u], s);
            v = fma(b[u], x[u], v);
          }
        }
        const double l = open ? s * rd : 0.0;
        if (t == p) open = false;
        d = open ? fma(-l, l, d) : 0.0;
        if (t < wl) {
          M2[k * LDA + t] = l;
          Wi[k * LDA + t] = t < k ? -rd * v : (t == k ? rd : 0.0);
        }
        if (t == 0) {
          piv[k] = p;
          ipiv[p] = k;
        }
        // one wave: its LDS writes are read in order by the next step
        wave_order();
      }
      if (t == 0) rank = k;
    } else {
      // the other waves prepare the rotations' table meanwhile
      jacobi_table(&tab, wl + (wl & 1), 64, kRRThreads - 64);
    }
    __syncthreads();
    const int k = rank;
    if (k >= m || attempt == 1 || a.p_begin >= w) {
      if (k < m) {
        // breakdown: keep X as it is
        for (int e = t; e < kMaxW * kMaxNev; e += blockDim.x) {
          int i = e / kMaxNev, c = e - i * kMaxNev;
          Y[e] = (i == c && c < m) ? 1.0 : 0.0;
        }
        if (t == 0) {
          st->kept = k;
          st->restarted = restarted;
          st->breakdown = 1;
        }
        return;
      }
      // Ap = As(piv, piv) -> M1; the table again if columns were dropped
      if (k + (k & 1) != wl + (wl & 1)) jacobi_table(&tab, k + (k & 1), 0, kRRThreads);
      for (int i = ty; i < k; i += 16)
        for (int j = tx; j < k; j += 16) M1[i * LDA + j] = M3[piv[i] * LDA + piv[j]];
      __syncthreads();
      // T = Ap W^T -> M2 (W lower triangular: j <= c)
      for (int i = ty; i < k; i += 16)
        for (int c = tx; c < k; c += 16) {
          double s0 = 0.0, s1 = 0.0;
          int j = 0;
#pragma unroll 4
          for (; j + 1 <= c; j += 2) {
            s0 = fma(M1[i * LDA + j], Wi[c * LDA + j], s0);
            s1 = fma(M1[i * LDA + j + 1], Wi[c * LDA + j + 1], s1);
          }
          if (j <= c) s0 = fma(M1[i * LDA + j], Wi[c * LDA + j], s0);
          M2[i * LDA + c] = s0 + s1;
        }
      __syncthreads();
      // A' = W T -> M3 (j <= i), upper triangle computed and mirrored
      for (int i = ty; i < k; i += 16)
        for (int c = tx; c < k; c += 16) {
          if (i > c) continue;
          double s0 = 0.0, s1 = 0.0;
          int j = 0;
#pragma unroll 4
          for (; j + 1 <= i; j += 2) {
            s0 = fma(Wi[i * LDA + j], M2[j * LDA + c], s0);
            s1 = fma(Wi[i * LDA + j + 1], M2[(j + 1) * LDA + c], s1);
          }
          if (j <= i) s0 = fma(Wi[i * LDA + j], M2[j * LDA + c], s0);
          M3[i * LDA + c] = s0 + s1;
          M3[c * LDA + i] = s0 + s1;
        }
      __syncthreads();
      // eigenpairs of A'
      const double *Z = jacobi_eig(M3, Msh, &tab, k, lam, flags);
      const int kk = k + (k & 1);
      if (t < k) {
        int below = 0;
        double v = lam[t];
#pragma unroll 4
        for (int j = 0; j < k; ++j)
          below += ((lam[j] < v) | ((lam[j] == v) & (j < t))) ? 1 : 0;
        perm[below] = t;
      }
      __syncthreads();
      // Y (basis row i, Ritz vector c) = sc_i (W^T z_perm[c])[position of
      // i], 0 if dropped
      for (int e = t; e < kMaxW * kMaxNev; e += blockDim.x) {
        int i = e / kMaxNev, c = e - i * kMaxNev;
        double v = 0.0;
        if (i < wl && c < m && ipiv[i] >= 0) {
          const int r = ipiv[i], zc = jacobi_place(perm[c], kk);
          double s0 = 0.0, s1 = 0.0;
          int j = r;
#pragma unroll 4
          for (; j + 1 < k; j += 2) {
            s0 = fma(Wi[j * LDA + r], Z[j * JLD + zc], s0);
            s1 = fma(Wi[(j + 1) * LDA + r], Z[(j + 1) * JLD + zc], s1);
          }
          if (j < k) s0 = fma(Wi[j * LDA + r], Z[j * JLD + zc], s0);
          v = sc[i] * (s0 + s1);
        }
        Y[e] = v;
      }
      if (t < m) theta[t] = lam[perm[t]];
      if (t == 0) {
        st->kept = k;
        st->restarted = restarted;
        st->breakdown = 0;
      }
      return;
    }
    restarted = 1;
    __syncthreads();
  }
}

// --------------------------------------------------- polynomial roots
// Harmonic Ritz values of a Lanczos projection (the roots of the GMRES
// residual polynomial): H is (k1 + 1) x k1 row-major (stride k1).  They are
// the eigenvalues of the pencil (H^T H, H_k) with H_k the leading k1 x k1
// block (symmetrised): H_k = L L^T (Cholesky), C = L^-1 H^T H L^-T, cyclic
// Jacobi.  The roots are written in modified Leja order: the largest first,
// then each maximising the sum of log distances to those already chosen
// (lowest index on ties).  status: 0, or 1 if H_k is not positive definite.
__global__ __launch_bounds__(kJacobiThreads) void k_harmonic_ritz(const double *__restrict__ Hg, int k1,
                                                       double *theta, int *status) {
  constexpr int MS = kMaxW * LDA;
  __shared__ __align__(16) double Msh[kJWork + MS];
  __shared__ JTab tab;
  double *Mk = Msh, *Mv = Msh + kJBuf, *Mc = Msh + kJWork;
  __shared__ double lam[kMaxW];
  __shared__ int flags[3], bad;
  const int t = threadIdx.x;
  // Mk = sym(H_k), Mc = H^T H
  for (int e = t; e < k1 * k1; e += blockDim.x) {
    const int i = e / k1, j = e - i * k1;
    Mk[i * LDA + j] = 0.5 * (Hg[i * k1 + j] + Hg[j * k1 + i]);
    double sum = 0.0;
    for (int r = 0; r <= k1; ++r) sum += Hg[r * k1 + i] * Hg[r * k1 + j];
    Mc[i * LDA + j] = sum;
  }
  if (t == 0) bad = 0;
  jacobi_table(&tab, k1 + (k1 & 1), 0, kJacobiThreads);
  __syncthreads();
  // Cholesky of Mk in place (lower), one thread
  if (t == 0) {
    for (int j = 0; j < k1 && !bad; ++j) {
      double d = Mk[j * LDA + j];
      for (int q = 0; q < j; ++q) d -= Mk[j * LDA + q] * Mk[j * LDA + q];
      if (!(d > 0.0)) { bad = 1; break; }
      d = sqrt(d);
      Mk[j * LDA + j] = d;
      for (int i = j + 1; i < k1; ++i) {
        double v = Mk[i * LDA + j];
        for (int q = 0; q < j; ++q) v -= Mk[i * LDA + q] * Mk[j * LDA + q];
        Mk[i * LDA + j] = v / d;
      }
    }
  }
  __syncthreads();
  if (bad) {
    if (t == 0) *status = 1;
    return;
  }
  // T = L^-1 Mc (column per thread) -> Mv
  if (t < k1) {
    for (int i = 0; i < k1; ++i) {
      double v = Mc[i * LDA + t];
      for (int q = 0; q < i; ++q) v -= Mk[i * LDA + q] * Mv[q * LDA + t];
      Mv[i * LDA + t] = v / Mk[i * LDA + i];
    }
  }
  __syncthreads();
  // C = L^-1 T^T (column c has right-hand side row c of T) -> Mc
  if (t < k1) {
    for (int i = 0; i < k1; ++i) {
      double v = Mv[t * LDA + i];
      for (int q = 0; q < i; ++q) v -= Mk[i * LDA + q] * Mc[q * LDA + t];
      Mc[i * LDA + t] = v / Mk[i * LDA + i];
    }
  }
  __syncthreads();
  for (int e = t; e < k1 * k1; e += blockDim.x) {
    const int i = e / k1, j = e - i * k1;
    if (i < j) {
      const double v = 0.5 * (Mc[i * LDA + j] + Mc[j * LDA + i]);
      Mc[i * LDA + j] = v;
      Mc[j * LDA + i] = v;
    }
  }
  __syncthreads();
  // Mk (the factor) and Mv are free now: they lie in the rotations' buffers
  (void)jacobi_eig(Mc, Msh, &tab, k1, lam, flags);
  if (t == 0) {
    bool used[kMaxW];
    for (int i = 0; i < k1; ++i) used[i] = false;
    int first = 0;
    for (int i = 1; i < k1; ++i)
      if (fabs(lam[i]) > fabs(lam[first])) first = i;
    theta[0] = lam[first];
    used[first] = true;
    double score[kMaxW];
    for (int i = 0; i < k1; ++i) score[i] = 0.0;
    int last = first;
    for (int q = 1; q < k1; ++q) {
      int best = -1;
      for (int i = 0; i < k1; ++i) {
        if (used[i]) continue;
        score[i] += log(fabs(lam[i] - lam[last]));
        if (best < 0 || score[i] > score[best]) best = i;
      }
      theta[q] = lam[best];
      used[best] = true;
      last = best;
    }
    *status = 0;
  }
}

// --------------------------------------------------------------- update
struct UpdDev {
  int64_t n;
  int pos[kMaxNev];   // column -> position among the active ones, or -1
  int use_h, use_p;
  int offH, offP;     // rows of Y for the H and P parts
  int update_lp;      // also LP <- LH y_H + LP y_P
};

// One row per thread, M = m columns in registers; the Rayleigh-Ritz
// coefficients are the same for every thread, so they come through the scalar
// cache.  Every output is a sum in a fixed order: the H part over the active
// columns, then the P part, plus the X part over k.  Bound by the blocks'
// bytes.  With rows and coefficients in LDS each multiply-add waited on two
// LDS reads; what a row per thread costs instead is registers and lines read in
// parts, so
//  - a thread has one row only: over several, the compiler keeps the
//    coefficients from one to the next, in scalar registers and then in lanes of
//    vector ones (1306 lane moves among 3856 instructions at 16 FP64 columns);
//  - FP32 and padded rows form P, then X, then L P, each from its own loads
//    (kPhased); FP64 rows of exactly M values load X, H and P at once, up to 8
//    columns also L H and L P (kFront: small solves are bound by latency);
//  - padded rows (LD > M) are read and written whole by 16-byte accesses, the
//    padding as zeros: their M values alone were written as parts of lines.
// us per update, with LDS, with all rows in registers, and now: 2 M rows of 7
// FP32 columns 90, 48, 45; of 16 FP64 columns 431, 561, 385; 860,000 rows (R-MAT
// 20) of 5 FP32 columns 33.8, 23.7, 20.9; of 16 FP64 columns 152, 209, 141.  On
// 190,000 rows (R-MAT 18), which the cache holds, 14 and 16 FP64 columns take
// 39.5, 50.8, 48.1 and 46.2, 73.8, 48.8.
template <typename T, int LD>
__device__ __forceinline__ void upd_load(const T *__restrict__ p, T (&x)[LD]) {
  constexpr int E = 16 / (int)sizeof(T);
  if constexpr (LD % E == 0) {
    typedef T V __attribute__((ext_vector_type(E)));
#pragma unroll
    for (int v = 0; v < LD / E; ++v) {
      const V q = reinterpret_cast<const V *>(p)[v];
#pragma unroll
      for (int e = 0; e < E; ++e) x[v * E + e] = q[e];
    }
  } else {
#pragma unroll
    for (int c = 0; c < LD; ++c) x[c] = p[c];
  }
}
template <typename T, int M, int LD>
__device__ __forceinline__ void upd_store(T *p, const double (&x)[M]) {
  constexpr int E = 16 / (int)sizeof(T);
  if constexpr (LD % E == 0) {
    typedef T V __attribute__((ext_vector_type(E)));
#pragma unroll
    for (int v = 0; v < LD / E; ++v) {
      V q;
#pragma unroll
      for (int e = 0; e < E; ++e) q[e] = v * E + e < M ? T(x[v * E + e < M ? v * E + e : 0]) : T(0);
      reinterpret_cast<V *>(p)[v] = q;
    }
  } else {
#pragma unroll
    for (int c = 0; c < LD; ++c) p[c] = c < M ? T(x[c < M ? c : 0]) : T(0);
  }
}

template <typename T, int M, int LD>
__global__ __launch_bounds__(256) void k_update(T *X, const T *__restrict__ H, T *P,
                                                const T *__restrict__ LH, T *LP,
                                                const double *__restrict__ Y, UpdDev a) {
  constexpr bool kPhased = sizeof(T) == 4 || LD != M, kFront = !kPhased && M <= 8;
  const bool write_p = a.use_h || a.use_p;
  const bool lp_too = a.update_lp;
  // s += sum over the active columns k of v_k Y[off + pos_k], in increasing k
  auto add = [&](double (&s)[M], const T (&v)[LD], int off) {
#pragma unroll
    for (int k = 0; k < M; ++k)
      if (a.pos[k] >= 0) {
        const double *y = Y + (off + a.pos[k]) * kMaxNev;
        const double vd = double(v[k]);
#pragma unroll
        for (int c = 0; c < M; ++c) s[c] = fma(vd, y[c], s[c]);
      }
  };
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.n) return;
  const int64_t o = i * LD;
  T xr[LD], hr[LD], pr[LD], lh[LD], lp[LD];
  double p[M], x[M];
  auto load_l = [&]() {
    if (a.use_h) upd_load<T, LD>(LH + o, lh);
    if (a.use_p) upd_load<T, LD>(LP + o, lp);
  };
  if constexpr (!kPhased) upd_load<T, LD>(X + o, xr);
  if (a.use_h) upd_load<T, LD>(H + o, hr);
  if (a.use_p) upd_load<T, LD>(P + o, pr);
  if (kFront && lp_too) load_l();
#pragma unroll
  for (int c = 0; c < M; ++c) p[c] = x[c] = 0.0;
  if (a.use_h) add(p, hr, a.offH);
  if (a.use_p) add(p, pr, a.offP);
  if constexpr (kPhased) {
    __builtin_amdgcn_sched_barrier(0);
    upd_load<T, LD>(X + o, xr);
  }
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const double v = double(xr[k]);
#pragma unroll
    for (int c = 0; c < M; ++c) x[c] = fma(v, Y[k * kMaxNev + c], x[c]);
  }
#pragma unroll
  for (int c = 0; c < M; ++c) x[c] += p[c];
  upd_store<T, M, LD>(X + o, x);
  if (write_p) upd_store<T, M, LD>(P + o, p);
  if constexpr (kPhased) __builtin_amdgcn_sched_barrier(0);
  if (lp_too) {
    double l[M];
#pragma unroll
    for (int c = 0; c < M; ++c) l[c] = 0.0;
    if constexpr (!kFront) load_l();
    if (a.use_h) add(l, lh, a.offH);
    if (a.use_p) add(l, lp, a.offP);
    upd_store<T, M, LD>(LP + o, l);
  }
}

// ------------------------------------------------------------- finalize
// Sum the sum-major partials (sum q of block b at partials[q * stride + b])
// over b in a fixed order -> out[q] for the 2m sums q < m and
// kMaxNev <= q < kMaxNev + m.  One wavefront per sum: lanes stride over the
// blocks into eight accumulators (independent loads in flight), which are
// combined in a fixed tree, then a butterfly across lanes.
constexpr int kSumThreads = 1024;
__device__ void sum_partials_block(const double *partials, int nblocks, int stride, int m,
                                   double *out) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  for (int j = wave; j < 2 * m; j += nw) {
    const int q = j < m ? j : kMaxNev + (j - m);
    const double *p = partials + (int64_t)q * stride;
    double v[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int b = lane;
    for (; b + 7 * 64 < nblocks; b += 8 * 64) {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] += p[b + u * 64];
    }
#pragma unroll
    for (int u = 0; u < 7; ++u)
      if (b + u * 64 < nblocks) v[u] += p[b + u * 64];
    double r = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    for (int off = 32; off >= 1; off >>= 1) r += __shfl_xor(r, off);
    if (lane == 0) out[q] = r;
  }
  __syncthreads();
}

// Residuals rho from the norm partials, one lane per column, and the active
// list; the whole status also goes to the host's copy (pinned, mapped), which
// the host reads after the stream's synchronisation.
__global__ __launch_bounds__(kSumThreads) void k_finalize(const double *partials, int nblocks,
                                                          int m, const double *theta,
                                                          double tol, int locking,
                                                          DevStatus *st, DevStatus *host) {
  __shared__ double sums[2 * kMaxNev];
  __shared__ DevStatus now;
  static_assert(sizeof(DevStatus) % 4 == 0 && sizeof(DevStatus) / 4 <= kSumThreads, "status words");
  const int t = threadIdx.x;
  constexpr int kWords = sizeof(DevStatus) / 4;
  if (t < kWords) reinterpret_cast<int *>(&now)[t] = reinterpret_cast<const int *>(st)[t];
  const int c = t < m ? t : 0;
  const double th = theta[c], floor_th = m > 1 ? theta[1] : theta[0];
  sum_partials_block(partials, nblocks, kMaxNormBlocks, m, sums);
  if (t < 64) {
    double scale = fmax(th, floor_th);
    if (!(scale > 0.0)) scale = 1.0;
    const double rn = sqrt(sums[c]), xn = sqrt(sums[kMaxNev + c]);
    const double rho = xn > 0.0 ? rn / (scale * xn) : INFINITY;
    const bool conv = rho <= tol;
    const int nconv = __popcll(__ballot(t < m && conv));
    const bool act = t < m && (!conv || (!locking && nconv < m));
    const unsigned long long who = __ballot(act);
    if (t < m) {
      now.rho[t] = rho;
      now.theta[t] = th;
    }
    if (act) now.act[__popcll(who & ((1ull << t) - 1ull))] = t;
    if (t == 0) {
      now.nact = __popcll(who);
      now.nconv = nconv;
    }
  }
  __syncthreads();
  if (t < kWords) {
    const int v = reinterpret_cast<const int *>(&now)[t];
    reinterpret_cast<int *>(st)[t] = v;
    reinterpret_cast<int *>(host)[t] = v;
  }
  __threadfence_system();
}

__global__ __launch_bounds__(kSumThreads) void k_sum_partials(const double *partials,
                                                              int nblocks, int stride, int m,
                                                              double *out) {
  __shared__ double sums[2 * kMaxNev];
  if (threadIdx.x < 2 * kMaxNev) sums[threadIdx.x] = 0.0;
  __syncthreads();
  sum_partials_block(partials, nblocks, stride, m, sums);
  if (threadIdx.x < 2 * kMaxNev) out[threadIdx.x] = sums[threadIdx.x];
}

// Per-column block sums with a fixed lane -> column assignment, stored
// sum-major with stride kRqStride.
__device__ void colsum2(int c, double v1, double v2, int m, double *partials) {
  __shared__ double s1[256], s2[256];
  __shared__ int sc[256];
  int t = threadIdx.x;
  s1[t] = v1;
  s2[t] = v2;
  sc[t] = c;
  __syncthreads();
  if (t < m) {
    double a = 0.0, b = 0.0;
    for (int u = 0; u < (int)blockDim.x; ++u)
      if (sc[u] == t) { a += s1[u]; b += s2[u]; }
    partials[(int64_t)t * kRqStride + blockIdx.x] = a;
    partials[(int64_t)(kMaxNev + t) * kRqStride + blockIdx.x] = b;
  }
}

// Rayleigh quotient partials: sum x.lx and sum b x^2 per column (blocks of
// row stride ld; thread t takes column t % lanes of rows t / lanes).
template <typename T>
__global__ __launch_bounds__(256) void k_rq(const T *X, const double *LX, int64_t n, int m,
                                            int ld, int lanes, const double *bdiag,
                                            double *partials) {
  const int rc = 256 / lanes;
  const int row = threadIdx.x / lanes;
  const int c = threadIdx.x % lanes;
  const bool live = threadIdx.x < rc * lanes && c < m;
  double a = 0.0, b = 0.0;
  if (live)
    for (int64_t r = (int64_t)blockIdx.x * rc + row; r < n; r += (int64_t)gridDim.x * rc) {
      double x = double(X[r * ld + c]);
      double bd = bdiag ? bdiag[r] : 1.0;
      a += x * LX[r * ld + c];
      b += bd * x * x;
    }
  colsum2(live ? c : -1, a, b, m, partials);
}

// Residual partials: sum (lx - theta b x)^2 / b and sum b x^2 per column.
template <typename T>
__global__ __launch_bounds__(256) void k_res(const T *X, const double *LX, int64_t n, int m,
                                             int ld, int lanes, const double *bdiag,
                                             const double *theta, double *partials) {
  const int rc = 256 / lanes;
  const int row = threadIdx.x / lanes;
  const int c = threadIdx.x % lanes;
  const bool live = threadIdx.x < rc * lanes && c < m;
  double a = 0.0, b = 0.0;
  if (live) {
    double th = theta[c];
    for (int64_t r = (int64_t)blockIdx.x * rc + row; r < n; r += (int64_t)gridDim.x * rc) {
      double x = double(X[r * ld + c]);
      double bd = bdiag ? bdiag[r] : 1.0;
      double res = LX[r * ld + c] - th * bd * x;
      a += res * res / bd;
      b += bd * x * x;
    }
  }
  colsum2(live ? c : -1, a, b, m, partials);
}

// Column argmax |x| (lowest index on ties): block partials (value, index).
template <typename T>
__global__ __launch_bounds__(256) void k_colmax(const T *X, int64_t n, int m, double *pv,
                                                int64_t *pi) {
  const int rc = 256 / m;
  const int row = threadIdx.x / m;
  const int c = threadIdx.x % m;
  const bool live = threadIdx.x < rc * m;
  double bv = -1.0;
  int64_t bi = INT64_MAX;
  if (live)
    for (int64_t r = (int64_t)blockIdx.x * rc + row; r < n; r += (int64_t)gridDim.x * rc) {
      double v = fabs(double(X[r * m + c]));
      if (v > bv || (v == bv && r < bi)) { bv = v; bi = r; }
    }
  __shared__ double sv[256];
  __shared__ int64_t si[256];
  __shared__ int scol[256];
  sv[threadIdx.x] = bv;
  si[threadIdx.x] = bi;
  scol[threadIdx.x] = live ? c : -1;
  __syncthreads();
  if (threadIdx.x < m) {
    double v = -1.0;
    int64_t ix = INT64_MAX;
    for (int u = threadIdx.x; u < rc * m; u += m)
      if (scol[u] == (int)threadIdx.x)
        if (sv[u] > v || (sv[u] == v && si[u] < ix)) { v = sv[u]; ix = si[u]; }
    pv[blockIdx.x * kMaxNev + threadIdx.x] = v;
    pi[blockIdx.x * kMaxNev + threadIdx.x] = ix;
  }
}

// one wavefront per column: lanes over the blocks' maxima, then a butterfly
// (larger value, then lower index: the order does not matter)
template <typename T>
__global__ __launch_bounds__(64 * kMaxNev) void k_colsign(const T *X, int m, int nblocks,
                                                          const double *pv, const int64_t *pi,
                                                          double *sign) {
  const int c = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (c >= m) return;                   // uniform over the wave
  double v = -1.0;
  int64_t ix = INT64_MAX;
  for (int b = lane; b < nblocks; b += 64) {
    const double bv = pv[b * kMaxNev + c];
    const int64_t bi = pi[b * kMaxNev + c];
    if (bv > v || (bv == v && bi < ix)) { v = bv; ix = bi; }
  }
  for (int off = 32; off >= 1; off >>= 1) {
    const double ov = __shfl_xor(v, off);
    const int64_t oi = (int64_t)__shfl_xor((long long)ix, off);
    if (ov > v || (ov == v && oi < ix)) { v = ov; ix = oi; }
  }
  if (lane == 0) {
    const double x = (ix == INT64_MAX) ? 1.0 : double(X[ix * m + c]);
    sign[c] = x < 0 ? -1.0 : 1.0;
  }
}

struct Scales { double s[kMaxNev]; };

template <typename T>
__global__ void k_colscale(T *X, int64_t n, int m, const double *sign, Scales sc) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * m;
       e += (int64_t)gridDim.x * blockDim.x) {
    int c = (int)(e % m);
    X[e] = T(double(X[e]) * sign[c] * sc.s[c]);
  }
}

template <typename Tin, typename Tout>
__global__ void k_convert(const Tin *in, Tout *out, int64_t count) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * blockDim.x)
    out[e] = Tout(in[e]);
}

template <typename T>
__global__ void k_copy_cols(const T *in, int ldin, T *out, int ldout, int64_t n, int m) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * m;
       e += (int64_t)gridDim.x * blockDim.x) {
    int64_t i = e / m;
    int c = (int)(e - i * m);
    out[i * ldout + c] = in[i * ldin + c];
  }
}

}  // namespace

// ------------------------------------------------------------ launchers
template <typename T>
void launch_init_random(T *X, int64_t n, int m, int ld, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL((k_init_random<T>), dim3(grid_for(n * ld, 256, 4096)), dim3(256), 0, s,
                     X, n, m, ld, seed);
}
template <typename T>
void launch_init_piecewise(T *X, int64_t n, int m, int ld, hipStream_t s) {
  hipLaunchKernelGGL((k_init_piecewise<T>), dim3(grid_for(n * ld, 256, 4096)), dim3(256), 0,
                     s, X, n, m, ld);
}

size_t gram_partial_doubles(int max_blocks) {
  return (size_t)max_blocks * 2 * kMaxW * kMaxW;
}

template <typename T>
int gram(const T *X, const T *LX, const T *H, const T *LH, const T *P, const T *LP,
         const GramArgs &a, double *partials, int max_blocks, double *gram_out,
         hipStream_t s) {
  GramDev d;
  d.n = a.n;
  d.m = a.m;
  d.ld = a.ld;
  int na = a.act.count;
  d.use_h = a.use_h && na > 0;
  d.use_p = a.use_p && na > 0;
  d.offH = a.m;
  d.offP = a.m + (d.use_h ? na : 0);
  d.w = a.m + (d.use_h ? na : 0) + (d.use_p ? na : 0);
  for (int c = 0; c < kMaxNev; ++c) d.inv[c] = -1;
  for (int q = 0; q < na; ++q) d.inv[a.act.col[q]] = q;
  d.bdiag = a.bdiag;
  int NT = (d.w + 15) / 16;
  int64_t rows_per_block = ceil_div(a.n, max_blocks);
  rows_per_block = ceil_div(rows_per_block, kCh) * kCh;
  int nb = (int)ceil_div(a.n, rows_per_block);
  if (nb < 1) nb = 1;
  GramSrc<T> sp{{X, LX, H, LH, P, LP}};
  switch (NT) {
    case 1:
      hipLaunchKernelGGL((k_gram<T, 1>), dim3(nb), dim3(256), 0, s, d, sp, rows_per_block,
                         partials);
      break;
    case 2:
      if (d.w <= 24)
        hipLaunchKernelGGL((k_gram<T, 2, true>), dim3(nb), dim3(256), 0, s, d, sp,
                           rows_per_block, partials);
      else
        hipLaunchKernelGGL((k_gram<T, 2>), dim3(nb), dim3(256), 0, s, d, sp, rows_per_block,
                           partials);
      break;
    case 3:
      hipLaunchKernelGGL((k_gram<T, 3>), dim3(nb), dim3(256), 0, s, d, sp, rows_per_block,
                         partials);
      break;
    default:
      return SPHX_E_INVALID_ARG;
  }
  int W = 16 * NT;
  hipLaunchKernelGGL(k_gram_reduce, dim3((unsigned)ceil_div(2 * W * W, 16)), dim3(256), 0, s,
                     (const double *)partials, nb, NT, d.w, gram_out);
  return hipGetLastError() == hipSuccess ? SPHX_OK : SPHX_E_HIP;
}

void launch_harmonic_ritz(const double *H, int k1, double *theta, int *status,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_harmonic_ritz, dim3(1), dim3(kJacobiThreads), 0, s, H, k1, theta, status);
}

void launch_rr(const double *gram_out, const RRArgs &a, double *Y, double *theta,
               DevStatus *st, hipStream_t s) {
  hipLaunchKernelGGL(k_rr, dim3(1), dim3(kRRThreads), 0, s, gram_out, a, Y, theta, st);
}

template <typename T>
int launch_update(T *X, const T *H, T *P, const T *LH, T *LP, const double *Y,
                  const UpdateArgs &a, hipStream_t s) {
  UpdDev d;
  d.n = a.n;
  const int na = a.act.count;
  for (int c = 0; c < kMaxNev; ++c) d.pos[c] = -1;
  for (int q = 0; q < na; ++q) d.pos[a.act.col[q]] = q;
  d.use_h = a.use_h && na > 0;
  d.use_p = a.use_p && na > 0;
  d.offH = a.m;
  d.offP = a.m + (d.use_h ? na : 0);
  d.update_lp = LP != nullptr && (d.use_h || d.use_p);
  const unsigned gb = (unsigned)ceil_div(a.n, 256);   // n < 2^31
  auto go = [&](auto m, auto ld) {
    hipLaunchKernelGGL((k_update<T, decltype(m)::value, decltype(ld)::value>), dim3(gb),
                       dim3(256), 0, s, X, H, P, LH, LP, Y, d);
  };
#define SPHX_UPD(M_)                                                                \
  case M_: {                                                                        \
    constexpr int kExact = M_ < 2 ? 2 : M_, kPadded = padded_ld(M_, sizeof(T));     \
    const std::integral_constant<int, M_> m;                                        \
    if (a.ld == kExact) go(m, std::integral_constant<int, kExact>{});               \
    else if (a.ld == kPadded) go(m, std::integral_constant<int, kPadded>{});        \
    else return SPHX_E_INVALID_ARG;                                                 \
    break;                                                                          \
  }
  switch (a.m) {
    SPHX_UPD(1) SPHX_UPD(2) SPHX_UPD(3) SPHX_UPD(4) SPHX_UPD(5) SPHX_UPD(6) SPHX_UPD(7)
    SPHX_UPD(8) SPHX_UPD(9) SPHX_UPD(10) SPHX_UPD(11) SPHX_UPD(12) SPHX_UPD(13) SPHX_UPD(14)
    SPHX_UPD(15) SPHX_UPD(16)
    default: return SPHX_E_INVALID_ARG;
  }
#undef SPHX_UPD
  return hipGetLastError() == hipSuccess ? SPHX_OK : SPHX_E_HIP;
}

void launch_finalize(const double *norm_partials, int n_blocks, int m, const double *theta,
                     double tol, int locking, DevStatus *st, DevStatus *host, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kSumThreads), 0, s, norm_partials, n_blocks, m,
                     theta, tol, locking, st, host);
}

template <typename T>
void launch_rq_partials(const T *X, const double *LX, int64_t n, int m, int ld, int lanes,
                        const double *bdiag, double *partials, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL((k_rq<T>), dim3(nblocks), dim3(256), 0, s, X, LX, n, m, ld, lanes,
                     bdiag, partials);
}
template <typename T>
void launch_res_partials(const T *X, const double *LX, int64_t n, int m, int ld, int lanes,
                         const double *bdiag, const double *theta, double *partials,
                         int nblocks, hipStream_t s) {
  hipLaunchKernelGGL((k_res<T>), dim3(nblocks), dim3(256), 0, s, X, LX, n, m, ld, lanes,
                     bdiag, theta, partials);
}
void launch_sum_partials(const double *partials, int nblocks, int cols, double *out,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kSumThreads), 0, s, partials, nblocks,
                     kRqStride, cols, out);
}

constexpr int kColBlocks = 256;
size_t normalize_scratch_bytes() {
  return (size_t)kColBlocks * kMaxNev * (sizeof(double) + sizeof(int64_t)) + 256 * 8;
}

template <typename T>
int normalize_columns(T *X, int64_t n, int m, const double *scale_host, void *scratch,
                      hipStream_t s) {
  double *pv = static_cast<double *>(scratch);
  int64_t *pi = reinterpret_cast<int64_t *>(pv + kColBlocks * kMaxNev);
  double *sign = reinterpret_cast<double *>(pi + kColBlocks * kMaxNev);
  int nb = (int)grid_for(n, 256 / m, kColBlocks);
  hipLaunchKernelGGL((k_colmax<T>), dim3(nb), dim3(256), 0, s, X, n, m, pv, pi);
  hipLaunchKernelGGL((k_colsign<T>), dim3(1), dim3(64 * kMaxNev), 0, s, X, m, nb, pv, pi, sign);
  Scales sc;
  for (int c = 0; c < kMaxNev; ++c) sc.s[c] = c < m ? scale_host[c] : 1.0;
  hipLaunchKernelGGL((k_colscale<T>), dim3(grid_for(n * m, 256, 4096)), dim3(256), 0, s, X, n,
                     m, (const double *)sign, sc);
  return hipGetLastError() == hipSuccess ? SPHX_OK : SPHX_E_HIP;
}

template <typename Tin, typename Tout>
void launch_convert(const Tin *in, Tout *out, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL((k_convert<Tin, Tout>), dim3(grid_for(count, 256, 4096)), dim3(256), 0, s,
                     in, out, count);
}
template <typename T>
void launch_copy_cols(const T *in, int ldin, T *out, int ldout, int64_t n, int m,
                      hipStream_t s) {
  hipLaunchKernelGGL((k_copy_cols<T>), dim3(grid_for(n * m, 256, 4096)), dim3(256), 0, s, in,
                     ldin, out, ldout, n, m);
}

#define SPHX_INST(T)                                                                        \
  template void launch_init_random<T>(T *, int64_t, int, int, uint64_t, hipStream_t);      \
  template void launch_init_piecewise<T>(T *, int64_t, int, int, hipStream_t);             \
  template int gram<T>(const T *, const T *, const T *, const T *, const T *, const T *,   \
                       const GramArgs &, double *, int, double *, hipStream_t);            \
  template int launch_update<T>(T *, const T *, T *, const T *, T *, const double *,      \
                                 const UpdateArgs &, hipStream_t);                         \
  template void launch_rq_partials<T>(const T *, const double *, int64_t, int, int, int,   \
                                      const double *, double *, int, hipStream_t);         \
  template void launch_res_partials<T>(const T *, const double *, int64_t, int, int, int,  \
                                       const double *, const double *, double *, int,      \
                                       hipStream_t);                                       \
  template int normalize_columns<T>(T *, int64_t, int, const double *, void *, hipStream_t); \
  template void launch_copy_cols<T>(const T *, int, T *, int, int64_t, int, hipStream_t);
SPHX_INST(float)
SPHX_INST(double)
#undef SPHX_INST
template void launch_convert<float, double>(const float *, double *, int64_t, hipStream_t);
template void launch_convert<double, float>(const double *, float *, int64_t, hipStream_t);
template void launch_convert<double, double>(const double *, double *, int64_t, hipStream_t);
template void launch_convert<float, float>(const float *, float *, int64_t, hipStream_t);

}  // namespace sphx
