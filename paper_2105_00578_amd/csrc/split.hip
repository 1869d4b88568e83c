// Coordinate split of the spectral embedding into K parts (Algorithm 2, the
// multi-jagged split of Sec. 4).
//
// One level per prime factor p of K, largest first; level l splits every
// current section into p children along coordinate l mod ncoord.  The
// members of a section are ordered by the composite key (value, vertex id),
// value mapped to an order-preserving unsigned integer with -0 == +0, so every
// key is unique.  Cut j (1 <= j < p) of a section of weight W follows the
// prefix whose weight C minimises |p C - j W|, the shorter prefix on ties
// (for p = 2: |2 W_lo - W|); children are the members between consecutive
// cuts and part ids are the mixed-radix digits, most significant first.
//
// A cut is found without sorting: for every (section, cut) target a radix
// select over the bytes of the composite key (most significant first) finds
// the first member e* whose inclusive prefix weight C reaches j W / p; e*
// itself is included iff that brings |p C - j W| strictly down.  Integer
// vertex weights make every histogram exact, so the result does not depend
// on the order of the atomic additions.
//
// Levels of up to kFastSections sections and kFastCuts cuts narrow each target
// down first (split_levels): the composite keys of a sorted random sample cut
// the coordinate into bins of about equal weight (2048 over all sections),
// one pass bins every member, the bin that holds a target is found from the
// sections' histograms, and only its members (about n / 2048) go through the
// radix select, in one workgroup's LDS.  The bins are intervals of the
// composite order, so ties and any distribution of the values are as good as
// another, unless the levels before have cut a section out of few of its
// coordinate's bins: a target whose bin is too full for its list raises a flag,
// its level and those after select nothing, and the radix passes over all members
// (in split_mj, also for more sections or cuts, and where fast_levels expects
// such bins) are run instead.  2 M members, K = 64, FP32: 1.13 ms by the radix
// passes (8 per level, each over all members, the first ones with most
// members in a few counters), 0.35 ms by sample bins, of which the strided
// reads of the coordinates take about a third.
#include <algorithm>
#include <cstring>
#include <vector>

#include "kernels.h"

namespace sphx {
namespace {

template <typename T> struct Ord;
template <> struct Ord<float> {
  using K = uint32_t;
  __device__ static K map(float v, bool &nan) {
    if (v != v) { nan = true; return 0; }
    if (v == 0.0f) v = 0.0f;                      // -0 -> +0
    uint32_t u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  }
};
template <> struct Ord<double> {
  using K = uint64_t;
  __device__ static K map(double v, bool &nan) {
    if (v != v) { nan = true; return 0; }
    if (v == 0.0) v = 0.0;
    uint64_t u = (uint64_t)__double_as_longlong(v);
    return (u & 0x8000000000000000ull) ? ~u : (u | 0x8000000000000000ull);
  }
};

template <typename T>
__global__ void k_keys(const T *coords, int ld, int c, int64_t n, typename Ord<T>::K *keys,
                       int *flag) {
  bool nan = false;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    keys[i] = Ord<T>::map(coords[i * ld + c], nan);
  if (nan) atomicOr(flag, 1);
}

// byte d of the composite key (ord, id), most significant first
template <typename K>
__device__ __forceinline__ int digit(K ord, uint32_t id, int d) {
  constexpr int OB = sizeof(K);
  if (d < OB) return (int)((ord >> (8 * (OB - 1 - d))) & 0xFF);
  return (int)((id >> (8 * (3 - (d - OB)))) & 0xFF);
}

// do the first d bytes of (ord, id) equal those of the prefix (pord, pid)?
// (prefix bytes beyond d are zero)
template <typename K>
__device__ __forceinline__ bool prefix_match(K ord, uint32_t id, K pord, uint32_t pid, int d) {
  constexpr int OB = sizeof(K);
  if (d == 0) return true;
  if (d < OB) {
    K mask = ~K(0) << (8 * (OB - d));
    return (ord & mask) == pord;
  }
  if (ord != pord) return false;
  int dd = d - OB;
  if (dd == 0) return true;
  uint32_t mask = dd >= 4 ? ~0u : (~0u << (8 * (4 - dd)));
  return (id & mask) == pid;
}

// Up to 32 targets count in LDS first (16 or 32 rows of 256 bins), more in
// global memory.
constexpr int kLdsTargets = 32;

// Histogram of byte d over the members of every target's section whose first
// d key bytes match the target's prefix.  Target t = s * (p - 1) + j - 1.
// LT: targets held in LDS (0: global atomics).
template <typename K, int LT>
__global__ __launch_bounds__(256) void k_hist(int64_t n, const K *__restrict__ keys,
                                              const int32_t *__restrict__ part,
                                              const int32_t *__restrict__ vwgt, int d, int p,
                                              int ntgt, const K *__restrict__ pord,
                                              const uint32_t *__restrict__ pid,
                                              unsigned long long *hist) {
  constexpr bool kLds = LT > 0;
  __shared__ unsigned long long h[kLds ? LT * 256 : 1];
  if constexpr (kLds) {
    for (int e = threadIdx.x; e < ntgt * 256; e += blockDim.x) h[e] = 0;
    __syncthreads();
  }
  const int pm = p - 1;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int s = part[i];
    const K o = keys[i];
    const uint32_t id = (uint32_t)i;
    const unsigned long long wt = vwgt ? (unsigned long long)vwgt[i] : 1ull;
    const int b = digit(o, id, d);
    for (int j = 0; j < pm; ++j) {
      const int t = s * pm + j;
      if (!prefix_match(o, id, pord[t], pid[t], d)) continue;
      if constexpr (kLds) atomicAdd(&h[t * 256 + b], wt);
      else atomicAdd(&hist[(int64_t)t * 256 + b], wt);
    }
  }
  if constexpr (kLds) {
    __syncthreads();
    for (int e = threadIdx.x; e < ntgt * 256; e += blockDim.x)
      if (h[e]) atomicAdd(&hist[e], h[e]);
  }
}

// One wavefront per target: choose byte d (the first bucket where p * C
// reaches j * W), clear the histogram row.  Lane l holds buckets 4l .. 4l+3;
// the weight before a lane's buckets is an exclusive scan over the lanes, and
// the lowest lane with a qualifying bucket holds the choice.
template <typename K>
__global__ __launch_bounds__(256) void k_select(int ntgt, int p, int d, int nd,
                                                unsigned long long *hist, K *pord,
                                                uint32_t *pid, long long *base,
                                                const long long *W, long long *wstar) {
  constexpr int OB = sizeof(K);
  const int lane = threadIdx.x & 63;
  const int t = (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (t >= ntgt) return;   // wave-uniform
  const int s = t / (p - 1);
  const long long jW = (long long)(t % (p - 1) + 1) * W[s];
  unsigned long long *row = hist + (int64_t)t * 256 + 4 * lane;
  long long v[4], local = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    v[u] = (long long)row[u];
    row[u] = 0;
    local += v[u];
  }
  long long incl = local;
  for (int off = 1; off < 64; off <<= 1) {
    const long long y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  long long cum = base[t] + (incl - local);
  int pick = -1;
  long long hb = 0, at = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (pick < 0) {
      if (v[u] > 0 && (long long)p * (cum + v[u]) >= jW) {
        pick = 4 * lane + u;
        hb = v[u];
        at = cum;
      } else {
        cum += v[u];
      }
    }
  }
  const unsigned long long mask = __ballot(pick >= 0);
  if (mask == 0ull) return;   // empty section
  const int first = __ffsll((long long)mask) - 1;
  const int chosen = __shfl(pick, first);
  hb = __shfl(hb, first);
  at = __shfl(at, first);
  if (lane == 0) {
    base[t] = at;
    if (d < OB) pord[t] |= (K)chosen << (8 * (OB - 1 - d));
    else pid[t] |= (uint32_t)chosen << (8 * (3 - (d - OB)));
    if (d == nd - 1) wstar[t] = hb;
  }
}

// Per target: include e* or not; lo[t] = weight of the prefix before the cut.
__global__ void k_finish_targets(int ntgt, int p, const long long *base, const long long *W,
                                 const long long *wstar, int *incl, long long *lo) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ntgt) return;
  const int s = t / (p - 1);
  const long long Ws = W[s], b = base[t], ws = wstar[t];
  const long long jW = (long long)(t % (p - 1) + 1) * Ws;
  int inc = 0;
  if (Ws > 0) inc = ((long long)p * (b + ws) - jW) < (jW - (long long)p * b) ? 1 : 0;
  incl[t] = inc;
  lo[t] = Ws > 0 ? b + (inc ? ws : 0) : 0;
}

// Per section: the weights of its p children.
__global__ void k_finish_sections(int nsec, int p, const long long *lo, const long long *W,
                                  long long *Wnext) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nsec) return;
  long long prev = 0;
  for (int c = 0; c < p; ++c) {
    const long long cur = c < p - 1 ? lo[s * (p - 1) + c] : W[s];
    Wnext[(int64_t)s * p + c] = cur - prev;
    prev = cur;
  }
}

// child = number of cuts of the member's section that it lies after
template <typename K>
__global__ void k_assign(int64_t n, const K *keys, int32_t *part, int p, const K *pord,
                         const uint32_t *pid, const int *incl, const long long *W) {
  const int pm = p - 1;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int s = part[i];
    const K o = keys[i];
    const uint32_t id = (uint32_t)i;
    int child = 0;
    if (W[s] != 0)
      for (int j = 0; j < pm; ++j) {
        const int t = s * pm + j;
        const K po = pord[t];
        const uint32_t pi = pid[t];
        bool low;
        if (o != po) low = o < po;
        else if (id != pi) low = id < pi;
        else low = incl[t] != 0;
        child += low ? 0 : 1;
      }
    part[i] = s * p + child;
  }
}

template <typename K>
__global__ void k_reset(int nsec, K *pord, uint32_t *pid, long long *base) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nsec) { pord[s] = 0; pid[s] = 0; base[s] = 0; }
}

__global__ __launch_bounds__(256) void k_wsum(int64_t n, const int32_t *vwgt, long long *out) {
  long long acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    acc += vwgt ? vwgt[i] : 1;
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) atomicAdd((unsigned long long *)out, (unsigned long long)acc);
}

__global__ __launch_bounds__(256) void k_split_clear(unsigned long long *hist, int *flag) {
  for (int q = threadIdx.x; q < 2048; q += 256) hist[q] = 0ull;
  if (threadIdx.x < 4) flag[threadIdx.x] = 0;
}

__global__ __launch_bounds__(256) void k_zero_parts(int64_t n, int32_t *part) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    part[i] = 0;
}

// ---- sample bins
constexpr int kSample = 2048;         // sorted sample keys per coordinate
constexpr int kBins = 2048;           // bins of a level over all its sections
constexpr int kFastSections = 256;
constexpr int kFastCuts = 63;         // cuts per section
constexpr int kFastTargets = 4096;
constexpr int kFastLds = 4096;        // candidates kept in LDS
constexpr int kFastCap = 65536;       // candidates per target (see fast_cap)
constexpr int kCutThreads = 1024;
// Candidates of a target are appended through kSub counters, a cache line
// each, to kSub runs of its list: appends to one counter go one after the
// other at about 0.2 us (with one counter per target the pass over 2 M members
// took 218 us).  A block has its run, so that neighbouring members share lines
// of the list (runs chosen by a hash of the id: 14.5 instead of 9.4 us); a full
// run passes the member on to the next, so that the whole list is a target's
// room wherever its members lie (without that, lattices in natural order, whose
// late sections lie in few blocks, ran into the radix passes: 16,000 vertices,
// K = 256, FP32 910 us, now 289).
constexpr int kSub = 32;
constexpr int kSubStride = 16;
enum : int { F_NAN = 1, F_CROWDED = 2 };

// splitmix64 (Steele, Lea, Flood 2014)
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

template <typename K>
__device__ __forceinline__ bool before(K ao, uint32_t ai, K bo, uint32_t bi) {
  return (ao < bo) | ((ao == bo) & (ai < bi));
}

// Sorted composite keys of kSample random members, one block per coordinate
// (a bitonic sort in LDS).  Random positions: a fixed stride meets one plane
// of a lattice only.
template <typename T>
__global__ __launch_bounds__(1024) void k_sample(const T *coords, int ld, int64_t n,
                                                 typename Ord<T>::K *sord, uint32_t *sid) {
  using K = typename Ord<T>::K;
  __shared__ K o[kSample];
  __shared__ uint32_t id[kSample];
  const int c = blockIdx.x, t = threadIdx.x;
  for (int q = t; q < kSample; q += 1024) {
    const int64_t i = (int64_t)(mix64((uint64_t)q * 977 + c) % (uint64_t)n);
    bool nan = false;
    o[q] = Ord<T>::map(coords[i * ld + c], nan);
    id[q] = (uint32_t)i;
  }
  // pairs up to 64 apart lie within the 128 values of one wave, whose LDS
  // operations are in order: only wider steps need the block's barrier
  bool wide = true;
  for (int w = 2; w <= kSample; w <<= 1)
    for (int j = w >> 1; j >= 1; j >>= 1) {
      if (wide || j > 64) __syncthreads();
      else wave_order();
      wide = j > 64;
      const int a = 2 * t - (t & (j - 1)), b = a + j;   // pairs j apart
      const bool up = (a & w) == 0;
      const K oa = o[a], ob = o[b];
      const uint32_t ia = id[a], ib = id[b];
      if (before(ob, ib, oa, ia) == up) {
        o[a] = ob;
        id[a] = ib;
        o[b] = oa;
        id[b] = ia;
      }
    }
  __syncthreads();
  for (int q = t; q < kSample; q += 1024) {
    sord[(int64_t)c * kSample + q] = o[q];
    sid[(int64_t)c * kSample + q] = id[q];
  }
}

// Targets of a level: cut keys (ord, id), whether the member at the key is
// before the cut, and the weight before the cut.
template <typename K>
struct Cuts {
  int p;             // children per section (0: no level before)
  K *ord;
  uint32_t *id;
  int *incl;
  long long *lo;
  long long *W;      // weights of the level's sections
};

// One pass over the members: the child of the level before (if any), the key
// of this level's coordinate, its bin, and the sections' bin weights (in LDS
// first).  Bound by the strided reads of the coordinate column (a row of the
// block per member).  H: LDS counter type (unsigned for unit weights).
template <typename T, typename H>
__global__ __launch_bounds__(512) void k_level(const T *__restrict__ coords, int ld, int c,
                                               int64_t n, typename Ord<T>::K *keys,
                                               uint16_t *bins, int32_t *part,
                                               const int32_t *__restrict__ vwgt,
                                               Cuts<typename Ord<T>::K> prev, int first,
                                               const typename Ord<T>::K *__restrict__ sord,
                                               const uint32_t *__restrict__ sid, int B, int nsec,
                                               unsigned long long *hist, int *flag) {
  using K = typename Ord<T>::K;
  __shared__ K so[kSample];
  __shared__ uint32_t si[kSample];
  __shared__ H h[kBins];
  for (int q = threadIdx.x; q < B - 1; q += 512) {
    const int at = (int)((int64_t)(q + 1) * kSample / B);
    so[q] = sord[at];
    si[q] = sid[at];
  }
  for (int q = threadIdx.x; q < B * nsec; q += 512) h[q] = 0;
  __syncthreads();
  bool nan = false;
  for (int64_t i = (int64_t)blockIdx.x * 512 + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * 512) {
    const uint32_t id = (uint32_t)i;
    const K o = Ord<T>::map(coords[i * ld + c], nan);
    int s = 0;
    if (prev.p) {
      const int s0 = first ? 0 : part[i];
      const K ko = keys[i];
      const int pm = prev.p - 1;
      int child = 0;
      for (int j = 0; j < pm; ++j) {
        const int t = s0 * pm + j;
        const K po = prev.ord[t];
        const uint32_t pi = prev.id[t];
        const bool low = before(ko, id, po, pi) | ((ko == po) & (id == pi) & (prev.incl[t] != 0));
        child += low ? 0 : 1;
      }
      s = s0 * prev.p + child;
      part[i] = s;
    }
    keys[i] = o;
    // bin: the number of splitters at or before the member
    int lo = 0, len = B - 1;
    while (len > 0) {
      const int half = len >> 1, mid = lo + half;
      const bool right = !before(o, id, so[mid], si[mid]);
      lo = right ? mid + 1 : lo;
      len = right ? len - half - 1 : half;
    }
    bins[i] = (uint16_t)lo;
    atomicAdd(&h[s * B + lo], (H)(vwgt ? vwgt[i] : 1));
  }
  if (nan) atomicOr(flag, F_NAN);
  __syncthreads();
  for (int q = threadIdx.x; q < B * nsec; q += 512)
    if (h[q]) atomicAdd(&hist[q], (unsigned long long)h[q]);
}

// One block per section: its weight (from the level before), and for each of
// its cuts j the first bin whose end reaches j W / p, with the weight before
// it; clears the section's bins and the cuts' candidate counters.
template <typename K>
__global__ __launch_bounds__(256) void k_find_bins(int B, int p, Cuts<K> prev, long long total,
                                                   unsigned long long *hist, long long *W,
                                                   int *tbin, long long *base, int *cnt) {
  __shared__ long long sh[4];
  const int s = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  long long Ws = total;
  if (prev.p) {
    const int par = s / prev.p, ch = s - par * prev.p;
    const long long *lo = prev.lo + (int64_t)par * (prev.p - 1);
    const long long a = ch ? lo[ch - 1] : 0;
    Ws = (ch < prev.p - 1 ? lo[ch] : prev.W[par]) - a;
  }
  if (t == 0) W[s] = Ws;
  for (int j = t; j < p - 1; j += 256) {
    const int tg = s * (p - 1) + j;
    tbin[tg] = -1;
    base[tg] = 0;
  }
  for (int q = t; q < (p - 1) * kSub; q += 256)
    cnt[((int64_t)s * (p - 1) * kSub + q) * kSubStride] = 0;
  const int per = (B + 255) / 256;
  const int b0 = min(B, t * per), b1 = min(B, b0 + per);
  long long own = 0;
  for (int b = b0; b < b1; ++b) own += (long long)hist[(int64_t)s * B + b];
  long long incl = own;
  for (int off = 1; off < 64; off <<= 1) {
    const long long y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  long long cum = incl - own;
  for (int q = 0; q < wave; ++q) cum += sh[q];
  if (Ws <= 0) return;          // uniform; an empty section's bins are zero
  for (int b = b0; b < b1; ++b) {
    const long long v = (long long)hist[(int64_t)s * B + b];
    hist[(int64_t)s * B + b] = 0;
    if (v > 0) {
      // the cuts j with p cum < j W <= p (cum + v)
      const long long jl = (long long)p * cum / Ws + 1, jh = (long long)p * (cum + v) / Ws;
      for (long long j = jl; j <= jh && j < p; ++j) {
        const int tg = s * (p - 1) + (int)j - 1;
        tbin[tg] = b;
        base[tg] = cum;
      }
    }
    cum += v;
  }
}

// the members of every target's bin (in no particular order); cap: of a run
__global__ __launch_bounds__(256) void k_candidates(int64_t n, const uint16_t *__restrict__ bins,
                                                    const int32_t *__restrict__ part, int first,
                                                    int p, int ntgt, const int *__restrict__ tbin,
                                                    int cap, int *cnt, uint32_t *list,
                                                    int *flag) {
  __shared__ int tb[kFastTargets];
  for (int q = threadIdx.x; q < ntgt; q += 256) tb[q] = tbin[q];
  __syncthreads();
  const int pm = p - 1;
  // appends member i to run `run` of target t, unless it is full
  auto append = [&](int t, unsigned run, uint32_t i) {
    const int64_t r = (int64_t)t * kSub + run;
    const int at = atomicAdd(&cnt[r * kSubStride], 1);
    if (at < cap) list[r * cap + at] = i;
    return at < cap;
  };
  const unsigned own = blockIdx.x & (kSub - 1);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * 256) {
    const int b = bins[i], t0 = (first ? 0 : part[i]) * pm;
    for (int j = 0; j < pm; ++j)
      if (tb[t0 + j] == b && !append(t0 + j, own, (uint32_t)i)) {
        unsigned q = 1;
        for (; q < kSub; ++q) {
          const unsigned run = (own + q) & (kSub - 1);
          const int have =
              __hip_atomic_load(&cnt[((int64_t)(t0 + j) * kSub + run) * kSubStride],
                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (have < cap && append(t0 + j, run, (uint32_t)i)) break;
        }
        if (q == kSub) atomicOr(flag, F_CROWDED);
      }
  }
}

// One block per target: radix select of the cut's member among the bin's
// members, 8 bits at a time of the keys less their minimum, then of the ids
// (a bin is a narrow range of the order, so its raw leading bytes would put
// nearly all members into one or two counters); a bucket with one member ends
// the search.  Then the cut: whether that member is before it, and the weight
// before it.  Measured at 1000 members: 15 us (raw bytes: 19 us).
template <typename K>
__global__ __launch_bounds__(kCutThreads) void k_cut_bin(int64_t n, int p, const K *__restrict__ keys,
                                                  const int32_t *__restrict__ vwgt,
                                                  uint32_t *list, int cap,
                                                  const int *__restrict__ cnt,
                                                  const long long *__restrict__ base_in,
                                                  const int *__restrict__ flag, Cuts<K> out) {
  __shared__ K ck[kFastLds];
  __shared__ uint32_t ci[kFastLds];
  __shared__ unsigned long long h[256];
  __shared__ unsigned hc[256];
  __shared__ int at[kSub + 1];
  __shared__ K pord, pref, kmn[kCutThreads / 64], kmx[kCutThreads / 64];
  __shared__ uint32_t pid, ipref, imn[kCutThreads / 64], imx[kCutThreads / 64];
  __shared__ long long base, hit;
  __shared__ int one;
  const int tg = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int s = tg / (p - 1);
  const int stop = *flag & F_CROWDED;
  const long long Ws = out.W[s];
  const long long jW = (long long)(tg - s * (p - 1) + 1) * Ws;
  // the runs' starts among the target's candidates
  if (t < 64) {
    const int own = t < kSub ? min(cnt[((int64_t)tg * kSub + t) * kSubStride], cap) : 0;
    int incl = own;
    for (int off = 1; off < kSub; off <<= 1) {
      const int y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    if (t < kSub) at[t + 1] = incl;
    if (t == 0) {
      at[0] = 0;
      pord = 0;
      pid = 0;
      pref = 0;
      ipref = 0;
      base = base_in[tg];
      hit = 0;
      one = 0;
    }
  }
  __syncthreads();
  if (stop) return;
  const int c = at[kSub];
  const uint32_t *mine = list + (int64_t)tg * kSub * cap;
  const bool lds = c <= kFastLds;
  auto member = [&](int q) -> uint32_t {       // candidate q: run by bisection
    int lo = 0, hi = kSub - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (at[mid] <= q) lo = mid; else hi = mid - 1;
    }
    return mine[(int64_t)lo * cap + (q - at[lo])];
  };
  K ka = ~K(0), kb = 0;
  uint32_t ia = ~0u, ib = 0;
  for (int q = t; q < c; q += kCutThreads) {
    const uint32_t i = member(q);
    const K o = keys[i];
    if (lds) {
      ci[q] = i;
      ck[q] = o;
    }
    ka = min(ka, o);
    kb = max(kb, o);
    ia = min(ia, i);
    ib = max(ib, i);
  }
  for (int off = 32; off >= 1; off >>= 1) {
    ka = min(ka, (K)__shfl_xor((unsigned long long)ka, off));
    kb = max(kb, (K)__shfl_xor((unsigned long long)kb, off));
    ia = min(ia, (uint32_t)__shfl_xor((int)ia, off));
    ib = max(ib, (uint32_t)__shfl_xor((int)ib, off));
  }
  if (lane == 0) {
    kmn[wave] = ka;
    kmx[wave] = kb;
    imn[wave] = ia;
    imx[wave] = ib;
  }
  __syncthreads();
  for (int q = 0; q < kCutThreads / 64; ++q) {
    ka = min(ka, kmn[q]);
    kb = max(kb, kmx[q]);
    ia = min(ia, imn[q]);
    ib = max(ib, imx[q]);
  }
  // bits left of the keys (less ka), then of the ids (less ia)
  int kbits = c > 0 && kb > ka ? 64 - __clzll((long long)(uint64_t)(kb - ka)) : 0;
  int ibits = c > 0 ? max(1, 32 - __clz((int)(ib - ia))) : 0;
  while (kbits + ibits > 0) {
    const bool on_key = kbits > 0;
    const int w = min(8, on_key ? kbits : ibits);
    const int sh = (on_key ? kbits : ibits) - w;
    if (t < 256) {
      h[t] = 0;
      hc[t] = 0;
    }
    __syncthreads();
    const K kp = pref;
    const uint32_t ip = ipref;
    // bucket of a candidate that matches the prefix, or -1
    auto bucket = [&](K o, uint32_t i) -> int {
      const uint64_t x = on_key ? (uint64_t)(o - ka) : (uint64_t)(i - ia);
      if (!on_key && o - ka != kp) return -1;
      const uint64_t want = on_key ? (uint64_t)kp : (uint64_t)ip;
      // (shifts of w + sh <= 64 in two steps)
      return ((x >> sh) >> w) == want ? (int)((x >> sh) & ((1u << w) - 1)) : -1;
    };
    for (int q = t; q < c; q += kCutThreads) {
      const uint32_t i = lds ? ci[q] : member(q);
      const int b = bucket(lds ? ck[q] : keys[i], i);
      if (b >= 0) {
        atomicAdd(&h[b], (unsigned long long)(vwgt ? vwgt[i] : 1));
        atomicAdd(&hc[b], 1u);
      }
    }
    __syncthreads();
    if (t < 64) {
      // the first bucket where p C reaches j W (as in k_select)
      long long v[4], local = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = (long long)h[4 * lane + u];
        local += v[u];
      }
      long long incl = local;
      for (int off = 1; off < 64; off <<= 1) {
        const long long y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
      }
      long long cum = base + (incl - local);
      int pick = -1;
      long long hb = 0, bb = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (pick < 0) {
          if (v[u] > 0 && (long long)p * (cum + v[u]) >= jW) {
            pick = 4 * lane + u;
            hb = v[u];
            bb = cum;
          } else {
            cum += v[u];
          }
        }
      }
      const unsigned long long mask = __ballot(pick >= 0);
      if (mask) {
        const int first = __ffsll((long long)mask) - 1;
        if (lane == first) {
          base = bb;
          hit = hb;
          one = hc[pick] == 1u;
          if (on_key) pref = (kp << w) | (K)pick;
          else ipref = (ip << w) | (uint32_t)pick;
        }
      }
    }
    __syncthreads();
    (on_key ? kbits : ibits) = sh;
    if (one || kbits + ibits == 0) {           // uniform: the member itself
      const uint64_t kw = pref, iw = ipref;
      for (int q = t; q < c; q += kCutThreads) {
        const uint32_t i = lds ? ci[q] : member(q);
        const K o = lds ? ck[q] : keys[i];
        const bool is = on_key ? ((uint64_t)(o - ka) >> sh) == kw
                               : ((o - ka) == (K)kw) & (((uint64_t)(i - ia) >> sh) == iw);
        if (is) {
          pord = o;
          pid = i;
        }
      }
      __syncthreads();
      break;
    }
  }
  if (t == 0) {
    const long long b = base, ws = hit;
    int inc = 0;
    if (Ws > 0) inc = ((long long)p * (b + ws) - jW) < (jW - (long long)p * b) ? 1 : 0;
    out.ord[tg] = pord;
    out.id[tg] = pid;
    out.incl[tg] = inc;
    out.lo[tg] = Ws > 0 ? b + (inc ? ws : 0) : 0;
  }
}

}  // namespace

std::vector<int> section_counts(int K) {
  std::vector<int> f;
  int k = K;
  for (int q = 2; (int64_t)q * q <= k; ++q)
    while (k % q == 0) {
      f.push_back(q);
      k /= q;
    }
  if (k > 1) f.push_back(k);
  std::sort(f.begin(), f.end(), [](int a, int b) { return a > b; });
  return f;
}

// Candidates per run (kSub of them per target) of a level with ntgt targets:
// in all at most 4 n + 256 ntgt, and per target at most kFastCap or 32 average
// bins (a bin lies between two neighbours of the sorted sample, so its size
// varies like an exponential variable's: 16 times the average once in 10^6).
static int fast_cap(int64_t n, int ntgt) {
  const int64_t most = std::max<int64_t>(kFastCap, n / kBins * 32);
  return (int)(std::min<int64_t>(most, std::max<int64_t>(256, 4 * n / ntgt)) / kSub);
}

// Every level of K within the sample bins' limits (n = 0), and with n members
// in ncoord coordinates worth them: a section that earlier levels have cut r-fold
// along the level's coordinate lies in one r-th of the coordinate's bins, so a
// target's bin holds about n r / kBins members (at most the section), which one
// workgroup goes over.  Measured against the radix passes (FP32, with r up to
// 32 and 8 M members in one coordinate 5.8 instead of 2.8 ms, with r up to 8 and
// 32 M 6.2 instead of 4.3; in two coordinates, r up to 8, 64 M members into 256
// parts 23 instead of 45 ms): beyond kFastCap / 2 members it loses from r = 8 on
// where the radix passes count in LDS, and from some r above 9 where they count
// in memory.
static bool fast_levels(const std::vector<int> &counts, int64_t n = 0, int ncoord = 1) {
  int64_t nsec = 1;
  std::vector<int64_t> cut(counts.size(), 1);   // r per coordinate in use
  for (size_t l = 0; l < counts.size(); ++l) {
    const int p = counts[l];
    const int64_t ntgt = nsec * (p - 1);
    if (nsec > kFastSections || p - 1 > kFastCuts || ntgt > kFastTargets) return false;
    int64_t &r = cut[l % (size_t)ncoord];
    if (std::min(n / kBins * r, n / nsec) > kFastCap / 2 && r > (ntgt <= kLdsTargets ? 4 : 9))
      return false;
    r *= p;
    nsec *= p;
  }
  return !counts.empty();
}

// of the radix passes: targets of a level (nsec * (p - 1)), sections and
// children all fit in K
static size_t radix_bytes(int64_t n, int64_t ns) {
  size_t b = 0;
  b += align_up(sizeof(uint64_t) * n, 256);                 // keys
  b += align_up(sizeof(unsigned long long) * ns * 256, 256); // hist (one row per target)
  b += align_up(sizeof(uint64_t) * ns, 256);                // pord
  b += align_up(sizeof(uint32_t) * ns, 256);                // pid
  b += align_up(sizeof(long long) * ns, 256) * 4;           // base, wstar, W, lo
  b += align_up(sizeof(long long) * ns, 256);               // Wnext
  b += align_up(sizeof(int) * ns, 256);                     // incl
  return b + 1024;
}

// of the sample bins
static size_t bins_bytes(int64_t n, int64_t ns) {
  size_t f = 0;
  f += align_up(sizeof(uint64_t) * n, 256);               // keys
  f += align_up(sizeof(uint16_t) * n, 256);               // bins
  f += align_up(sizeof(uint32_t) * (4 * n + 256 * ns), 256);   // candidates
  f += align_up(sizeof(unsigned long long) * kBins, 256);
  f += align_up(sizeof(uint64_t) * kSample * 64, 256) +   // samples: a coordinate per level
       align_up(sizeof(uint32_t) * kSample * 64, 256);
  f += 2 * (align_up(sizeof(uint64_t) * ns, 256) * 3 + align_up(sizeof(int) * ns, 256) * 2);
  f += align_up(sizeof(int) * ns, 256) + align_up(sizeof(long long) * ns, 256) +
       align_up(sizeof(int) * ns * kSub * kSubStride, 256);
  return f + 1024;
}

size_t split_scratch_bytes(int64_t n, int K) {
  const int ns = K < 1 ? 1 : K;
  const size_t b = radix_bytes(n, ns);
  return fast_levels(section_counts(ns)) ? std::max(b, bins_bytes(n, ns)) : b;
}

// Both parts grow with K, but the sample bins' is only there for some K: for at
// most kFastSections * p parts with kFastSections * (p - 1) <= kFastTargets.
// (Callers ask for sizes before every call, so the factors of the K between
// are not looked at: a bound.)
size_t split_scratch_max(int64_t n, int klo, int khi) {
  const int kf = std::min(khi, kFastTargets + kFastSections);
  return std::max(radix_bytes(n, khi), kf >= klo ? bins_bytes(n, kf) : 0);
}

// The levels by sample bins.  *flags: F_NAN, F_CROWDED (part is then not
// usable).
template <typename T>
static int split_levels(sphx_graph *g, const T *coords, int ld, int ncoord, int K,
                        const std::vector<int> &counts, int32_t *part, void *scratch,
                        void *pinned, hipStream_t s, std::string *err, int *flags) {
  using KT = typename Ord<T>::K;
  const int64_t n = g->n;
  const int nlev = (int)counts.size();
  const int nc = std::min(ncoord, nlev);      // coordinates in use
  Arena a;
  a.base = static_cast<char *>(scratch);
  KT *keys = a.take<KT>(n);
  uint16_t *bins = a.take<uint16_t>(n);
  uint32_t *list = a.take<uint32_t>(4 * n + 256 * (int64_t)K);
  unsigned long long *hist = a.take<unsigned long long>(kBins);
  KT *sord = a.take<KT>(kSample * 64);
  uint32_t *sid = a.take<uint32_t>(kSample * 64);
  Cuts<KT> cut[2];
  for (auto &x : cut) {
    x.p = 0;
    x.ord = a.take<KT>(K);
    x.lo = a.take<long long>(K);
    x.W = a.take<long long>(K);
    x.id = a.take<uint32_t>(K);
    x.incl = a.take<int>(K);
  }
  int *tbin = a.take<int>(K);
  int *cnt = a.take<int>((int64_t)K * kSub * kSubStride);
  long long *base = a.take<long long>(K);
  int *flag = a.take<int>(4);
  long long *total = reinterpret_cast<long long *>(flag + 2);
  int *fh = static_cast<int *>(pinned);
  hipLaunchKernelGGL(k_split_clear, dim3(1), dim3(256), 0, s, hist, flag);
  long long W = n;
  if (g->vwgt) {
    hipLaunchKernelGGL(k_wsum, dim3(grid_for(n, 256 * 8, 1024)), dim3(256), 0, s, n, g->vwgt,
                       total);
    if (hipMemcpyAsync(fh + 2, total, sizeof(long long), hipMemcpyDeviceToHost, s) !=
            hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
      *err = "split: stream error";
      return SPHX_E_HIP;
    }
    std::memcpy(&W, fh + 2, sizeof(W));
  }
  hipLaunchKernelGGL((k_sample<T>), dim3(nc), dim3(1024), 0, s, coords, ld, n, sord, sid);
  const unsigned gl = grid_for(n, 512 * 8, 512), gn = grid_for(n, 256 * 4, 2048);
  int nsec = 1;
  for (int l = 0; l < nlev; ++l) {
    const int p = counts[l], ntgt = nsec * (p - 1), c = l % ncoord;
    int B = kBins;
    while (B * nsec > kBins) B >>= 1;
    const Cuts<KT> &prev = cut[(l + 1) & 1];
    Cuts<KT> &now = cut[l & 1];
    const int cap = fast_cap(n, ntgt);
    const KT *so = sord + (int64_t)c * kSample;
    const uint32_t *si = sid + (int64_t)c * kSample;
    if (g->vwgt)
      hipLaunchKernelGGL((k_level<T, unsigned long long>), dim3(gl), dim3(512), 0, s, coords, ld,
                         c, n, keys, bins, part, g->vwgt, prev, l == 1 ? 1 : 0, so, si, B, nsec,
                         hist, flag);
    else
      hipLaunchKernelGGL((k_level<T, unsigned>), dim3(gl), dim3(512), 0, s, coords, ld, c, n,
                         keys, bins, part, g->vwgt, prev, l == 1 ? 1 : 0, so, si, B, nsec, hist,
                         flag);
    hipLaunchKernelGGL((k_find_bins<KT>), dim3(nsec), dim3(256), 0, s, B, p, prev, W, hist,
                       now.W, tbin, base, cnt);
    hipLaunchKernelGGL(k_candidates, dim3(gn), dim3(256), 0, s, n, (const uint16_t *)bins,
                       (const int32_t *)part, l == 0 ? 1 : 0, p, ntgt, (const int *)tbin, cap,
                       cnt, list, flag);
    now.p = p;
    hipLaunchKernelGGL((k_cut_bin<KT>), dim3(ntgt), dim3(kCutThreads), 0, s, n, p, (const KT *)keys,
                       g->vwgt, list, cap, (const int *)cnt,
                       (const long long *)base, (const int *)flag, now);
    nsec *= p;
  }
  const Cuts<KT> &z = cut[(nlev - 1) & 1];
  if (nlev == 1) hipLaunchKernelGGL(k_zero_parts, dim3(gn), dim3(256), 0, s, n, part);
  hipLaunchKernelGGL((k_assign<KT>), dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, n, keys,
                     part, z.p, z.ord, z.id, z.incl, z.W);
  if (hipGetLastError() != hipSuccess) {
    *err = "split kernel launch failed";
    return SPHX_E_HIP;
  }
  if (hipMemcpyAsync(fh, flag, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    *err = "split: stream error";
    return SPHX_E_HIP;
  }
  *flags = *fh;
  return SPHX_OK;
}

template <typename T>
int split_mj(sphx_graph *g, const T *coords, int ld, int ncoord, int K, int32_t *part,
             void *scratch, void *pinned, hipStream_t s, std::string *err) {
  using KT = typename Ord<T>::K;
  const int64_t n = g->n;
  const std::vector<int> counts = section_counts(K);
  if (fast_levels(counts, n, ncoord)) {
    int flags = 0;
    const int r = split_levels<T>(g, coords, ld, ncoord, K, counts, part, scratch, pinned, s,
                                  err, &flags);
    if (r != SPHX_OK) return r;
    if (flags & F_NAN) {
      *err = "NaN coordinate";
      return SPHX_E_INVALID_ARG;
    }
    if (!(flags & F_CROWDED)) return SPHX_OK;
  }
  // radix passes over all members
  Arena a;
  a.base = static_cast<char *>(scratch);
  a.cap = split_scratch_bytes(n, K);
  KT *keys = a.take<KT>(n);
  unsigned long long *hist = a.take<unsigned long long>((size_t)K * 256);
  KT *pord = a.take<KT>(K);
  uint32_t *pid = a.take<uint32_t>(K);
  long long *base = a.take<long long>(K);
  long long *wstar = a.take<long long>(K);
  long long *W = a.take<long long>(K);
  long long *lo = a.take<long long>(K);
  long long *Wnext = a.take<long long>(K);
  int *incl = a.take<int>(K);
  int *flag = a.take<int>(4);
  bool ok = hipMemsetAsync(part, 0, sizeof(int32_t) * n, s) == hipSuccess;
  ok &= hipMemsetAsync(hist, 0, sizeof(unsigned long long) * (size_t)K * 256, s) == hipSuccess;
  ok &= hipMemsetAsync(W, 0, sizeof(long long) * K, s) == hipSuccess;
  ok &= hipMemsetAsync(flag, 0, sizeof(int) * 4, s) == hipSuccess;
  hipLaunchKernelGGL(k_wsum, dim3(grid_for(n, 256, 1024)), dim3(256), 0, s, n, g->vwgt, W);
  const int nd = (int)sizeof(KT) + 4;
  const unsigned gn = grid_for(n, 256, 4096);
  int nsec = 1;
  for (size_t l = 0; l < counts.size(); ++l) {
    const int p = counts[l];
    const int ntgt = nsec * (p - 1);
    const int c = (int)(l % (size_t)ncoord);
    const unsigned gt = grid_for(ntgt, 256, 1 << 16);
    const unsigned gw = (unsigned)ceil_div(ntgt, 4);   // one wavefront per target
    hipLaunchKernelGGL((k_keys<T>), dim3(gn), dim3(256), 0, s, coords, ld, c, n, keys, flag);
    hipLaunchKernelGGL((k_reset<KT>), dim3(gt), dim3(256), 0, s, ntgt, pord, pid, base);
    for (int d = 0; d < nd; ++d) {
      if (ntgt <= 16)
        hipLaunchKernelGGL((k_hist<KT, 16>), dim3(gn), dim3(256), 0, s, n, keys, part,
                           g->vwgt, d, p, ntgt, pord, pid, hist);
      else if (ntgt <= kLdsTargets)
        hipLaunchKernelGGL((k_hist<KT, kLdsTargets>), dim3(gn), dim3(256), 0, s, n, keys, part,
                           g->vwgt, d, p, ntgt, pord, pid, hist);
      else
        hipLaunchKernelGGL((k_hist<KT, 0>), dim3(gn), dim3(256), 0, s, n, keys, part,
                           g->vwgt, d, p, ntgt, pord, pid, hist);
      hipLaunchKernelGGL((k_select<KT>), dim3(gw), dim3(256), 0, s, ntgt, p, d, nd, hist, pord,
                         pid, base, W, wstar);
    }
    hipLaunchKernelGGL(k_finish_targets, dim3(gt), dim3(256), 0, s, ntgt, p, base, W, wstar,
                       incl, lo);
    hipLaunchKernelGGL(k_finish_sections, dim3(grid_for(nsec, 256, 1 << 16)), dim3(256), 0, s,
                       nsec, p, lo, W, Wnext);
    hipLaunchKernelGGL((k_assign<KT>), dim3(gn), dim3(256), 0, s, n, keys, part, p, pord, pid,
                       incl, W);
    nsec *= p;
    ok &= hipMemcpyAsync(W, Wnext, sizeof(long long) * nsec, hipMemcpyDeviceToDevice, s) ==
          hipSuccess;
  }
  if (!ok || hipGetLastError() != hipSuccess) {
    *err = "split kernel launch failed";
    return SPHX_E_HIP;
  }
  int *fh = static_cast<int *>(pinned);
  if (hipMemcpyAsync(fh, flag, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    *err = "split: stream error";
    return SPHX_E_HIP;
  }
  if (*fh) {
    *err = "NaN coordinate";
    return SPHX_E_INVALID_ARG;
  }
  return SPHX_OK;
}

template int split_mj<float>(sphx_graph *, const float *, int, int, int, int32_t *, void *,
                             void *, hipStream_t, std::string *);
template int split_mj<double>(sphx_graph *, const double *, int, int, int, int32_t *, void *,
                              void *, hipStream_t, std::string *);

}  // namespace sphx
