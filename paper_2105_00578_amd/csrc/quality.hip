// Partition quality (Sec. 3.1): cutsize of Eq. 1, part weights W_k and the
// imbalance max_k W_k / W_avg.
//
// Exactness: unit weights are counted in int64.  Float edge weights are
// summed exactly in 128-bit fixed point: with e0 the exponent of the last
// mantissa bit of the smallest weight, every weight is an integer multiple of
// 2^e0, so the cut is an exact integer times 2^e0, rounded once at the end.
#include <cmath>

#include "fixed.h"
#include "kernels.h"

namespace sphx {
namespace {

// Each block takes a contiguous run of chunks of kCutChunk CSR entries, and
// each thread 4 consecutive entries of a chunk (one 16-byte load, then the
// parts of the neighbours above the row as independent gathers).  The row of
// a thread's first entry (the largest i with row_ptr[i] <= k) comes from a
// binary search over the chunk's row pointers in LDS, the rows of the others
// by stepping on; the rows' parts are staged beside the pointers.  The block's
// first row is found by all threads together (256-fold narrowing), the next
// chunk's is where this one ended.  Each thread accumulates an exact partial;
// a tree adds them.  What is left is the gathers: 13.7 M random words in 102
// us on R-MAT 20 (27.5 M entries; reading them once takes 25 us), half of what
// the L2 can serve.  One binary search per entry, and one through global
// memory per chunk and end by a single thread, took 205 us there and 190 us on
// a weighted 27-point mesh of 883,200 rows, now 65.  Not kept: 16 or 8 entries
// per thread (127 and 110 us), the next chunk's columns loaded ahead (128 us).
//
// A chunk is served from LDS when the row behind its last is staged too, so
// kCutRows allows one more pass of the block than rows of one entry need: with
// room for kCutChunk rows only, the leaves of a star (16 M of them) were
// searched through memory, call 576 us, now 223.
constexpr int kCutPer = 4;
constexpr int kCutChunk = 256 * kCutPer;
constexpr int kCutRows = kCutChunk + 256;

template <typename IdxT, typename WT>
__global__ __launch_bounds__(256) void k_cut(int64_t n, int64_t nnz, const IdxT *rp,
                                             const int32_t *col, const WT *w,
                                             const int32_t *part, int e0, int64_t cpb,
                                             unsigned long long *out) {
  __shared__ int srp[kCutRows + 1];     // row_ptr - k0 of the chunk's rows, within 0..kCutChunk
  __shared__ int spart[kCutRows];       // and their parts
  __shared__ int64_t next_row;
  __shared__ int wn[4];
  const int tid = threadIdx.x, wave = tid >> 6;
  U128 acc{0, 0};
  const int64_t c0 = (int64_t)blockIdx.x * cpb;
  const int64_t c1 = min((nnz + kCutChunk - 1) / kCutChunk, c0 + cpb);
  // the row of entry k in [lo, n - 1] by the whole block: in each step the
  // threads' probes split the range into 256 parts and the last probe at or
  // below the entry is kept (row_ptr[lo] <= k)
  auto locate = [&](int64_t k, int64_t lo) {
    int64_t hi = n - 1;
    while (lo < hi) {
      const int64_t step = (hi - lo + 256) / 256;
      const int64_t at = lo + (int64_t)(tid + 1) * step;
      const bool below = at <= hi && (int64_t)rp[at] <= k;
      const unsigned long long m = __ballot(below);
      if ((tid & 63) == 0) wn[wave] = __popcll(m);
      __syncthreads();
      const int q = wn[0] + wn[1] + wn[2] + wn[3];   // a prefix of the probes
      __syncthreads();
      lo += (int64_t)q * step;
      hi = min(hi, lo + step - 1);
    }
    return lo;
  };
  int64_t r0 = c0 < c1 ? locate(c0 * kCutChunk, 0) : 0;
  for (int64_t c = c0; c < c1; ++c) {
    const int64_t k0 = c * kCutChunk;
    const int len = (int)min((int64_t)kCutChunk, nnz - k0);
    // row pointers from r0 on until one lies past the chunk
    int rows = 0;                       // rows whose pointer is staged
    bool whole = false;                 // the chunk's last row is among them
    while (rows < kCutRows) {
      const int64_t i = r0 + rows + tid;
      int v = kCutChunk + 1;            // past the end
      if (i <= n - 1) {
        const int64_t x = (int64_t)rp[i] - k0;
        v = x < 0 ? 0 : (x > kCutChunk ? kCutChunk + 1 : (int)x);
      }
      srp[rows + tid] = v;
      spart[rows + tid] = i <= n - 1 ? part[i] : 0;
      const int over = __syncthreads_or(v >= len ? 1 : 0);
      rows += 256;
      if (over) {
        whole = true;
        break;
      }
    }
    const int top = min((int64_t)rows - 1, n - 1 - r0);   // last staged row (less r0)
    auto find = [&](int64_t k) {        // the row of entry k, less r0
      if (whole) {
        int lo = 0, hi = top;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (srp[mid] <= (int)(k - k0)) lo = mid; else hi = mid - 1;
        }
        return (int64_t)lo;
      }
      int64_t lo = 0, hi = n - 1 - r0;  // many empty rows: through memory
      while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if ((int64_t)rp[r0 + mid] <= k) lo = mid; else hi = mid - 1;
      }
      return lo;
    };
    const int b = tid * kCutPer;
    if (b < len) {
      const int cnt = min(kCutPer, len - b);
      const int64_t k = k0 + b;
      typedef int i4 __attribute__((ext_vector_type(4), aligned(4)));
      int j[kCutPer], pi[kCutPer], pj[kCutPer];
      if (cnt == kCutPer) {
#pragma unroll
        for (int q = 0; q < kCutPer; q += 4) {
          const i4 v = *reinterpret_cast<const i4 *>(col + k + q);
          j[q] = v[0];
          j[q + 1] = v[1];
          j[q + 2] = v[2];
          j[q + 3] = v[3];
        }
      } else {
#pragma unroll
        for (int q = 0; q < kCutPer; ++q) j[q] = q < cnt ? col[k + q] : 0;
      }
      // the entries' rows, stepping through LDS; j = -1 where j <= i
      int64_t i = r0;
      if (whole) {
        int r = (int)find(k);
        int end = srp[r + 1];
#pragma unroll
        for (int q = 0; q < kCutPer; ++q) {
          if (q < cnt && b + q >= end) {  // the next row, or past empty ones
            ++r;
            end = srp[r + 1];
            if (b + q >= end) {
              r = (int)find(k + q);
              end = srp[r + 1];
            }
          }
          pi[q] = spart[r];
          j[q] = q < cnt && (int64_t)j[q] > r0 + r ? j[q] : -1;
        }
        i += r;
      } else {
#pragma unroll
        for (int q = 0; q < kCutPer; ++q) {
          if (q < cnt) i = r0 + find(k + q);
          pi[q] = part[i];
          j[q] = q < cnt && (int64_t)j[q] > i ? j[q] : -1;
        }
      }
#pragma unroll
      for (int q = 0; q < kCutPer; ++q) pj[q] = j[q] >= 0 ? part[j[q]] : pi[q];
      if constexpr (std::is_same_v<WT, Unit>) {
        int cuts = 0;
#pragma unroll
        for (int q = 0; q < kCutPer; ++q) cuts += pj[q] != pi[q] ? 1 : 0;
        add128(acc, (unsigned long long)cuts, 0ull);
      } else {
        WT x[kCutPer];
#pragma unroll
        for (int q = 0; q < kCutPer; ++q) x[q] = pj[q] != pi[q] ? w[k + q] : WT(0);
#pragma unroll
        for (int q = 0; q < kCutPer; ++q)
          if (pj[q] != pi[q]) {
            unsigned long long l, h;
            fixed_of(x[q], e0, l, h);
            add128(acc, l, h);
          }
      }
      // the thread with the chunk's last entry holds the last row
      if (b + cnt == len) next_row = i;
    }
    __syncthreads();
    if (c + 1 < c1) {
      r0 = next_row;
      const int64_t kn = k0 + kCutChunk;
      if ((int64_t)rp[r0 + 1] <= kn) {  // it ended with the chunk: the next row, or past
        ++r0;                           // empty ones (the same in every thread)
        if ((int64_t)rp[r0 + 1] <= kn) r0 = locate(kn, r0);
      }
    }
    __syncthreads();   // srp and next_row are rewritten for the next chunk
  }
  __shared__ unsigned long long slo[256], shi[256];
  slo[tid] = acc.lo;
  shi[tid] = acc.hi;
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if (tid < h) {
      U128 t{slo[tid], shi[tid]};
      add128(t, slo[tid + h], shi[tid + h]);
      slo[tid] = t.lo;
      shi[tid] = t.hi;
    }
    __syncthreads();
  }
  if (tid == 0) {
    out[2 * blockIdx.x] = slo[0];
    out[2 * blockIdx.x + 1] = shi[0];
  }
}

// Part weights: integer sums, so the order of the additions does not matter.
// Up to kLdsParts parts are counted in LDS first (no global contention).
constexpr int kLdsParts = 4096;

__global__ __launch_bounds__(256) void k_part_weights(int64_t n, const int32_t *part,
                                                      const int32_t *vwgt, int K,
                                                      unsigned long long *pw, int *bad) {
  __shared__ unsigned long long h[kLdsParts];
  const bool lds = K <= kLdsParts;
  if (lds) {
    for (int k = threadIdx.x; k < K; k += blockDim.x) h[k] = 0;
    __syncthreads();
  }
  int f = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    int p = part[i];
    if (p < 0 || p >= K) { f = 1; continue; }
    unsigned long long wt = (unsigned long long)(vwgt ? vwgt[i] : 1);
    if (lds) atomicAdd(&h[p], wt);
    else atomicAdd(&pw[p], wt);
  }
  if (f) atomicOr(bad, 1);
  if (lds) {
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += blockDim.x)
      if (h[k]) atomicAdd(&pw[k], h[k]);
  }
}

constexpr int kCutBlocks = 2048;

// Clears n 64-bit words (a kernel rather than a memset node, so that the
// clearing is an ordinary launch on the stream).
__global__ __launch_bounds__(256) void k_zero_u64(unsigned long long *p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0ull;
}

double u128_to_double(unsigned __int128 v) {
  if (v == 0) return 0.0;
  int nb = 0;
  for (unsigned __int128 t = v; t; t >>= 1) ++nb;
  if (nb <= 53) return (double)(unsigned long long)v;
  int sh = nb - 53;
  unsigned __int128 top = v >> sh;
  unsigned __int128 rem = v - (top << sh);
  unsigned __int128 half = (unsigned __int128)1 << (sh - 1);
  if (rem > half || (rem == half && (top & 1))) top += 1;   // nearest, ties to even
  return std::ldexp((double)(unsigned long long)top, sh);
}

}  // namespace

size_t quality_scratch_bytes(int K) {
  return align_up(sizeof(unsigned long long) * 2 * kCutBlocks, 256) +
         align_up(sizeof(unsigned long long) * (size_t)(K > 0 ? K : 1), 256) + 1024;
}

int quality(sphx_graph *g, const int32_t *part, int K, double *cut, double *imbalance,
            int64_t *part_weights, void *scratch, void *pinned, hipStream_t s,
            std::string *err, unsigned __int128 *cut_fixed) {
  Arena a;
  a.base = static_cast<char *>(scratch);
  unsigned long long *cp = a.take<unsigned long long>(2 * kCutBlocks);
  unsigned long long *pw = a.take<unsigned long long>(K);
  // the bad-part flag shares the zeroed region: one 64-bit word after pw
  unsigned long long *bad = a.take<unsigned long long>(1);
  // the weight range (and its e0) is known from the degree pass
  int e0 = 0;
  if (g->wdt == SPHX_F32) e0 = fixed_exponent<float>(g->wmin);
  if (g->wdt == SPHX_F64) e0 = fixed_exponent<double>(g->wmin);
  const int64_t nz = (int64_t)(reinterpret_cast<char *>(bad + 1) -
                               reinterpret_cast<char *>(pw)) / 8;
  hipLaunchKernelGGL(k_zero_u64, dim3(grid_for(nz, 256, 1024)), dim3(256), 0, s, pw, nz);
  hipLaunchKernelGGL(k_part_weights, dim3(grid_for(g->n, 256 * 16, 1024)), dim3(256), 0, s,
                     g->n, part, g->vwgt, K, pw, reinterpret_cast<int *>(bad));
  const int64_t chunks = ceil_div(g->nnz, kCutChunk);
  const int64_t cpb = std::max<int64_t>(1, ceil_div(chunks, kCutBlocks));
  const unsigned nb = (unsigned)std::max<int64_t>(1, ceil_div(chunks, cpb));
  auto go = [&](auto it, auto wt) {
    using IdxT = decltype(it);
    using WT = decltype(wt);
    hipLaunchKernelGGL((k_cut<IdxT, WT>), dim3(nb), dim3(256), 0, s, g->n, g->nnz,
                       (const IdxT *)g->rowptr, g->col, (const WT *)g->w, part, e0, cpb, cp);
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
  if (hipGetLastError() != hipSuccess) {
    *err = "quality kernel launch failed";
    return SPHX_E_HIP;
  }
  // results come back through the pinned host buffer (kQualityPinnedWords
  // 64-bit words), so no host memory is allocated here: cut partials, part
  // weights and flag in one copy where they fit, else the part weights follow
  // in chunks
  unsigned long long *hb = static_cast<unsigned long long *>(pinned);
  const int64_t words = (bad + 1) - cp;
  const bool at_once = words <= kQualityPinnedWords;
  auto copy = [&](unsigned long long *to, const unsigned long long *from, int64_t cnt) {
    return hipMemcpyAsync(to, from, sizeof(unsigned long long) * cnt, hipMemcpyDeviceToHost, s) ==
           hipSuccess;
  };
  bool ok = at_once ? copy(hb, cp, words)
                    : copy(hb, cp, 2 * nb) && copy(hb + 2 * kCutBlocks, bad, 1);
  if (!ok || hipStreamSynchronize(s) != hipSuccess) {
    *err = "quality: copy failed";
    return SPHX_E_HIP;
  }
  if (hb[at_once ? words - 1 : 2 * kCutBlocks]) {
    *err = "part id out of range [0, K)";
    return SPHX_E_INVALID_ARG;
  }
  unsigned __int128 tot = 0;
  for (unsigned b = 0; b < nb; ++b)
    tot += ((unsigned __int128)hb[2 * b + 1] << 64) + hb[2 * b];
  if (cut_fixed) *cut_fixed = tot;
  double c = u128_to_double(tot);
  if (g->wdt != SPHX_UNIT) c = std::ldexp(c, e0);
  if (cut) *cut = c;
  unsigned long long mx = 0, sum = 0;
  auto weights = [&](const unsigned long long *v, int k0, int cnt) {
    for (int k = 0; k < cnt; ++k) {
      mx = std::max(mx, v[k]);
      sum += v[k];
      if (part_weights) part_weights[k0 + k] = (int64_t)v[k];
    }
  };
  if (at_once) {
    weights(hb + (pw - cp), 0, K);
  } else {
    for (int k0 = 0; k0 < K; k0 += kQualityPinnedWords) {
      const int cnt = std::min(K - k0, kQualityPinnedWords);
      if (!copy(hb, pw + k0, cnt) || hipStreamSynchronize(s) != hipSuccess) {
        *err = "quality: copy failed";
        return SPHX_E_HIP;
      }
      weights(hb, k0, cnt);
    }
  }
  if (imbalance) *imbalance = sum ? (double)(mx * (unsigned long long)K) / (double)sum : 1.0;
  return SPHX_OK;
}

}  // namespace sphx
