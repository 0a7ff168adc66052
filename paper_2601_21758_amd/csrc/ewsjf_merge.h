// Exact selection over candidates in one workgroup's LDS and registers: the
// building blocks of the merge kernels, of the pools one workgroup answers and
// of Algorithm 1's batch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ewsjf_device.h"

namespace ewsjf {

struct MergeShared {
  uint64_t X[kMergeCap];
  uint64_t S[kSortMax];
  uint32_t cnt[4096];
  uint64_t red[kWavesPerBlock];
  uint64_t wmax[kWavesPerBlock];
  uint64_t wmin[kWavesPerBlock];
  uint64_t wbound[kWavesPerBlock];  // largest completeness bound of each wave's shares
  int iscan[kWavesPerBlock];
  int wtot[kWavesPerBlock];
  int cntX;
  int cntS;
  int cut_bin;
  int cut_cnt;
};

// Exact top-B of the nonzero entries of X[0..U) (distinct composites; when
// U <= max(B, kSortMax) every entry must be nonzero), sorted descending into
// X[0..min(U, B)).  Returns the number selected.  More than kSortMax of them:
// the candidates at or above a histogram cut (between B and kSortMax) are
// gathered first.  The set is then ordered by a counting sort.
__device__ inline int select_top(MergeShared& ms, int U, int B) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  if (U == 0) return 0;
  const uint64_t* src = ms.X;
  int nS = U;
  if (U > B && U > kSortMax) {
    const uint64_t cut = find_cut(ms.X, U, B, kSortMax, ms.cnt, ms.iscan, ms.red);
    if (tid == 0) ms.cntS = 0;
    __syncthreads();
    for (int i0 = 0; i0 < U; i0 += kBlock) {
      const int i = i0 + tid;
      const uint64_t x = i < U ? ms.X[i] : 0ull;
      const bool p = x >= cut && x != 0ull;
      const uint64_t bal = __ballot(p);
      if (bal) {
        int b0 = 0;
        if (lane == 0) b0 = atomicAdd(&ms.cntS, __popcll(bal));
        b0 = __shfl(b0, 0);
        const int pos = b0 + __popcll(bal & lanemask_lt());
        if (p && pos < kSortMax) ms.S[pos] = x;
      }
    }
    __syncthreads();
    nS = ms.cntS < kSortMax ? ms.cntS : kSortMax;
    src = ms.S;
  }
  // X is free now: its upper part is the scatter buffer, its head the output.
  bucket_sort_desc(src, nS, ms.X + kSortMax, ms.X, ms.cnt, ms.iscan, ms.red);
  return nS < B ? nS : B;
}

// Exact top-B of the block's entries v (0 = none; entry r of thread tid has the
// place tid + r * kBlock < places <= kMergeCap): sorted descending into
// ms.X[0..U), U = min(B, entries), returned.  A histogram of 4,096 linear
// buckets over the entries' range, the bucket where the count from the top
// reaches B, a scatter of the entries at or above it, and each one's rank
// inside its bucket.  *max_bound = the largest `bound` of the block.
template <int kR>
__device__ __forceinline__ int rank_registers(MergeShared& ms, const uint64_t (&v)[kR], int places, int B,
                                              uint64_t bound, uint64_t* max_bound) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  // Exact range and count (registers -> wave -> LDS) while the histogram is
  // cleared.
  uint64_t mx = 0, mn = ~0ull;
  int nz = 0;
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    mx = v[r] > mx ? v[r] : mx;
    mn = (v[r] != 0ull && v[r] < mn) ? v[r] : mn;
    nz += v[r] != 0ull;
  }
  mx = wave_max_u64(mx);
  mn = wave_min_u64(mn);
  nz = (int)__ockl_wfred_add_u32((uint32_t)nz);
  const uint64_t tb = wave_max_u64(bound);
  for (int i = tid; i < 4096; i += kBlock) ms.cnt[i] = 0u;
  if (lane == 0) {
    ms.wmax[wv] = mx;
    ms.wmin[wv] = mn;
    ms.iscan[wv] = nz;
    ms.wbound[wv] = tb;
  }
  __syncthreads();
  // Every wave reduces the kWavesPerBlock partials itself, one per lane.
  static_assert(kWavesPerBlock <= kWave, "one partial per lane");
  const bool pl = lane < kWavesPerBlock;
  const int total = (int)__ockl_wfred_add_u32(pl ? (uint32_t)ms.iscan[lane] : 0u);
  *max_bound = wave_max_u64(pl ? ms.wbound[lane] : 0ull);
  if (total == 0) return 0;
  const uint64_t hi = wave_max_u64(pl ? ms.wmax[lane] : 0ull);
  const uint64_t lo = wave_min_u64(pl ? ms.wmin[lane] : ~0ull);
  const uint64_t diff = hi - lo;
  const int bits = diff == 0 ? 0 : 64 - __clzll((long long)diff);
  const int shift = bits > 12 ? bits - 12 : 0;
#pragma unroll
  for (int r = 0; r < kR; ++r)
    if (v[r] != 0ull) atomicAdd(&ms.cnt[(int)((v[r] - lo) >> shift)], 1u);
  __syncthreads();
  // Bucket offsets from the top: this thread's 4 buckets, a wave scan, then
  // the waves' totals (one per lane) for the offset of this wave.
  const int want = B < total ? B : total;
  uint32_t cb[4];
  int s4 = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    cb[q] = ms.cnt[4095 - 4 * tid - q];
    s4 += (int)cb[q];
  }
  const int incl = wave_incl_scan_add(s4);
  if (lane == kWave - 1) ms.wtot[wv] = incl;
  __syncthreads();
  const int wt = pl ? ms.wtot[lane] : 0;
  const int wincl = wave_incl_scan_add(wt);
  const int before = __builtin_amdgcn_readlane(wincl - wt, wv);  // totals of the waves before this one
  int run = before + incl - s4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int b = 4095 - 4 * tid - q;
    ms.cnt[b] = (uint32_t)run;  // bucket start, used as a cursor
    if (run < want && run + (int)cb[q] >= want) {
      ms.cut_bin = b;
      ms.cut_cnt = run + (int)cb[q];
    }
    run += (int)cb[q];
  }
  __syncthreads();
  const int cstar = ms.cut_bin, cum_at = ms.cut_cnt;
  if (cum_at > kSortMax) {  // uniform: too many in the cut's bucket
#pragma unroll
    for (int r = 0; r < kR; ++r)
      if (tid + r * kBlock < places) ms.X[tid + r * kBlock] = v[r];
    __syncthreads();
    return select_top(ms, places, B);
  }
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    if (v[r] != 0ull) {
      const int b = (int)((v[r] - lo) >> shift);
      if (b >= cstar) ms.S[atomicAdd(&ms.cnt[b], 1u)] = v[r];
    }
  }
  __syncthreads();
  // ms.cnt[b] is now the end of bucket b, and the end of bucket b+1 is its
  // start: rank each element inside its bucket.
  for (int i = tid; i < cum_at; i += kBlock) {
    const uint64_t x = ms.S[i];
    const int b = (int)((x - lo) >> shift);
    const int start = b == 4095 ? 0 : (int)ms.cnt[b + 1];
    const int end = (int)ms.cnt[b];
    int rank = 0;
    for (int j = start; j < end; ++j) rank += ms.S[j] > x;
    ms.X[start + rank] = x;
  }
  __syncthreads();
  return want;
}

// Count of entries greater than v in the descending array a[0..len).
__device__ __forceinline__ int count_greater_desc(const uint64_t* a, int len, uint64_t v) {
  int lo = 0, hi = len;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (a[mid] > v)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// X[0..U0) holds the current top entries sorted descending, S[0..k) new
// entries (distinct from them).  Leaves the top min(B, U0 + k) of both
// sorted in X and returns that count.  A short S is sorted by rank counting
// and merged by binary searches; a long one goes through select_top.
constexpr int kMergeNewRank = 512;
__device__ inline int merge_new(MergeShared& ms, int U0, int k, int B) {
  const int tid = threadIdx.x;
  if (k == 0) return U0;
  if (k > kMergeNewRank || U0 + k > kMergeCap) {
    for (int i = tid; i < k; i += kBlock) ms.X[U0 + i] = ms.S[i];
    __syncthreads();
    return select_top(ms, U0 + k, B);
  }
  for (int e = tid; e < k; e += kBlock) {
    const uint64_t y = ms.S[e];
    int r = 0;
#pragma unroll 8
    for (int j = 0; j < k; ++j) r += ms.S[j] > y;
    ms.X[U0 + r] = y;
  }
  __syncthreads();
  const int total = U0 + k < B ? U0 + k : B;
  const uint64_t* N = ms.X + U0;
  for (int i = tid; i < U0; i += kBlock) {
    const uint64_t x = ms.X[i];
    const int r = i + count_greater_desc(N, k, x);
    if (r < total) ms.S[r] = x;
  }
  for (int j = tid; j < k; j += kBlock) {
    const uint64_t y = N[j];
    const int r = j + count_greater_desc(ms.X, U0, y);
    if (r < total) ms.S[r] = y;
  }
  __syncthreads();
  for (int i = tid; i < total; i += kBlock) ms.X[i] = ms.S[i];
  __syncthreads();
  return total;
}

}  // namespace ewsjf
