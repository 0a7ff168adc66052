// Refine-and-Prune (Section 4.2) on the GPU.
//
// The paper sorts the window (the O(N log N) step of the strategic loop).
// Prompt lengths are bounded integers, so a length histogram carries exactly
// the information of the sorted window: the distinct values in order and
// their multiplicities.  Kernels:
//
//   window_hist      LDS-privatized histogram of clamped window lengths, one
//                    partial histogram per workgroup (no global atomics).
//   hist_reduce      column sums of the partial histograms.
//   hist_clear /     the same histogram into a caller-owned array (of a
//   window_hist_add  window kept as a range of a ring of recent lengths),
//                    flushed with one global atomic per non-empty bin per
//                    workgroup; the partition can start from it.
//   window_hist_move the window moved forward by n entries: the counts of
//                    the lengths that leave it go to the ones that join it.
//   rp_distinct      distinct values v[], counts c[] and exact int64 prefix
//                    sums of counts and of count * value.
//   rp_km_corners /  the exact 1-D 3-means initializer over the splits (i, j) of
//   rp_kmeans3       the distinct values, binary64 objective, ties to the
//                    smallest (i, j); tiles of splits that cannot hold the
//                    maximum are skipped.
//   rp_refine_prune  one workgroup: Stage 1 cluster starts, Stage 2 as
//                    level-synchronous passes (every significant gap of every
//                    current cluster is cut in the same pass; a pass without a
//                    new cut ends the recursion), then the leaves (the queue
//                    table when they fit the budget).
//   rp_merge         one workgroup: Stage 3, greedy merges of the
//                    lowest-utility adjacent pair, then the queue table.
//
// Every binary64 expression is evaluated in the same order as the oracle's
// definition and the library is built without floating-point contraction, so
// boundaries, counts, sums and means agree bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ewsjf_device.h"
#include "ewsjf_launch.h"

namespace ewsjf {

namespace {

constexpr int kHistPerBlock = 16384;   // window entries per histogram workgroup
constexpr int kMaxHistBlocks = 64;
constexpr int kKmeansBlocks = 256;
constexpr int kKmTile = 64;            // 3-means splits are taken in tiles of kKmTile x kKmTile
constexpr int kKmCorners = 64;         // workgroups of the corner pass
// tiles one workgroup of rp_kmeans3 tests
constexpr int kKmMaxTests = (EWSJF_MAX_LEN / kKmTile) * (EWSJF_MAX_LEN / kKmTile) / kKmeansBlocks;
constexpr int kLeafLds = 2048;         // Stage-3 leaves kept in LDS
constexpr uint64_t kInfBits = 0x7FF0000000000000ull;  // +inf as binary64 bits

// A Stage-3 leaf with its neighbours' links and the density and mean of the
// leaf after it (so one merge needs two rounds of LDS reads).  48 bytes.
struct alignas(16) Leaf {
  int64_t n, S;
  double rho, mean;      // n / (hi - lo + 1), S / n
  double rho_n, mean_n;  // the same of the next leaf (unused when nxt < 0)
  int32_t lo, hi;
  int32_t nxt, prv;      // -1: none; prv == -2 marks a merged-away leaf
};

struct PartWs {
  uint32_t* partial;  // [Gh][hist_row(L)]
  uint32_t* hist_buf; // [hist_row(L)] the window's histogram when the partition builds it
  const uint32_t* hist;  // the histogram the partition reads: hist_buf or the caller's
  int32_t* v;         // [L] distinct values
  uint32_t* c;        // [L] multiplicities
  int64_t* PN;        // [L+1] prefix sums of c
  int64_t* PS;        // [L+1] prefix sums of c * v
  int32_t* meta;      // [16]: 0 V, 3 leaves
  double* km_F;       // [kKmeansBlocks]
  int32_t* km_ij;     // [kKmeansBlocks][2]
  double* km_Q;       // [EWSJF_MAX_LEN / kKmTile] sums of squares of the value tiles
  double* km_corner;  // [kKmCorners]
  int64_t* gN;        // [L+1] leaves: exclusive prefix sums of their counts
  int64_t* gS;        // [L+1] ... and of their sums
  int32_t* glo;       // [L]
  int32_t* ghi;       // [L]
  Leaf* grec;         // [L] Stage-3 records (or chain arrays) when the leaves exceed LDS
  uint64_t* gU;       // [L]
  int Gh;
};

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

int hist_blocks(int64_t n) {
  int64_t g = (n + kHistPerBlock - 1) / kHistPerBlock;
  if (g < 1) g = 1;
  if (g > kMaxHistBlocks) g = kMaxHistBlocks;
  return (int)g;
}

// Workgroups of window_hist_add: 4,096 entries each up to 16 of them (one round
// of loads; the 65,536-length recount and its repartition take 77.5 us with 16,
// 79.4 us with four), 16,384 each from then on: every workgroup adds each of
// its lengths to the histogram once, so smaller shares only add the same
// lengths more often (262,144 and 524,288 uniform lengths: 12.5 and 14.1 us with
// 64 workgroups, 11.9 and 12.2 us with 16 and 32).
int add_blocks(int64_t n) {
  const int64_t small = std::clamp<int64_t>((n + 4 * kBlock - 1) / (4 * kBlock), 1, 16);
  return std::max((int)small, hist_blocks(n));
}

// Entries of one partial histogram: L + 1 bins, padded to whole 16-byte vectors.
__host__ __device__ inline int hist_row(int L) { return (L + 4) & ~3; }

PartWs carve_part(void* ws, int64_t n, int L) {
  PartWs w;
  w.Gh = hist_blocks(n);
  char* b = static_cast<char*>(ws);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* p = b + o;
    o += up256(bytes);
    return p;
  };
  w.partial = reinterpret_cast<uint32_t*>(take((size_t)w.Gh * hist_row(L) * 4));
  w.hist_buf = reinterpret_cast<uint32_t*>(take((size_t)hist_row(L) * 4));
  w.hist = w.hist_buf;
  w.v = reinterpret_cast<int32_t*>(take((size_t)L * 4));
  w.c = reinterpret_cast<uint32_t*>(take((size_t)L * 4));
  w.PN = reinterpret_cast<int64_t*>(take((size_t)(L + 1) * 8));
  w.PS = reinterpret_cast<int64_t*>(take((size_t)(L + 1) * 8));
  w.meta = reinterpret_cast<int32_t*>(take(16 * 4));
  w.km_F = reinterpret_cast<double*>(take(kKmeansBlocks * 8));
  w.km_ij = reinterpret_cast<int32_t*>(take(kKmeansBlocks * 8));
  w.km_Q = reinterpret_cast<double*>(take(EWSJF_MAX_LEN / kKmTile * 8));
  w.km_corner = reinterpret_cast<double*>(take(kKmCorners * 8));
  w.gN = reinterpret_cast<int64_t*>(take((size_t)(L + 1) * 8));
  w.gS = reinterpret_cast<int64_t*>(take((size_t)(L + 1) * 8));
  w.glo = reinterpret_cast<int32_t*>(take((size_t)L * 4));
  w.ghi = reinterpret_cast<int32_t*>(take((size_t)L * 4));
  w.grec = reinterpret_cast<Leaf*>(take((size_t)L * sizeof(Leaf)));
  w.gU = reinterpret_cast<uint64_t*>(take((size_t)L * 8));
  return w;
}

size_t carve_size(int64_t n, int L) {
  PartWs w = carve_part(nullptr, n, L);
  return reinterpret_cast<size_t>(w.gU) + up256((size_t)L * 8);
}

// ---------------------------------------------------------------------------
// A window length as the partition counts it: clamped to [1, L].
__device__ __forceinline__ int clamp_len(int32_t b, int L) { return b < 1 ? 1 : (b > L ? L : b); }

// The entry i < n of a window kept as ring[(begin + i) mod cap] (begin < cap,
// n <= cap, so one subtraction wraps it).
__device__ __forceinline__ int32_t ring_at(const int32_t* __restrict__ ring, int64_t cap, int64_t begin, int64_t i) {
  int64_t j = begin + i;
  if (j >= cap) j -= cap;
  return ring[j];
}

// Histogram bins in LDS, in whole 16-byte vectors.
constexpr int kHistVecs = (EWSJF_MAX_LEN + 4) / 4;

__device__ __forceinline__ void lds_hist_clear(i32x4* h, int L) {
  for (int i = threadIdx.x; i < hist_row(L) / 4; i += kBlock) h[i] = i32x4{0, 0, 0, 0};
}

// This workgroup's share of the n window entries counted into h[0..L] (LDS,
// the rest of h's vectors 0).  Four entries in flight per thread, the first
// four while the bins are cleared.
__device__ void lds_window_hist(const int32_t* __restrict__ ring, int64_t cap, int64_t begin, int64_t n, int L,
                                uint32_t* h) {
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t beg = per * blockIdx.x;
  const int64_t end = beg + per < n ? beg + per : n;
  int32_t x[4];
  auto load = [&](int64_t i) {
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = i + u * kBlock < end ? ring_at(ring, cap, begin, i + u * kBlock) : 0;
  };
  int64_t i = beg + threadIdx.x;
  load(i);
  lds_hist_clear(reinterpret_cast<i32x4*>(h), L);
  __syncthreads();
  while (i < end) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * kBlock < end) atomicAdd(&h[clamp_len(x[u], L)], 1u);
    i += 4 * kBlock;
    load(i);
  }
  __syncthreads();
}

__global__ __launch_bounds__(kBlock) void window_hist(const int32_t* __restrict__ win, int64_t n, int L,
                                                      uint32_t* __restrict__ partial) {
  __shared__ i32x4 h[kHistVecs];
  lds_window_hist(win, n, 0, n, L, reinterpret_cast<uint32_t*>(h));
  i32x4* out = reinterpret_cast<i32x4*>(partial + (size_t)blockIdx.x * hist_row(L));
  for (int i = threadIdx.x; i < hist_row(L) / 4; i += kBlock) out[i] = h[i];
}

__global__ void hist_clear(uint32_t* __restrict__ hist, int L) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b <= L) hist[b] = 0u;
}

__global__ __launch_bounds__(kBlock) void window_hist_add(const int32_t* __restrict__ ring, int64_t cap,
                                                          int64_t begin, int64_t n, int L,
                                                          uint32_t* __restrict__ hist) {
  __shared__ i32x4 hv[kHistVecs];
  uint32_t* h = reinterpret_cast<uint32_t*>(hv);
  lds_window_hist(ring, cap, begin, n, L, h);
  // A wave adds to 64 neighbouring bins: two cache lines an instruction.  Four
  // bins per thread (vector reads of LDS) are eight lines, each touched four
  // times: 1M lengths of two modes took 18.3 us, uniform ones 47.8 us; 10.5 and
  // 16.1 us with these.  Eight reads of LDS in flight.
  constexpr int kFlush = 8;
  for (int b0 = threadIdx.x; b0 <= L; b0 += kFlush * kBlock) {
    uint32_t x[kFlush];
#pragma unroll
    for (int u = 0; u < kFlush; ++u) x[u] = b0 + u * kBlock <= L ? h[b0 + u * kBlock] : 0u;
#pragma unroll
    for (int u = 0; u < kFlush; ++u)
      if (x[u] != 0u) atomicAdd(&hist[b0 + u * kBlock], x[u]);
  }
}

// Column sums of the partial histograms.  Four bins per thread and four
// groups of rows per workgroup, so a thread's 16 loads of the largest window
// (64 rows) are in flight together: 6.3 us for the
// 1M window's 8 MiB of partials, against 18 us with one bin per thread and one
// row at a time.
constexpr int kReduceVecs = 64, kReduceRows = 4;
__global__ __launch_bounds__(kReduceVecs * kReduceRows) void hist_reduce(const uint32_t* __restrict__ partial, int Gh,
                                                                         int L, uint32_t* __restrict__ hist) {
  __shared__ i32x4 part[kReduceRows][kReduceVecs];
  const int c = threadIdx.x % kReduceVecs, g0 = threadIdx.x / kReduceVecs;
  const int nv = hist_row(L) / 4, i = blockIdx.x * kReduceVecs + c;
  const i32x4* src = reinterpret_cast<const i32x4*>(partial) + min(i, nv - 1);
  i32x4 s{0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < kMaxHistBlocks / kReduceRows; ++u) {
    const int g = g0 + u * kReduceRows;
    if (g < Gh) s += src[(size_t)g * nv];
  }
  part[g0][c] = s;
  __syncthreads();
  if (g0 == 0 && i < nv) {
#pragma unroll
    for (int r = 1; r < kReduceRows; ++r) s += part[r][c];
    reinterpret_cast<i32x4*>(hist)[i] = s;
  }
}

// The window moves forward by n entries: the counts of the n lengths that
// leave it (ring[(sub + i) mod cap]) move to the n that join it
// (ring[(add + i) mod cap]).  Per-workgroup signed deltas in LDS, flushed as
// modular uint32 adds: the final counts are exact in any flush order.
__global__ __launch_bounds__(kBlock) void window_hist_move(const int32_t* __restrict__ ring, int64_t cap, int64_t add,
                                                           int64_t sub, int64_t n, int L,
                                                           uint32_t* __restrict__ hist) {
  __shared__ i32x4 dv[kHistVecs];
  int32_t* d = reinterpret_cast<int32_t*>(dv);
  lds_hist_clear(dv, L);
  __syncthreads();
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t beg = per * blockIdx.x;
  const int64_t end = beg + per < n ? beg + per : n;
  for (int64_t i = beg + threadIdx.x; i < end; i += kBlock) {
    const int ca = clamp_len(ring_at(ring, cap, add, i), L);
    const int cs = clamp_len(ring_at(ring, cap, sub, i), L);
    if (ca != cs) {
      atomicAdd(&d[ca], 1);
      atomicSub(&d[cs], 1);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b <= L; b += kBlock)
    if (d[b]) atomicAdd(&hist[b], (uint32_t)d[b]);
}

// Distinct values and exact prefix sums.  Workgroup w takes the bins (lengths)
// 1024 w + 1 .. 1024 w + 1024, one per thread, and sums the bins before them
// itself (at most 31 loads per thread, from L2 after the first workgroup), so
// no workgroup waits for another.  Bound by latency: one round of loads and
// one of LDS, 6.2 us (8.9 us with eight loads in flight and every thread
// reading all waves' partials; 30-45 us on one workgroup over all bins).
__global__ __launch_bounds__(kBlock) void rp_distinct(PartWs w, int L) {
  __shared__ int64_t sN[kWavesPerBlock], sS[kWavesPerBlock], tN[kWavesPerBlock], tS[kWavesPerBlock];
  __shared__ int sV[kWavesPerBlock], tV[kWavesPerBlock];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  const int b = (int)blockIdx.x * kBlock + tid + 1;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w.hist), (short)0, (L + 1) * 4, kBufferWord3);
  const uint32_t h = __builtin_amdgcn_raw_buffer_load_b32(rs, b * 4, 0, 0);  // past bin L: 0
  // The bins of the workgroups before this one, all loads in flight together
  // (an offset past the buffer reads 0).
  constexpr int kBefore = EWSJF_MAX_LEN / kBlock - 1;
  static_assert(EWSJF_MAX_LEN % kBlock == 0, "at most kBefore workgroups before one");
  uint32_t x[kBefore];
#pragma unroll
  for (int q = 0; q < kBefore; ++q)
    x[q] = __builtin_amdgcn_raw_buffer_load_b32(rs, q < (int)blockIdx.x ? (q * kBlock + tid + 1) * 4 : (L + 1) * 4, 0, 0);
  int v0 = 0;
  int64_t n0 = 0, s0 = 0;
#pragma unroll
  for (int q = 0; q < kBefore; ++q) {
    v0 += x[q] != 0u;
    n0 += x[q];
    s0 += (int64_t)x[q] * (q * kBlock + tid + 1);
  }
  // Inclusive scans over the wave of this workgroup's bins, wave sums of the
  // bins before it.
  const uint64_t live = __ballot(h != 0u);
  int64_t n = h, s = (int64_t)h * b;
  for (int off = 1; off < kWave; off <<= 1) {
    const int64_t yn = __shfl_up(n, off), ys = __shfl_up(s, off);
    if (lane >= off) {
      n += yn;
      s += ys;
    }
    n0 += __shfl_xor(n0, off);
    s0 += __shfl_xor(s0, off);
  }
  v0 = wave_sum_i32(v0);
  if (lane == kWave - 1) {
    sV[wv] = (int)__popcll(live);
    sN[wv] = n;
    sS[wv] = s;
    tV[wv] = v0;
    tN[wv] = n0;
    tS[wv] = s0;
  }
  __syncthreads();
  // Each wave sums the partials before it itself, one wave's per lane.
  static_assert(kWavesPerBlock == 16, "the sums below are over 16 lanes");
  const int p = lane & (kWavesPerBlock - 1);
  const bool mine = p < wv;
  int pos = tV[p] + (mine ? sV[p] : 0);
  int64_t pn = tN[p] + (mine ? sN[p] : 0), ps = tS[p] + (mine ? sS[p] : 0);
#pragma unroll
  for (int off = 1; off < kWavesPerBlock; off <<= 1) {
    pos += __shfl_xor(pos, off);
    pn += __shfl_xor(pn, off);
    ps += __shfl_xor(ps, off);
  }
  pos += lanes_below(live);
  if (h != 0u) {
    w.v[pos] = b;
    w.c[pos] = h;
    w.PN[pos] = pn + n - h;
    w.PS[pos] = ps + s - (int64_t)h * b;
  }
  if (blockIdx.x == gridDim.x - 1 && tid == kBlock - 1) {
    const int V = pos + (h != 0u);
    w.PN[V] = pn + n;
    w.PS[V] = ps + s;
    w.meta[0] = V;
  }
}

// ---------------------------------------------------------------------------
// Exact 1-D 3-means over the splits 1 <= i < j <= V-1 of the distinct values:
// the largest F(i, j) = f(0, i) + f(i, j) + f(j, V), f(x, y) = (sum)^2 / count
// of the values x..y-1 (the least squared error), ties to the smallest (i, j).
//
// The splits form a V x V triangle, 148 million pairs for 17,000 values, of
// which few can hold the maximum.  They are taken in tiles of 64 x 64.  For
// every split of a tile the three clusters contain [0, i0), [i1, j0) and
// [j1, V) (i0..i1 and j0..j1 the tile's ranges), and the values between add at
// most their squares to F (adding a value to a cluster never lowers its
// squared error), so
//   F <= f(0, i0) + f(i1, j0) + f(j1, V) + Q(i0..i1) + Q(j0..j1),
// Q a sum of squares.  Tiles whose bound is below the best F at any tile's
// corner are skipped, the rest evaluated pair by pair in the definition's
// expression order.  Of 37,128 tiles (17,362 values, a 262,144 window of three
// modes) 256 are evaluated, of 131,328 (32,768 values, each once) 601.
// On that window the two kernels take 19 us; every pair evaluated with three
// divisions took 400 us (and its one-thread pick 28 us).
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool km_better(double F, int i, int j, double bF, int bi, int bj) {
  if (F > bF) return true;
  if (F < bF) return false;
  return i < bi || (i == bi && j < bj);
}

// f(x, y) of the values x..y-1 (0 when there are none).
__device__ __forceinline__ double km_f(const PartWs& w, int x, int y) {
  const double n = (double)(w.PN[y] - w.PN[x]), s = (double)(w.PS[y] - w.PS[x]);
  return y > x ? (s * s) / n : 0.0;
}

// F at one split, in the definition's order.
__device__ __forceinline__ double km_F(double f1, double s2, double n2, double f3) {
  return (f1 + (s2 * s2) / n2) + f3;
}

// The best F at a tile's first split, and the sum of squares of each tile's
// values.
__global__ __launch_bounds__(kBlock) void rp_km_corners(PartWs w) {
  __shared__ double sF[kWavesPerBlock];
  const int V = w.meta[0];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  const int nb = (V + kKmTile - 1) / kKmTile;
  const int b = (int)blockIdx.x * kWavesPerBlock + wv;
  static_assert(kKmCorners * kWavesPerBlock >= EWSJF_MAX_LEN / kKmTile && kKmTile == kWave, "a wave per value tile");
  if (b < nb) {
    const int j = b * kKmTile + lane;
    double q = 0.0;
    if (j < V) {
      const double v = (double)w.v[j];
      q = (double)w.c[j] * (v * v);
    }
    for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off);
    if (lane == 0) w.km_Q[b] = q;
  }
  double best = 0.0;
  for (int t = (int)blockIdx.x * kBlock + tid; t < nb * nb; t += kKmCorners * kBlock) {
    const int ti = t / nb, tj = t - ti * nb;
    const int i = max(ti * kKmTile, 1), j = max(tj * kKmTile, i + 1);
    if (tj < ti || j > V - 1) continue;
    const double F = km_F(km_f(w, 0, i), (double)(w.PS[j] - w.PS[i]), (double)(w.PN[j] - w.PN[i]), km_f(w, j, V));
    best = F > best ? F : best;
  }
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(best, off);
    best = o > best ? o : best;
  }
  if (lane == 0) sF[wv] = best;
  __syncthreads();
  if (tid == 0) {
    for (int q = 1; q < kWavesPerBlock; ++q) best = sF[q] > best ? sF[q] : best;
    w.km_corner[blockIdx.x] = best;
  }
}

__global__ __launch_bounds__(kBlock) void rp_kmeans3(PartWs w) {
  __shared__ double sF[kWavesPerBlock];
  __shared__ int si[kWavesPerBlock], sj[kWavesPerBlock];
  __shared__ int tiles[kKmMaxTests];
  __shared__ int ntiles;
  const int V = w.meta[0];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  double bF = -1.0;
  int bi = 0x7fffffff, bj = 0x7fffffff;
  if (V > 3) {
    double best = w.km_corner[lane];
    static_assert(kKmCorners == kWave, "one corner maximum per lane");
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(best, off);
      best = o > best ? o : best;
    }
    if (tid == 0) ntiles = 0;
    __syncthreads();
    // Which of this workgroup's tiles can hold the maximum.  Every operand is
    // positive, so the bound and the corner values are within 1e-14 of their
    // exact values, far inside the margin.
    const int nb = (V + kKmTile - 1) / kKmTile;
    for (int t = (int)blockIdx.x + kKmeansBlocks * tid; t < nb * nb; t += kKmeansBlocks * kBlock) {
      const int ti = t / nb, tj = t - ti * nb;
      if (tj < ti) continue;
      const int i0 = max(ti * kKmTile, 1), i1 = min(ti * kKmTile + kKmTile - 1, V - 2);
      const int j0 = max(tj * kKmTile, 2), j1 = min(tj * kKmTile + kKmTile - 1, V - 1);
      if (i0 > i1 || j0 > j1) continue;
      const double ub = (km_f(w, 0, i0) + km_f(w, i1, j0)) + km_f(w, j1, V) +
                        (w.km_Q[ti] + (tj > ti ? w.km_Q[tj] : 0.0));
      if (ub * (1.0 + 1e-12) >= best) tiles[atomicAdd(&ntiles, 1)] = t;
    }
    __syncthreads();
    const int64_t NV = w.PN[V], SV = w.PS[V];
    for (int k = 0; k < ntiles; ++k) {  // a lane per j, a wave per i
      const int ti = tiles[k] / nb, tj = tiles[k] - ti * nb;
      const int j = tj * kKmTile + lane;
      const bool in = j >= 2 && j <= V - 1;
      const int64_t Nj = w.PN[in ? j : 0], Sj = w.PS[in ? j : 0];
      const double n3 = (double)(NV - Nj), s3 = (double)(SV - Sj);
      const double f3 = (s3 * s3) / n3;
#pragma unroll
      for (int r = 0; r < kKmTile / kWavesPerBlock; ++r) {
        const int i = ti * kKmTile + r * kWavesPerBlock + wv;  // wave-uniform
        if (i < 1 || i > V - 2) continue;
        const int64_t Ni = w.PN[i], Si = w.PS[i];
        const double n1 = (double)Ni, s1 = (double)Si;
        const double F = km_F((s1 * s1) / n1, (double)(Sj - Si), (double)(Nj - Ni), f3);
        if (in && j > i && km_better(F, i, j, bF, bi, bj)) {
          bF = F;
          bi = i;
          bj = j;
        }
      }
    }
  }
  // block argmax with the tie rule
  for (int off = 32; off > 0; off >>= 1) {
    const double oF = __shfl_xor(bF, off);
    const int oi = __shfl_xor(bi, off), oj = __shfl_xor(bj, off);
    if (km_better(oF, oi, oj, bF, bi, bj)) {
      bF = oF;
      bi = oi;
      bj = oj;
    }
  }
  if (lane == 0) {
    sF[wv] = bF;
    si[wv] = bi;
    sj[wv] = bj;
  }
  __syncthreads();
  if (tid == 0) {
    for (int q = 0; q < kWavesPerBlock; ++q)
      if (km_better(sF[q], si[q], sj[q], bF, bi, bj)) {
        bF = sF[q];
        bi = si[q];
        bj = sj[q];
      }
    w.km_F[blockIdx.x] = bF;
    w.km_ij[2 * blockIdx.x] = bi;
    w.km_ij[2 * blockIdx.x + 1] = bj;
  }
}

// The best split over rp_kmeans3's workgroups, in every lane of one wave.
__device__ __forceinline__ void km_pick(const PartWs& w, int* ki, int* kj) {
  const int lane = threadIdx.x & (kWave - 1);
  double bF = -1.0;
  int bi = 0x7fffffff, bj = 0x7fffffff;
  for (int q = lane; q < kKmeansBlocks; q += kWave)
    if (km_better(w.km_F[q], w.km_ij[2 * q], w.km_ij[2 * q + 1], bF, bi, bj)) {
      bF = w.km_F[q];
      bi = w.km_ij[2 * q];
      bj = w.km_ij[2 * q + 1];
    }
  for (int off = 32; off > 0; off >>= 1) {
    const double oF = __shfl_xor(bF, off);
    const int oi = __shfl_xor(bi, off), oj = __shfl_xor(bj, off);
    if (km_better(oF, oi, oj, bF, bi, bj)) {
      bF = oF;
      bi = oi;
      bj = oj;
    }
  }
  *ki = bi;
  *kj = bj;
}

// ---------------------------------------------------------------------------
// Stage 3 utility of the adjacent pair (a, b), Eq. 3 with density = count per
// token of value span.  Same binary64 expression order as the definition.
// ---------------------------------------------------------------------------
// rho = count / (hi - lo + 1) and m = sum / count of each are computed once.
__device__ __forceinline__ double utility_cached(double rho_a, double m_a, double rho_b, double m_b, double eps) {
  return (rho_a + rho_b) / (fabs(m_b - m_a) + eps);
}

__device__ __forceinline__ uint64_t dbits(double x) { return (uint64_t)__double_as_longlong(x); }

// ---------------------------------------------------------------------------
// Stages 1 and 2, one workgroup.  The distinct values sit in LDS; segment
// (cluster) starts are bits of 64-bit words, one word per 64 consecutive
// values (a wave's group), so the segment of a value is a count of bits.
//
// A level of Stage 2 cuts every gap g of a segment of VC values over a span
// with g (VC - 1) > alpha span (binary64, in this order).  The left side never
// falls as g grows, so a segment's test is a whole-number threshold on its
// gaps, found once per segment (a thread each) from a quotient and corrected
// with the test itself; a level is then one compare per value against its
// segment's threshold.  With the test evaluated for every gap a level took
// 14 us (two conversions and two binary64 products per gap, 32 gaps per
// thread whatever V), the kernel 78-87 us; it takes 34-46 us now, 5 to 7 us a level.
// ---------------------------------------------------------------------------
constexpr int kGroups = EWSJF_MAX_LEN / kWave;  // 512
constexpr int kNoCut = 0xFFFF;                  // above every gap
constexpr int kGroupsPerWave = kGroups / kWavesPerBlock;  // 32: group wv + 16 u is wave wv's u-th

struct RpShared {
  uint16_t v[EWSJF_MAX_LEN];
  uint16_t seg[EWSJF_MAX_LEN];  // of each segment: its start, then the gap threshold
  uint64_t start[kGroups];      // bit l of word g: value 64 g + l starts a segment
  uint64_t cut[kGroups];        // bit l of word g: the gap after value 64 g + l is cut
  uint16_t first[kGroups];      // segments that start before the group
  int iscr[kWavesPerBlock];
};

// The value of lane `src` (uniform) of a 64-bit register.
__device__ __forceinline__ uint64_t readlane_u64(uint64_t x, int src) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

// The segments' starts in order, sm.seg[0..nseg), from the start bits `mine`
// of group tid (tid < kGroups, also in sm.start); returns nseg.
__device__ int list_segments(RpShared& sm, uint64_t mine, int ng) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  int nseg = 0;
  const int before = block_exclusive_scan((int)__popcll(mine), sm.iscr, &nseg);
  if (tid < kGroups) sm.first[tid] = (uint16_t)before;  // below 32768 wherever the group has a start
  __syncthreads();
  const uint64_t gstart = lane < kGroupsPerWave ? sm.start[wv + lane * kWavesPerBlock] : 0ull;  // 0 past the groups in use
  const int gfirst = lane < kGroupsPerWave ? (int)sm.first[wv + lane * kWavesPerBlock] : 0;
  for (int u = 0; wv + u * kWavesPerBlock < ng; ++u) {
    const uint64_t m = readlane_u64(gstart, u);  // in scalar registers, as the lane mask of the store
    const int f = __builtin_amdgcn_readlane(gfirst, u);
    if (__builtin_amdgcn_inverse_ballot_w64(m))
      sm.seg[f + lanes_below(m)] = (uint16_t)((wv + u * kWavesPerBlock) * kWave + lane);
  }
  __syncthreads();
  return nseg;
}

// The largest gap that a segment of VC values over `span` (mm1: its VC - 1,
// or its entries - 1 in the multiset reading) does not cut.
__device__ __forceinline__ int gap_threshold(double alpha, int span, double mm1) {
  const double rhs = alpha * (double)span;
  const double q = rhs / mm1;
  if (!(q < 40000.0)) return kNoCut;
  int t = (int)q;
  while (t < 40000 && !((double)(t + 1) * mm1 > rhs)) ++t;
  while (t > 0 && (double)t * mm1 > rhs) --t;
  return t;
}

// The queue table from k queues in length order, given by the prefix sums of
// their counts and sums and their intervals.
__device__ void write_queues(ewsjf_queue_table* tab, int k, const int64_t* N, const int64_t* S, const int32_t* lo,
                             const int32_t* hi, int tid, int nthreads) {
  for (int i = tid; i < k; i += nthreads) {
    const int64_t cn = N[i + 1] - N[i], cs = S[i + 1] - S[i];
    const int32_t l = lo[i], h = hi[i];
    if (i > 0) tab->bounds[i - 1] = l;
    tab->lo[i] = l;
    tab->hi[i] = h;
    tab->count[i] = cn;
    tab->sum[i] = cs;
    tab->mean[i] = (double)cs / (double)cn;
  }
  if (tid == 0) tab->k = k;
}

__global__ __launch_bounds__(kBlock) void rp_refine_prune(PartWs w, ewsjf_partition_params p, int64_t n_window,
                                                          ewsjf_queue_table* tab) {
  __shared__ RpShared sm;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int V = w.meta[0];
  const int L = p.max_len;
  if (V == 0) {
    // An empty histogram (only a caller-kept one can be empty): one queue
    // that holds nothing and covers every length.
    if (tid == 0) {
      w.meta[3] = 0;
      tab->k = 1;
      tab->max_len = L;
      tab->n_distinct = tab->n_coarse = tab->n_leaves = tab->gapped = 0;
      tab->n_window = 0;
      tab->lo[0] = tab->hi[0] = 0;
      tab->count[0] = tab->sum[0] = 0;
      tab->mean[0] = 0.0;
    }
    return;
  }

  {
    // Sixteen loads in flight per thread (bounded: past V they read 0).
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(w.v, (short)0, V * 4, kBufferWord3);
    for (int j0 = tid; j0 < V; j0 += 16 * kBlock) {
      uint32_t x[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, (j0 + k * kBlock) * 4, 0, 0);
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (j0 + k * kBlock < V) sm.v[j0 + k * kBlock] = (uint16_t)x[k];
    }
  }
  if (tid < kGroups) sm.start[tid] = 0ull;
  __syncthreads();
  const int ng = (V + kWave - 1) / kWave;  // groups in use

  // ---- Stage 1: coarse cluster starts -------------------------------------
  if (p.init_mode == EWSJF_INIT_EQUAL_WIDTH) {
    // (v - lo) K < 2^30 (values and K are at most 32768): the 32-bit quotient
    // is the exact floor of the int64 definition.
    const uint32_t vlo = sm.v[0], width = (uint32_t)sm.v[V - 1] - vlo + 1u;
    auto bin = [&](int j) { return ((uint32_t)sm.v[j] - vlo) * (uint32_t)p.init_queues / width; };
    const int per = (ng + kWavesPerBlock - 1) / kWavesPerBlock;  // consecutive groups per wave
    const int g0 = wv * per, g1 = min(ng, g0 + per);
    uint32_t before = g0 > 0 && g0 < g1 ? bin(g0 * kWave - 1) : 0xFFFFFFFFu;  // the bin of the value before the group
    for (int g = g0; g < g1; ++g) {
      const int j = g * kWave + lane;
      const uint32_t b = bin(min(j, V - 1));
      const uint32_t up = (uint32_t)__shfl_up((int)b, 1);
      const uint64_t m = __ballot(j < V && b != (lane > 0 ? up : before));
      if (lane == 0) sm.start[g] = m;
      before = (uint32_t)__builtin_amdgcn_readlane((int)b, kWave - 1);
    }
  } else {
    int ki, kj;
    km_pick(w, &ki, &kj);  // every wave, the same result
    for (int g = wv; g < ng; g += kWavesPerBlock) {
      const int j = g * kWave + lane;
      const uint64_t m = __ballot(j < V && (V <= 3 || j == 0 || j == ki || j == kj));
      if (lane == 0) sm.start[g] = m;
    }
  }
  __syncthreads();
  uint64_t mine = tid < kGroups ? sm.start[tid] : 0ull;  // the start bits of group tid
  int nl = list_segments(sm, mine, ng);
  const int n_coarse = nl;

  // ---- Stage 2: level-synchronous refinement --------------------------------
  // The gap after each value (0 past the last: never cut), lane l of group
  // wv + 16 u in gap[u].
  int gap[kGroupsPerWave];
#pragma unroll
  for (int u = 0; u < kGroupsPerWave; ++u) {
    const int j = (wv + u * kWavesPerBlock) * kWave + lane;
    gap[u] = 0;
    if (wv + u * kWavesPerBlock < ng) gap[u] = (int)sm.v[min(j + 1, V - 1)] - (int)sm.v[min(j, V - 1)];
  }
  const bool distinct = p.gap_mode == EWSJF_GAPS_DISTINCT;
  const int min_distinct = distinct ? 3 : 2;
  for (;;) {
    // The threshold of every segment takes the place of its start (a tile of
    // starts is read, with the next segment's, before it is overwritten).
    for (int i0 = 0; i0 < nl; i0 += kBlock) {
      const int i = i0 + tid;
      int t = kNoCut;
      if (i < nl) {
        const int j = sm.seg[i], e = i + 1 < nl ? (int)sm.seg[i + 1] : V;
        const int span = (int)sm.v[e - 1] - (int)sm.v[j];
        if (e - j >= min_distinct && span >= p.min_width)
          t = gap_threshold(p.alpha, span, distinct ? (double)(e - j - 1) : (double)((w.PN[e] - w.PN[j]) - 1));
      }
      __syncthreads();
      if (i < nl) sm.seg[i] = (uint16_t)t;
    }
    __syncthreads();
    // Every gap against its segment's threshold (one LDS read per gap: the
    // gaps stay in registers and the groups' words come from other lanes).
    {
      const uint64_t gstart = lane < kGroupsPerWave ? sm.start[wv + lane * kWavesPerBlock] : 0ull;
      const int gfirst = lane < kGroupsPerWave ? (int)sm.first[wv + lane * kWavesPerBlock] : 0;
      uint64_t cuts = 0;  // lane u: the cuts of the wave's u-th group
#pragma unroll
      for (int u0 = 0; u0 < kGroupsPerWave; u0 += 8) {
        if (wv + u0 * kWavesPerBlock < ng) {  // uniform; eight reads in flight (groups past the last read its segment)
          int thr[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            // the starts up to this lane, this one included: bit 0 and the bits of m >> 1 below it
            const uint64_t m = readlane_u64(gstart, u0 + k);
            const int before = __builtin_amdgcn_readlane(gfirst, u0 + k) + (int)(m & 1ull) - 1;  // scalar
            thr[k] = sm.seg[before + lanes_below(m >> 1)];
          }
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const uint64_t cm = __ballot(gap[u0 + k] > thr[k]);
            cuts = lane == u0 + k ? cm : cuts;
          }
        }
      }
      if (lane < kGroupsPerWave) sm.cut[wv + lane * kWavesPerBlock] = cuts;
    }
    __syncthreads();
    // A cut gap starts a segment at the next value (a gap between two
    // segments is one already).
    uint64_t now = mine;
    if (tid < ng) now |= (sm.cut[tid] << 1) | (tid > 0 ? sm.cut[tid - 1] >> 63 : 0ull);
    const int any = __syncthreads_or(now != mine);
    mine = now;
    if (tid < ng) sm.start[tid] = mine;
    __syncthreads();
    nl = list_segments(sm, mine, ng);
    if (!any) break;
  }

  // ---- Leaves: one per segment, aggregates from the exact prefix sums -------
  for (int i = tid; i < nl; i += kBlock) {
    const int j = sm.seg[i], e = i + 1 < nl ? (int)sm.seg[i + 1] : V;
    w.gN[i] = w.PN[j];
    w.gS[i] = w.PS[j];
    w.glo[i] = sm.v[j];
    w.ghi[i] = sm.v[e - 1];
  }
  if (tid == 0) {
    w.gN[nl] = w.PN[V];
    w.gS[nl] = w.PS[V];
  }
  __syncthreads();  // (write_queues reads them back in this workgroup)
  if (tid == 0) {
    w.meta[3] = nl;
    tab->max_len = L;
    tab->n_distinct = V;
    tab->n_coarse = n_coarse;
    tab->n_leaves = nl;
    tab->gapped = 0;
    tab->n_window = n_window >= 0 ? n_window : w.PN[V];
  }
  // Within the queue budget: the leaves are the queues.  Otherwise Stage 3
  // (rp_merge) writes them.
  if (nl <= p.max_queues) write_queues(tab, nl, w.gN, w.gS, w.glo, w.ghi, tid, kBlock);
}

}  // namespace

// ---------------------------------------------------------------------------
// Stage 3: greedy merge of the adjacent pair with the smallest utility until
// at most max_queues remain (Section 4.2, "Stage 3", Eq. 3; ties to the
// leftmost pair).
//
// The merges are sequential, but they come in chains: a merged queue is
// sparser and further from its neighbours' means in a way that makes its next
// pair the lowest again, so the queue that was just merged (the hot queue)
// takes its neighbour next, almost always on the same side (of 1,421 merges
// of a 262,144-length window in three modes, 1,419 continue the chain, 15 on
// the other side).  A chain is not serial: after j further merges on one side
// the hot queue is the union of j + 1 consecutive leaves, whose count and sum
// are differences of prefix sums, so lane j evaluates the state after j
// merges, all lanes at once (chain_merge).  The merges up to the first lane
// where another pair is the lowest are committed together.
//
// Measured (rp_merge alone): the 1M window of two modes into 256 queues
// 37 us, where one merge at a time took 253 us; a 65,536 window into 64
// queues 24 us against 363 us; the 262,144 window of three modes into 64
// queues 19 us against 1,119 us.  One merge at a time (merge_list) is bound
// by latency, about 0.75 us each: two dependent divisions, two reductions
// over the wave and three rounds of LDS reads.
//
// Data without chains (every merge far from the one before) goes through
// merge_list, the linked list with a cached minimum per lane.
// ---------------------------------------------------------------------------
constexpr int kMergeThreads = kBlock;

// Lowest lane holding the wave's minimum of x, and that minimum (*m).  The
// high words are reduced first, the low words only when several lanes share
// the smallest high word (utilities rarely do).
__device__ __forceinline__ int wave_argmin_u64(uint64_t x, uint64_t* m) {
  const uint32_t xh = (uint32_t)(x >> 32);
  const uint32_t mh = __ockl_wfred_min_u32(xh);
  uint64_t cand = __ballot(xh == mh);
  if (__popcll(cand) > 1) {
    const uint32_t ml = __ockl_wfred_min_u32(xh == mh ? (uint32_t)x : 0xFFFFFFFFu);
    cand = __ballot(xh == mh && (uint32_t)x == ml);
  }
  const int src = (int)__builtin_ctzll(cand);
  *m = ((uint64_t)mh << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, src);
  return src;
}

// One merge at a time.  Leaves keep their index (a linked list replaces
// shifting), and lane l caches the minimum utility over the pairs it owns
// (left-leaf indices [l*P, l*P + P)).  A merge costs a two-step wave
// reduction for the global minimum, two rounds of record reads and a rescan
// by the few lanes whose pairs changed.  Utilities are non-negative binary64
// values, so their bit patterns order like the values; ties go to the smaller
// leaf index, which is the smaller position in the list.  The records live in
// LDS, or in the workspace when there are more leaves than LDS holds.
template <bool kInLds>
__device__ __forceinline__ void merge_list(Leaf* rec, uint64_t* U, const PartWs& w, int nl0,
                                           const ewsjf_partition_params& p, ewsjf_queue_table* tab, int* iscr) {
  const int tid = threadIdx.x;
  for (int i = tid; i < nl0; i += kMergeThreads) {
    Leaf r;
    r.n = w.gN[i + 1] - w.gN[i];
    r.S = w.gS[i + 1] - w.gS[i];
    r.lo = w.glo[i];
    r.hi = w.ghi[i];
    r.rho = (double)r.n / (double)((int64_t)r.hi - (int64_t)r.lo + 1);
    r.mean = (double)r.S / (double)r.n;
    r.nxt = i + 1 < nl0 ? i + 1 : -1;
    r.prv = i - 1;
    r.rho_n = r.mean_n = 0.0;
    if (i + 1 < nl0) {
      const int64_t n1 = w.gN[i + 2] - w.gN[i + 1], S1 = w.gS[i + 2] - w.gS[i + 1];
      r.rho_n = (double)n1 / (double)((int64_t)w.ghi[i + 1] - (int64_t)w.glo[i + 1] + 1);
      r.mean_n = (double)S1 / (double)n1;
    }
    rec[i] = r;
    U[i] = i + 1 < nl0 ? dbits(utility_cached(r.rho, r.mean, r.rho_n, r.mean_n, p.eps)) : kInfBits;
  }
  __syncthreads();
  if (tid < kWave) {
    const int lane = tid;
    // Each lane owns P slots, P the power of two >= nl0 / 64 (owners by shift).
    int lgP = 0;
    while ((kWave << lgP) < nl0) ++lgP;
    const int P = 1 << lgP;
    // This lane's minimum (first index on ties) over its P slots.
    auto scan_own = [&](uint64_t& mu, int& mi) {
      mu = kInfBits + 1;  // above every utility, +inf included
      mi = 0x7fffffff;
#pragma unroll 8
      for (int q = 0; q < P; ++q) {
        const int i = (lane << lgP) + q;
        const uint64_t u = i < nl0 ? U[i] : ~0ull;
        if (u < mu) {
          mu = u;
          mi = i;
        }
      }
    };
    uint64_t lane_u;
    int lane_i;
    scan_own(lane_u, lane_i);
    // Lane `owner`'s minimum recomputed by the whole wave, one slot per lane
    // (P <= kWave when the records are in LDS).
    auto rescan = [&](int owner) {
      if constexpr (kInLds) {
        const int i = (owner << lgP) + lane;
        const uint64_t u = (lane < P && i < nl0) ? U[i] : ~0ull;
        uint64_t m;
        const int src = wave_argmin_u64(u, &m);
        if (lane == owner) {
          lane_u = m == ~0ull ? kInfBits + 1 : m;
          lane_i = m == ~0ull ? 0x7fffffff : (owner << lgP) + src;
        }
      } else {
        if (lane == owner) scan_own(lane_u, lane_i);
      }
    };
    for (int alive = nl0; alive > p.max_queues; --alive) {
      uint64_t mu;
      const int a = __builtin_amdgcn_readlane(lane_i, wave_argmin_u64(lane_u, &mu));
      const int b = rec[a].nxt, pr = rec[a].prv;
      const int64_t na = rec[a].n + rec[b].n;
      const int64_t Sa = rec[a].S + rec[b].S;
      const int32_t hia = rec[b].hi;
      const int c = rec[b].nxt;
      const double rho_c = rec[b].rho_n, mean_c = rec[b].mean_n;
      const double rho_a = (double)na / (double)((int64_t)hia - (int64_t)rec[a].lo + 1);
      const double m_a = (double)Sa / (double)na;
      const uint64_t Ua = c >= 0 ? dbits(utility_cached(rho_a, m_a, rho_c, mean_c, p.eps)) : kInfBits;
      const uint64_t Upr = pr >= 0 ? dbits(utility_cached(rec[pr].rho, rec[pr].mean, rho_a, m_a, p.eps)) : kInfBits;
      if (lane == 0) {
        rec[a].n = na;
        rec[a].S = Sa;
        rec[a].hi = hia;
        rec[a].rho = rho_a;
        rec[a].mean = m_a;
        rec[a].rho_n = rho_c;
        rec[a].mean_n = mean_c;
        rec[a].nxt = c;
        rec[b].prv = -2;
        if (c >= 0) rec[c].prv = a;
        if (pr >= 0) {
          rec[pr].rho_n = rho_a;
          rec[pr].mean_n = m_a;
          U[pr] = Upr;
        }
        U[b] = kInfBits;
        U[a] = Ua;
      }
      // Lane 0's stores before anyone's next reads: LDS serves one wave in
      // order; the workspace needs a fence.
      if constexpr (!kInLds) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      // Cached minima that may be stale: a's owner (its minimum was a, now
      // Ua), b's owner if its minimum was b (now removed), pr's owner if its
      // minimum was pr (now Upr).  A value that improves a minimum is taken
      // directly; otherwise the owner's slots are rescanned.
      const int oa = a >> lgP, ob = b >> lgP, op = pr >= 0 ? pr >> lgP : -1;
      const bool lower_a = Ua < mu;  // still the global minimum: a keeps it
      bool stale = false;
      if (lane == oa) {
        if (lower_a) lane_u = Ua;  // lane_i == a already
        else stale = true;
      }
      if (lane == ob && lane_i == b) stale = true;
      if (lane == op) {
        if (Upr < lane_u || (Upr == lane_u && pr < lane_i)) {
          lane_u = Upr;
          lane_i = pr;
        } else if (lane_i == pr) {
          stale = true;
        }
      }
      uint64_t todo = __ballot(stale);
      while (todo != 0ull) {
        const int owner = (int)__builtin_ctzll(todo);
        todo &= todo - 1;
        rescan(owner);
      }
    }
  }
  __syncthreads();
  // Survivors in index (= length) order are the queues.
  const int per = (nl0 + kMergeThreads - 1) / kMergeThreads;
  const int i0 = tid * per;
  int cnt = 0;
  for (int q = 0; q < per; ++q)
    if (i0 + q < nl0 && rec[i0 + q].prv != -2) ++cnt;
  int tot = 0;
  int pos = block_exclusive_scan_n(cnt, iscr, &tot, kMergeThreads);
  for (int q = 0; q < per; ++q) {
    const int i = i0 + q;
    if (i < nl0 && rec[i].prv != -2) {
      const Leaf& r = rec[i];
      if (pos > 0) tab->bounds[pos - 1] = r.lo;
      tab->lo[pos] = r.lo;
      tab->hi[pos] = r.hi;
      tab->count[pos] = r.n;
      tab->sum[pos] = r.S;
      tab->mean[pos] = (double)r.S / (double)r.n;
      ++pos;
    }
  }
  if (tid == 0) tab->k = tot;
}

// The current queues (entries) of the chain merge: prefix sums (one more than
// entries) and intervals, the density and mean of each, the utility of each
// entry and the next, and the running minima of the utilities from the left
// (PM[i] = min U[0..i]) and from the right (SM[i] = min U[i..]).
struct ChainArrays {
  int64_t *N, *S;
  int32_t *lo, *hi;
  double *rho, *mean;
  uint64_t *U, *PM, *SM;
};
constexpr uint64_t kNoPair = ~0ull;  // above every utility's bits, +inf included

struct ChainLds {
  int64_t N[kLeafLds + 1], S[kLeafLds + 1];
  int32_t lo[kLeafLds], hi[kLeafLds];
  double rho[kLeafLds], mean[kLeafLds];
  uint64_t U[kLeafLds], PM[kLeafLds], SM[kLeafLds];
};
struct ListLds {
  Leaf rec[kLeafLds];
  uint64_t U[kLeafLds];
};
struct ChainState {
  uint64_t pmin[kWavesPerBlock], smin[kWavesPerBlock];
  double rho, mean;  // of the hot queue when its chain ended, and the utilities with its neighbours
  uint64_t ul, ur;
  int x, y;          // the hot queue is the union of entries x..y
  int alive;         // queues left
};

__device__ __forceinline__ uint64_t min_u64(uint64_t a, uint64_t b) { return a < b ? a : b; }

// One step of the wave scan below: the minimum with the value the DPP control
// brings (kNoPair where it brings none).
template <int kCtrl, int kRows>
__device__ __forceinline__ uint64_t dpp_min_u64(uint64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)(uint32_t)x, kCtrl, kRows, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)(uint32_t)(x >> 32), kCtrl, kRows, 0xF, false);
  return min_u64(x, ((uint64_t)hi << 32) | lo);
}

// Inclusive running minimum over the lanes, from lane 0 up (the steps of
// wave_incl_scan_add).
__device__ __forceinline__ uint64_t wave_incl_min_u64(uint64_t x) {
  x = dpp_min_u64<0x111, 0xF>(x);  // row_shr:1
  x = dpp_min_u64<0x112, 0xF>(x);  // row_shr:2
  x = dpp_min_u64<0x114, 0xF>(x);  // row_shr:4
  x = dpp_min_u64<0x118, 0xF>(x);  // row_shr:8
  x = dpp_min_u64<0x142, 0xA>(x);  // row_bcast:15
  x = dpp_min_u64<0x143, 0xC>(x);  // row_bcast:31
  return x;
}

// PM and SM from U[0..np), and st.x = the lowest pair, the leftmost of
// equals.  The whole block; a tile of PM from the left and the mirrored tile
// of SM from the right share their barriers, and each wave combines the waves'
// minima itself with one read and one scan.
__device__ void chain_minima(const ChainArrays& c, int np, ChainState& st) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  uint64_t pc = kNoPair, sc = kNoPair;
  for (int t0 = 0; t0 < np; t0 += kBlock) {
    const int i = t0 + tid, j = np - 1 - i;
    const uint64_t pm = wave_incl_min_u64(i < np ? c.U[i] : kNoPair);
    const uint64_t sm = wave_incl_min_u64(j >= 0 ? c.U[j] : kNoPair);
    if (lane == kWave - 1) {
      st.pmin[wv] = pm;
      st.smin[wv] = sm;
    }
    __syncthreads();
    const bool pl = lane < kWavesPerBlock;
    const uint64_t ps = wave_incl_min_u64(pl ? st.pmin[lane] : kNoPair);
    const uint64_t ss = wave_incl_min_u64(pl ? st.smin[lane] : kNoPair);
    const uint64_t pb = wv > 0 ? min_u64(pc, readlane_u64(ps, wv - 1)) : pc;  // before this wave
    const uint64_t sb = wv > 0 ? min_u64(sc, readlane_u64(ss, wv - 1)) : sc;
    pc = min_u64(pc, readlane_u64(ps, kWavesPerBlock - 1));
    sc = min_u64(sc, readlane_u64(ss, kWavesPerBlock - 1));
    const uint64_t here = min_u64(pb, pm);
    if (i < np) c.PM[i] = here;
    if (j >= 0) c.SM[j] = min_u64(sb, sm);
    if (np <= kBlock) {
      // One tile: pc is the lowest utility; the first place where the running
      // minimum reaches it.
      const uint64_t m = __ballot(i < np && here == pc);
      if (m != 0ull && pb != pc && lane == (int)__builtin_ctzll(m)) st.x = i;
    }
    __syncthreads();
  }
  if (np <= kBlock) return;
  for (int i = tid; i < np; i += kBlock)
    if (c.PM[i] == pc && (i == 0 || c.PM[i - 1] != pc)) st.x = i;
  __syncthreads();
}

// Entries x..x + d become entry x and the entries above move down by d
// places, m entries left; U is moved too (the merged entry's own U, rho and
// mean come from st).  The whole block: a tile of entries is read before it
// is written, and tiles go up, so no entry is overwritten before it moved.
__device__ void chain_compact(const ChainArrays& c, int x, int d, int m, const ChainState& st) {
  for (int t0 = x; t0 <= m; t0 += kBlock) {
    const int i = t0 + (int)threadIdx.x;  // N and S have one entry more
    int64_t N = 0, S = 0;
    int32_t lo = 0, hi = 0;
    double rho = 0.0, mean = 0.0;
    uint64_t U = 0;
    if (i <= m) {
      N = c.N[i + d];
      S = c.S[i + d];
    }
    if (i < m) {
      lo = c.lo[i + d];
      hi = c.hi[i + d];
      rho = c.rho[i + d];
      mean = c.mean[i + d];
    }
    if (i + 1 < m) U = c.U[i + d];
    __syncthreads();
    if (i == x) {  // its start stays
      c.hi[i] = hi;
      c.rho[i] = st.rho;
      c.mean[i] = st.mean;
      if (i + 1 < m) c.U[i] = st.ur;
      if (i > 0) c.U[i - 1] = st.ul;
    } else {
      if (i <= m) {
        c.N[i] = N;
        c.S[i] = S;
      }
      if (i < m) {
        c.lo[i] = lo;
        c.hi[i] = hi;
        c.rho[i] = rho;
        c.mean[i] = mean;
      }
      if (i + 1 < m) c.U[i] = U;
    }
    __syncthreads();
  }
}

// Merges until max_queues queues are left, or until the chains turn out
// short; returns the number of entries left (the queues, when it is at most
// max_queues).  The whole block; c holds nl > max_queues entries' N, S, lo, hi.
__device__ int chain_merge(const ChainArrays& c, int nl, const ewsjf_partition_params& p, ChainState& st) {
  const int tid = threadIdx.x;
  for (int i = tid; i < nl; i += kBlock) {
    const int64_t n = c.N[i + 1] - c.N[i], S = c.S[i + 1] - c.S[i];
    c.rho[i] = (double)n / (double)((int64_t)c.hi[i] - (int64_t)c.lo[i] + 1);
    c.mean[i] = (double)S / (double)n;
  }
  __syncthreads();
  for (int i = tid; i + 1 < nl; i += kBlock)
    c.U[i] = dbits(utility_cached(c.rho[i], c.mean[i], c.rho[i + 1], c.mean[i + 1], p.eps));
  __syncthreads();
  int m = nl;
  for (int chains = 1;; ++chains) {
    chain_minima(c, m - 1, st);
    if (tid < kWave) {
      int x = st.x, y = x + 1, left = m - 1;
      // st.x is read before a lane writes it again: one wave, in order
      bool go_left = true;
      while (left > p.max_queues) {
        // Lane j: the hot queue after j more merges on the current side.
        const int xj = x - (go_left ? tid : 0), yj = y + (go_left ? 0 : tid);
        const bool in = xj >= 0 && yj < m;
        const int a = in ? xj : x, b = in ? yj : y;
        const int64_t n = c.N[b + 1] - c.N[a], S = c.S[b + 1] - c.S[a];
        const double rho = (double)n / (double)((int64_t)c.hi[b] - (int64_t)c.lo[a] + 1);
        const double mean = (double)S / (double)n;
        const int al = a > 0 ? a - 1 : 0, br = b + 1 < m ? b + 1 : m - 1;
        const uint64_t ul = dbits(utility_cached(c.rho[al], c.mean[al], rho, mean, p.eps));
        const uint64_t ur = dbits(utility_cached(rho, mean, c.rho[br], c.mean[br], p.eps));
        const uint64_t UL = a > 0 ? ul : kNoPair, UR = b + 1 < m ? ur : kNoPair;
        const uint64_t PL = a >= 2 ? c.PM[a - 2] : kNoPair;      // the pairs left of its left neighbour
        const uint64_t PR = b + 2 < m ? c.SM[b + 1] : kNoPair;   // the pairs right of its right neighbour
        // the lowest pair is the one on its left / on its right (ties: the leftmost)
        const bool lo_l = in && UL != kNoPair && UL < PL && UL <= UR && UL <= PR;
        const bool lo_r = in && UR != kNoPair && UR < PL && UR < UL && UR <= PR;
        const uint64_t ml = __ballot(lo_l), mr = __ballot(lo_r);
        const uint64_t on = go_left ? ml : mr, off = go_left ? mr : ml;
        const int len = on == ~0ull ? kWave : (int)__builtin_ctzll(~on);
        const int run = min(len, left - p.max_queues);
        left -= run;
        if (go_left) x -= run;
        else y += run;
        if (len < kWave) {
          if (((off >> len) & 1ull) == 0ull) {  // another pair is the lowest: the chain ends
            if (tid == len) {                   // (read only when more merges are due, so run == len)
              st.rho = rho;
              st.mean = mean;
              st.ul = UL;
              st.ur = UR;
            }
            break;
          }
          go_left = !go_left;
        }
      }
      if (tid == 0) {
        st.x = x;
        st.y = y;
        st.alive = left;
      }
    }
    __syncthreads();
    const int x = st.x, d = st.y - x;
    m -= d;
    chain_compact(c, x, d, m, st);
    // A new chain costs about 2.5 us (the scans and the move), merge_list 0.75 us
    // a merge: chains pay from about four merges on.  Windows of the workloads
    // start with up to 20 short chains before their long one, so the first 32
    // are not judged; data without any chain loses about 0.1 ms here.
    if (m <= p.max_queues || (chains >= 32 && nl - m < 4 * chains)) return m;
  }
}

__global__ __launch_bounds__(kMergeThreads) void rp_merge(PartWs w, ewsjf_partition_params p,
                                                          ewsjf_queue_table* tab) {
  __shared__ union {
    ChainLds chain;
    ListLds list;
  } lds;
  __shared__ ChainState st;
  __shared__ int iscr[kMergeThreads / kWave];
  const int nl = w.meta[3];
  if (nl <= p.max_queues) return;  // rp_refine_prune wrote the queues
  const int tid = threadIdx.x;
  int m;
  if (nl <= kLeafLds) {
    ChainLds& cl = lds.chain;
    for (int i = tid; i <= nl; i += kBlock) {
      cl.N[i] = w.gN[i];
      cl.S[i] = w.gS[i];
      if (i < nl) {
        cl.lo[i] = w.glo[i];
        cl.hi[i] = w.ghi[i];
      }
    }
    __syncthreads();
    m = chain_merge(ChainArrays{cl.N, cl.S, cl.lo, cl.hi, cl.rho, cl.mean, cl.U, cl.PM, cl.SM}, nl, p, st);
    if (m <= p.max_queues) {
      write_queues(tab, m, cl.N, cl.S, cl.lo, cl.hi, tid, kBlock);
      return;
    }
    for (int i = tid; i <= m; i += kBlock) {
      w.gN[i] = cl.N[i];
      w.gS[i] = cl.S[i];
      if (i < m) {
        w.glo[i] = cl.lo[i];
        w.ghi[i] = cl.hi[i];
      }
    }
  } else {
    // five arrays of nl 8-byte entries in the room of nl records
    static_assert(sizeof(Leaf) >= 5 * 8, "the chain arrays fit the records");
    double* d = reinterpret_cast<double*>(w.grec);
    uint64_t* u = reinterpret_cast<uint64_t*>(d + 2 * (size_t)nl);
    m = chain_merge(ChainArrays{w.gN, w.gS, w.glo, w.ghi, d, d + nl, u, u + nl, u + 2 * (size_t)nl}, nl, p, st);
    if (m <= p.max_queues) {
      write_queues(tab, m, w.gN, w.gS, w.glo, w.ghi, tid, kBlock);
      return;
    }
  }
  __syncthreads();  // the chain arrays are done with (the records take their place)
  if (m <= kLeafLds)
    merge_list<true>(lds.list.rec, lds.list.U, w, m, p, tab, iscr);
  else
    merge_list<false>(w.grec, w.gU, w, m, p, tab, iscr);
}

size_t partition_ws_bytes(int64_t n_window, const ewsjf_partition_params& p) {
  return carve_size(n_window, p.max_len);
}

namespace {

// Stages 1-3 and the routing lut from the histogram w.hist (n_window < 0:
// the table records the histogram's total as the window size).
hipError_t launch_stages(const PartWs& w, const ewsjf_partition_params& p, int64_t n_window, ewsjf_queue_table* table,
                         hipStream_t stream) {
  const int L = p.max_len;
  hipLaunchKernelGGL(rp_distinct, dim3((L + kBlock - 1) / kBlock), dim3(kBlock), 0, stream, w, L);
  if (p.init_mode == EWSJF_INIT_KMEANS3) {
    hipLaunchKernelGGL(rp_km_corners, dim3(kKmCorners), dim3(kBlock), 0, stream, w);
    hipLaunchKernelGGL(rp_kmeans3, dim3(kKmeansBlocks), dim3(kBlock), 0, stream, w);
  }
  hipLaunchKernelGGL(rp_refine_prune, dim3(1), dim3(kBlock), 0, stream, w, p, n_window, table);
  hipLaunchKernelGGL(rp_merge, dim3(1), dim3(kMergeThreads), 0, stream, w, p, table);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_build_lut(table, stream);
}

}  // namespace

hipError_t launch_partition(const int32_t* window, int64_t n_window, const ewsjf_partition_params& p,
                            ewsjf_queue_table* table, void* ws, hipStream_t stream) {
  const int L = p.max_len;
  PartWs w = carve_part(ws, n_window, L);
  hipLaunchKernelGGL(window_hist, dim3(w.Gh), dim3(kBlock), 0, stream, window, n_window, L, w.partial);
  hipLaunchKernelGGL(hist_reduce, dim3((hist_row(L) / 4 + kReduceVecs - 1) / kReduceVecs),
                     dim3(kReduceVecs * kReduceRows), 0, stream, w.partial, w.Gh, L, w.hist_buf);
  return launch_stages(w, p, n_window, table, stream);
}

hipError_t launch_partition_hist(const uint32_t* hist, const ewsjf_partition_params& p, ewsjf_queue_table* table,
                                 void* ws, hipStream_t stream) {
  PartWs w = carve_part(ws, 0, p.max_len);
  w.hist = hist;
  return launch_stages(w, p, -1, table, stream);
}

hipError_t launch_window_histogram(const int32_t* ring, int64_t cap, int64_t begin, int64_t n, int L, uint32_t* hist,
                                   hipStream_t stream) {
  hipLaunchKernelGGL(hist_clear, dim3((L + 1 + 255) / 256), dim3(256), 0, stream, hist, L);
  if (n > 0)
    hipLaunchKernelGGL(window_hist_add, dim3(add_blocks(n)), dim3(kBlock), 0, stream, ring, cap, begin, n, L, hist);
  return hipGetLastError();
}

hipError_t launch_window_advance(const int32_t* ring, int64_t cap, int64_t add, int64_t sub, int64_t n, int L,
                                 uint32_t* hist, hipStream_t stream) {
  hipLaunchKernelGGL(window_hist_move, dim3(hist_blocks(n)), dim3(kBlock), 0, stream, ring, cap, add, sub, n, L,
                     hist);
  return hipGetLastError();
}

}  // namespace ewsjf
