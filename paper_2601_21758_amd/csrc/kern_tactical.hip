// Tactical step (Algorithm 1, Section 3.2): the paper's own batch rule.
//
//   tac_scan    (G workgroups)  one pass over the pool: per queue, the number
//                               of pending requests and the oldest one (its
//                               head), per workgroup.
//   tac_reduce  (k workgroups)  per queue: the totals, and Phi of the head
//                               (Eq. 1 / Eq. 4) in binary64.
//   tac_plan    (1 workgroup)   empty counters, ArgMax queue, how many
//                               requests GreedyFill and Backfill take from the
//                               queue and its two neighbours.
//   queue-order selection       the oldest requests of each of the (up to)
//                               three queues.  tac_scan collects a sample,
//                               tac_reduce takes an age threshold per queue
//                               from it, tac_gather lists the members at or
//                               above it, tac_finish orders them.  For the
//                               largest B and pools (gather_rank):
//                               local_clustered / merge_candidates with
//                               FifoSource.
//   tac_finish  (1 workgroup,   the batch in order, tombstones, and the
//                a row each)    removal of queues empty past the threshold
//                               (re-absorbed by the neighbour of lower Eq. 3
//                               utility), with the routing lut rebuilt.
//
// Readings the paper leaves open (the oracle takes the same ones): a queue
// is a FIFO in arrival order (equal arrivals by id, NaN arrival last);
// ArgMax ties go to the lower queue; the two neighbours backfill in order of
// their head scores (ties: the lower queue first); empty counters count
// consecutive empty steps; removals apply after the batch is built, lowest
// index first, and the last queue is never removed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "ewsjf_device.h"
#include "ewsjf_launch.h"
#include "ewsjf_lut.h"
#include "ewsjf_merge.h"

namespace ewsjf {
namespace {

constexpr int kLutVecs = kLutBytes / 16;
constexpr int kReduceThreads = 256;
constexpr int kCountCopies = 8;        // of each queue's counter in tac_scan, by lane
constexpr int kSampledChunks = 65536;  // at most, two requests of each
constexpr int kSampleMax = 2 * kSampledChunks;
constexpr int kGatherLds = 4096;       // members of one row that one workgroup of tac_gather holds

// The oldest members of the plan's queues by an age threshold.
struct Gather {
  // Sample s sits at place sample_slot(s).
  uint32_t* skey;   // [kSampleMax] FIFO keys of the sampled requests (0 = empty slot)
  uint8_t* sq;      // [kSampleMax] their queues
  uint64_t* tau;    // [EWSJF_MAX_QUEUES] the queue's members at or above it hold its oldest B
  int32_t* count;   // [kTacticalRows] members found (more than kMergeCap: some were dropped)
  uint64_t* list;   // [kTacticalRows][kMergeCap]
  int lg_step;      // every 2^lg_step-th chunk is sampled
  int lg_p;         // 16 << lg_p places
  int n;            // samples, two per sampled chunk
  int rank;         // members of the sample the thresholds lie at; 0: not used
};

struct TacWs {
  uint32_t* part_cnt;   // [EWSJF_MAX_QUEUES][G]
  uint64_t* part_head;  // [EWSJF_MAX_QUEUES][G]: (arrival_key << 32) | id, ~0 = none
  uint32_t* cnt;        // [EWSJF_MAX_QUEUES]
  uint64_t* head;       // [EWSJF_MAX_QUEUES]
  float* score;         // [EWSJF_MAX_QUEUES]: Phi of the head, NaN if empty
  TacticalPlan* plan;
  int32_t* row_ids;     // [kTacticalRows][B]
  float* row_top;       // [kTacticalRows][B]
  int32_t* row_n;       // [kTacticalRows]
  Gather g;
  void* select_ws;
};

// One chunk per wave up to 1M requests, so that small pools use many compute
// units and one workgroup's share (4,096 requests there) always fits
// tac_gather's lists: 1M requests 37 / 35 us a step (random / arrival order)
// with four chunks per wave, 33 / 31 with one.
int scan_grid(int64_t n) {
  const int64_t nchunks = (n + kChunk - 1) / kChunk;
  int64_t G = (nchunks + kWavesPerBlock - 1) / kWavesPerBlock;
  if (G < 1) G = 1;
  if (G > kMaxGrid) G = kMaxGrid;
  return (int)G;
}

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// The sampled places of a chunk, by its number among the sampled chunks: at
// and 128 + at, at in 0..127.
__device__ __forceinline__ uint32_t sample_place(uint32_t i) { return i * 0x9E3779B1u >> 25; }

// Where sample s lies: place 16 v + j, thread v reading the 16 places from 16 v
// on, and back.  The thresholds come from maxima over the threads with one v mod
// 256, and two of the oldest in one group put a threshold deeper.  So samples
// next to each other fall into different groups (v follows s, and neighbours
// share cache lines), and so do samples a power of two apart: the high part of s
// and j are mixed in.  With v = s mod 2^lg_p, a queue that lives in every 256th
// chunk fell into two groups, its threshold let every member through, and one
// workgroup read the pool (4M requests: 2.0 ms; 41 us so).
__device__ __forceinline__ int sample_slot(int s, int lg_p) {
  const int j = s >> lg_p, low = s & ((1 << lg_p) - 1);
  return 16 * (low ^ (low >> 8) ^ (17 * j)) + j;
}
// vv: v ^ (v >> 8); 17 j lies below 256.
__device__ __forceinline__ int sample_of_slot(int vv, int j, int lg_p) { return (vv ^ (17 * j)) + (j << lg_p); }

int sample_step(int64_t n) {
  const int64_t nchunks = (n + kChunk - 1) / kChunk;
  int lg = 0;
  while (((nchunks + (1ll << lg) - 1) >> lg) > kSampledChunks) ++lg;  // the first chunk of an incomplete group counts
  return lg;
}

// The rank of a queue's age threshold among its sampled members, or 0 where the
// gather is not used.  The rank: the mean number of the B oldest in the sample
// (about a Poisson count), four standard deviations and a few more.  The
// members at or above the threshold (rank / density of them) must fit a
// workgroup's list with five standard deviations to spare, unless every queue
// fits it anyway: any B up to 9,088 requests, B up to 1,962 for pools up to
// 16,777,216 (every chunk sampled), up to 443 for pools up to 33,554,432 (every
// second), none beyond.  Measured (us a step, random / arrival order, gathered
// against the lists of FifoSource): 27 / 27 against 54 / 39 at 4,096 requests
// and B = 64, 29 / 29 against 55 / 60 at 65,536 and 64, 34 / 31 against 42 / 84
// at 1M and 1,024, 38 / 35 against 40 / 55 at 4M and 64, 53 / 51 against 56 / 73
// at 8M and 64, 80 / 77 against 86 / 114 at 16M and 64; with queues that
// overflow the lists up to 100 times as much.
int gather_rank(int64_t n, int32_t B) {
  const double density = 2.0 / ((double)kChunk * (double)(1 << sample_step(n)));
  const double mean = B * density;
  const int rank = (int)std::ceil(mean + 4.0 * std::sqrt(mean) + 8.0);
  return n <= kMergeCap || (rank + 5.0 * std::sqrt((double)rank)) / density <= kMergeCap ? rank : 0;
}

size_t carve_tac(int64_t n, int32_t B, void* ws, TacWs* w) {
  const int G = scan_grid(n);
  char* b = static_cast<char*>(ws);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* p = b ? b + o : nullptr;
    o += up256(bytes);
    return p;
  };
  TacWs t;
  t.part_cnt = reinterpret_cast<uint32_t*>(take((size_t)EWSJF_MAX_QUEUES * G * 4));
  t.part_head = reinterpret_cast<uint64_t*>(take((size_t)EWSJF_MAX_QUEUES * G * 8));
  t.cnt = reinterpret_cast<uint32_t*>(take(EWSJF_MAX_QUEUES * 4));
  t.head = reinterpret_cast<uint64_t*>(take(EWSJF_MAX_QUEUES * 8));
  t.score = reinterpret_cast<float*>(take(EWSJF_MAX_QUEUES * 4));
  t.plan = reinterpret_cast<TacticalPlan*>(take(sizeof(TacticalPlan)));
  t.row_ids = reinterpret_cast<int32_t*>(take((size_t)kTacticalRows * B * 4));
  t.row_top = reinterpret_cast<float*>(take((size_t)kTacticalRows * B * 4));
  t.row_n = reinterpret_cast<int32_t*>(take(kTacticalRows * 4));
  t.g.skey = reinterpret_cast<uint32_t*>(take(kSampleMax * sizeof(uint32_t)));
  t.g.sq = reinterpret_cast<uint8_t*>(take(kSampleMax));
  t.g.tau = reinterpret_cast<uint64_t*>(take(EWSJF_MAX_QUEUES * sizeof(uint64_t)));
  t.g.count = reinterpret_cast<int32_t*>(take(kTacticalRows * sizeof(int32_t)));
  t.g.list = reinterpret_cast<uint64_t*>(take((size_t)kTacticalRows * kMergeCap * sizeof(uint64_t)));
  t.g.lg_step = sample_step(n);
  t.g.n = 2 * (int)(((n + kChunk - 1) / kChunk + (1ll << t.g.lg_step) - 1) >> t.g.lg_step);
  t.g.lg_p = 10;  // at least one vector per thread: few samples are few per thread
  while ((16 << t.g.lg_p) < t.g.n) ++t.g.lg_p;
  t.g.rank = gather_rank(n, B);
  t.select_ws = take(plan_select(n, kTacticalRows, B).ws_bytes);
  if (w) *w = t;
  return o;
}

// ---------------------------------------------------------------------------
// Head-of-line pass.  Chunk c of workgroup w at local index lc is
// c = w + G * lc; each wave keeps four chunks in flight.  Counters are kept
// once per lane of eight: most requests of a workload fall in a few queues, and
// lanes adding to one counter are served one after the other (4M requests: 12.2
// us, 14.5 us with one counter per queue, the sample included).
//
// Two requests of every sampled chunk go to the sample, 128 slots apart, at a
// place of the chunk that varies from chunk to chunk.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void tac_scan(const int32_t* __restrict__ len, const float* __restrict__ arrival,
                                                   int64_t n, const ewsjf_queue_table* __restrict__ tab, int G,
                                                   uint32_t* __restrict__ part_cnt, uint64_t* __restrict__ part_head,
                                                   Gather g) {
  __shared__ uint8_t lut[kLutBytes];
  __shared__ uint32_t cnt[EWSJF_MAX_QUEUES * kCountCopies];
  __shared__ uint64_t head[EWSJF_MAX_QUEUES];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  {
    const i32x4* src = reinterpret_cast<const i32x4*>(tab->lut);
    i32x4* dst = reinterpret_cast<i32x4*>(lut);
    for (int i = tid; i < kLutVecs; i += kBlock) dst[i] = src[i];
  }
  for (int i = tid; i < EWSJF_MAX_QUEUES * kCountCopies; i += kBlock) cnt[i] = 0u;
  if (tid < EWSJF_MAX_QUEUES) head[tid] = ~0ull;
  const int L = tab->max_len, k = tab->k;
  __syncthreads();
  const int64_t nchunks = (n + kChunk - 1) / kChunk;
  const int copy = lane & (kCountCopies - 1);
  for (int64_t lc0 = wv;; lc0 += 4 * kWavesPerBlock) {
    const int64_t c0 = (int64_t)blockIdx.x + (int64_t)G * lc0;
    if (c0 >= nchunks) break;
    i32x4 l[4], a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // chunks past the end read zeros
      const int64_t first = ((int64_t)blockIdx.x + (int64_t)G * (lc0 + (int64_t)j * kWavesPerBlock)) * kChunk;
      l[j] = chunk_load_i32x4(chunk_rsrc(len + first, n - first), lane);
      a[j] = chunk_load_i32x4(chunk_rsrc(arrival + first, n - first), lane);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t c = (int64_t)blockIdx.x + (int64_t)G * (lc0 + (int64_t)j * kWavesPerBlock);
      const int64_t first = c * kChunk;
      // the sampled element of lanes with this low part, -1 elsewhere, and its place
      int pick = -1, place = 0;
      if (g.rank > 0 && c < nchunks && (c & ((1ll << g.lg_step) - 1)) == 0) {  // uniform
        const uint32_t i = (uint32_t)(c >> g.lg_step), at = sample_place(i);
        pick = (int)(at >> 2) == (lane & 31) ? (int)(at & 3u) : -1;
        place = sample_slot(2 * (int)i, g.lg_p) ^ ((lane >> 5) << 4);  // sample 2 i + lane / 32 differs in v's lowest bit
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int b = l[j][e];
        const int q = b > 0 ? (int)lut[min(b, L)] : 0xFFFF;
        const uint32_t ak = arrival_key(__int_as_float(a[j][e]));
        const uint32_t id = (uint32_t)(first + 4 * lane + e);
        if (b > 0) {
          atomicAdd(&cnt[q * kCountCopies + copy], 1u);
          const uint64_t hk = ((uint64_t)ak << 32) | (uint64_t)id;
          if (hk < head[q]) atomicMin(reinterpret_cast<unsigned long long*>(&head[q]), (unsigned long long)hk);
        }
        if (pick == e) {
          g.skey[place] = b > 0 ? ~ak : 0u;
          g.sq[place] = (uint8_t)q;
        }
      }
    }
  }
  __syncthreads();
  if (tid < k) {
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < kCountCopies; ++i) c += cnt[tid * kCountCopies + i];
    part_cnt[(size_t)tid * G + blockIdx.x] = c;
    part_head[(size_t)tid * G + blockIdx.x] = head[tid];
  }
}

// ---------------------------------------------------------------------------
// Per queue: totals over the workgroups, the head's score in binary64 (Eq. 1 /
// Eq. 4, the oracle's expression order; no contraction) and, for the gather,
// the age threshold.  Every queue's threshold is taken here, on as many compute
// units, before the plan knows the queues it needs: one workgroup reading the
// whole sample after the plan took 10 us more.
// ---------------------------------------------------------------------------
__device__ float head_phi(int32_t len, float arrival, float now, int q, double mean, const ewsjf_theta& th,
                          const ewsjf_cost& c) {
#pragma clang fp contract(off)
  const double m = mean;
  const double w_base = (double)th.a_base * m + (double)th.b_base;
  const double w_urg = (double)th.a_urg * m + (double)th.b_urg;
  const double w_fair = (double)th.a_fair * m + (double)th.b_fair;
  double W = (double)now - (double)arrival;
  if (!(W > 0.0)) W = 0.0;
  const double b = (double)len;
  const double C = c.c0 + c.c1 * b + c.c2 * b * b;
  const double cs = W / C;
  const double qf = (double)(q + 1) / (b + 1.0);
  const double phi = qf * ((w_base + w_urg * cs) + w_fair * log(b + 1.0));
  const float key = (float)phi;
  return key != key ? -__builtin_huge_valf() : key;
}

// The age threshold of a queue: the composite at the rank among its sampled
// members, taken from the maxima of 256 groups of samples (two of the oldest
// in one group put the threshold one place deeper).
constexpr int kPlanGroups = 4;  // groups per lane of the wave that searches

// A threshold that at least k of the wave's kPlanGroups x 64 composites reach:
// the k-th largest high word, with the low word resolved only where so many
// share that high word that it would let too many through; 1 (everything) when
// fewer than k are nonzero.
__device__ uint64_t wave_threshold(const uint64_t* x, int k) {
  uint32_t hi = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = hi | (1u << bit);
    int c = 0;
#pragma unroll
    for (int e = 0; e < kPlanGroups; ++e) c += (int)__popcll(__ballot((uint32_t)(x[e] >> 32) >= cand));
    if (c >= k) hi = cand;
  }
  if (hi == 0) return 1ull;
  int above = 0, same = 0;
#pragma unroll
  for (int e = 0; e < kPlanGroups; ++e) {
    above += (int)__popcll(__ballot((uint32_t)(x[e] >> 32) > hi));
    same += (int)__popcll(__ballot((uint32_t)(x[e] >> 32) == hi));
  }
  // (the pool may hold far more of an equal arrival than the groups show)
  if (same == 1) return (uint64_t)hi << 32;
  uint32_t lo = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = lo | (1u << bit);
    int c = above;
#pragma unroll
    for (int e = 0; e < kPlanGroups; ++e)
      c += (int)__popcll(__ballot((uint32_t)(x[e] >> 32) == hi && (uint32_t)x[e] >= cand));
    if (c >= k) lo = cand;
  }
  return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(kBlock) void tac_reduce(const uint32_t* __restrict__ part_cnt,
                                                     const uint64_t* __restrict__ part_head, int G,
                                                     const int32_t* __restrict__ len,
                                                     const float* __restrict__ arrival, float now,
                                                     const ewsjf_queue_table* __restrict__ tab,
                                                     const ewsjf_theta* __restrict__ theta, ewsjf_cost cost,
                                                     uint32_t* cnt, uint64_t* head, float* score, Gather g) {
  __shared__ uint32_t sc[kReduceThreads / kWave];
  __shared__ uint64_t sh[kReduceThreads / kWave];
  __shared__ uint64_t oldest[kBlock];
  const int q = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  if (q >= tab->k) return;  // uniform over the workgroup
  uint32_t c = 0;
  uint64_t h = ~0ull;
  for (int w = tid; w < G; w += kBlock) {
    c += part_cnt[(size_t)q * G + w];
    const uint64_t x = part_head[(size_t)q * G + w];
    h = x < h ? x : h;
  }
  c = __ockl_wfred_add_u32(c);
  h = wave_min_u64(h);
  if (lane == 0 && wv < kReduceThreads / kWave) {  // (the partials are at most one per thread of these)
    sc[wv] = c;
    sh[wv] = h;
  }
  __syncthreads();
  c = sc[0];
  h = sh[0];
#pragma unroll
  for (int i = 1; i < kReduceThreads / kWave; ++i) {
    c += sc[i];
    h = sh[i] < h ? sh[i] : h;
  }
  if (tid == kWave) {  // (not the wave that searches below)
    cnt[q] = c;
    head[q] = h;
    float s = __builtin_nanf("");
    if (c > 0) {
      const uint32_t id = (uint32_t)h;
      s = head_phi(len[id], arrival[id], now, q, tab->mean[q], theta[0], cost);
    }
    score[q] = s;
  }
  if (g.rank == 0) return;  // uniform
  if (c <= (uint32_t)kMergeCap) {  // uniform: all of them fit the list
    if (tid == 0) g.tau[q] = 1ull;
    return;
  }
  // The largest composite (the oldest) of this queue among each thread's
  // samples.
  uint64_t best = 0;
  const i32x4* kv = reinterpret_cast<const i32x4*>(g.skey);
  const i32x4* qv = reinterpret_cast<const i32x4*>(g.sq);
  for (int v = tid; v < (1 << g.lg_p); v += kBlock) {
    const int vv = v ^ (v >> 8);
    const i32x4 sq = qv[v];
    i32x4 key[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) key[u] = kv[4 * v + u];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int s = sample_of_slot(vv, 4 * u + e, g.lg_p);
        if (s < g.n && (int)(((uint32_t)sq[u] >> (8 * e)) & 0xFFu) == q && key[u][e] != 0) {
          const uint64_t x = make_comp((uint32_t)key[u][e], (uint32_t)s);  // (ids rise with s)
          best = x > best ? x : best;
        }
      }
  }
  if (best != 0ull) {
    const uint32_t s = comp_id(best), i = s >> 1;  // its chunk among the sampled ones
    const uint32_t id = ((i << g.lg_step) * (uint32_t)kChunk) + sample_place(i) + 128u * (s & 1u);
    best = make_comp((uint32_t)(best >> 32), id);
  }
  oldest[tid] = best;
  __syncthreads();
  if (wv == 0) {
    uint64_t m[kPlanGroups] = {};
#pragma unroll
    for (int e = 0; e < kWavesPerBlock; ++e) {
      const uint64_t o = oldest[e * kWave + lane];
      m[e % kPlanGroups] = o > m[e % kPlanGroups] ? o : m[e % kPlanGroups];
    }
    const uint64_t tau = wave_threshold(m, g.rank);
    if (lane == 0) g.tau[q] = tau;
  }
}

// ---------------------------------------------------------------------------
// The batch plan (one workgroup, one thread per queue).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EWSJF_MAX_QUEUES) void tac_plan(const ewsjf_queue_table* __restrict__ tab,
                                                             const uint32_t* __restrict__ cnt,
                                                             const float* __restrict__ score, int32_t B,
                                                             int32_t empty_threshold, int32_t* empty_cnt,
                                                             TacticalPlan* plan, int32_t* q_prim, float* head_score, Gather g) {
  __shared__ uint64_t wbest[EWSJF_MAX_QUEUES / kWave];
  __shared__ int nmark[EWSJF_MAX_QUEUES / kWave];
  __shared__ uint32_t qcnt[EWSJF_MAX_QUEUES];
  __shared__ float qscore[EWSJF_MAX_QUEUES];
  const int q = threadIdx.x, lane = q & (kWave - 1), wv = q / kWave;
  const int k = tab->k;
  const bool live = q < k;
  const uint32_t c = live ? cnt[q] : 0u;
  const float s = live ? score[q] : __builtin_nanf("");
  bool mark = false;
  qcnt[q] = c;
  qscore[q] = s;
  if (q < kTacticalRows) g.count[q] = 0;  // tac_gather's
  if (live) {
    const int ec = c > 0 ? 0 : empty_cnt[q] + 1;
    empty_cnt[q] = ec;
    mark = c == 0 && ec > empty_threshold;
    if (head_score) head_score[q] = s;
  }
  // ArgMax over the non-empty queues; equal scores go to the lower queue.
  const uint64_t key = c > 0 ? make_comp(ukey_of(s), (uint32_t)q) : 0ull;
  const uint64_t wm = wave_max_u64(key);
  const int nm = (int)__popcll(__ballot(mark));
  if (lane == 0) {
    wbest[wv] = wm;
    nmark[wv] = nm;
  }
  __syncthreads();
  if (q == 0) {
    uint64_t best = 0;
    int marks = 0;
    for (int i = 0; i < EWSJF_MAX_QUEUES / kWave; ++i) {
      best = wbest[i] > best ? wbest[i] : best;
      marks += nmark[i];
    }
    TacticalPlan p;
    p.k = k;
    p.n_removed = marks;
    p.pad = 0;
    for (int r = 0; r < kTacticalRows; ++r) {
      p.q_sel[r] = -1;
      p.take[r] = 0;
    }
    p.q_prim = best == 0 ? -1 : (int)comp_id(best);
    if (p.q_prim >= 0) {
      const int prim = p.q_prim;
      p.q_sel[0] = prim;
      int64_t left = B;
      const int64_t t0 = (int64_t)qcnt[prim] < left ? (int64_t)qcnt[prim] : left;
      p.take[0] = (int)t0;
      left -= t0;
      // Backfill: the non-empty neighbours, higher head score first.
      int nb[2], nn = 0;
      if (prim > 0 && qcnt[prim - 1] > 0) nb[nn++] = prim - 1;
      if (prim + 1 < k && qcnt[prim + 1] > 0) nb[nn++] = prim + 1;
      if (nn == 2 && qscore[nb[1]] > qscore[nb[0]]) {
        const int x = nb[0];
        nb[0] = nb[1];
        nb[1] = x;
      }
      for (int i = 0; i < nn; ++i) {
        const int64_t ti = (int64_t)qcnt[nb[i]] < left ? (int64_t)qcnt[nb[i]] : left;
        p.q_sel[1 + i] = nb[i];
        p.take[1 + i] = (int)ti;
        left -= ti;
      }
    }
    *plan = p;
    *q_prim = p.q_prim;
  }
}

// ---------------------------------------------------------------------------
// The members of the plan's queues at or above their thresholds, one pass over
// the pool (four chunks in flight).  Bound by HBM and, behind it, by the handling
// of what arrives: a wave's requests are tested for age first, and routed only
// where one of them is old enough.  4M requests: 8.6 us (3.9 TB/s), 10.2 us with
// every request routed; tac_finish orders the 2,000 to 4,500 members in 5 us more
// than it took.  The lists of local_clustered took 16.9 us and their merge 24 to
// 40 us, since the oldest of a queue sit together in a pool in arrival order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void tac_gather(const int32_t* __restrict__ len, const float* __restrict__ arrival,
                                                     int64_t n, const ewsjf_queue_table* __restrict__ tab, int G,
                                                     const TacticalPlan* __restrict__ plan, Gather g) {
  __shared__ uint64_t route[kRouteWords];
  __shared__ uint64_t out[kTacticalRows][kGatherLds];
  __shared__ int nout[kTacticalRows], base[kTacticalRows];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  const i32x4* lsrc = reinterpret_cast<const i32x4*>(tab->route);
  for (int i = tid; i < kRouteWords / 2; i += kBlock) reinterpret_cast<i32x4*>(route)[i] = lsrc[i];
  const int L = tab->max_len;
  int qs[kTacticalRows];
  uint64_t tau[kTacticalRows];
#pragma unroll
  for (int r = 0; r < kTacticalRows; ++r) {
    qs[r] = plan->take[r] > 0 ? plan->q_sel[r] : -2;  // no request's queue
    tau[r] = qs[r] >= 0 ? g.tau[qs[r]] : ~0ull;
  }
  // The least key any row takes: most requests are younger and need no route.
  uint32_t min_key = ~0u;
#pragma unroll
  for (int r = 0; r < kTacticalRows; ++r) min_key = min(min_key, (uint32_t)(tau[r] >> 32));
  if (tid < kTacticalRows) nout[tid] = 0;
  __syncthreads();
  const int64_t nchunks = (n + kChunk - 1) / kChunk;
  auto pass = [&](auto some) {  // some: not every age is taken
    for (int64_t lc0 = wv;; lc0 += 4 * kWavesPerBlock) {
      const int64_t c0 = (int64_t)blockIdx.x + (int64_t)G * lc0;
      if (c0 >= nchunks) break;
      i32x4 l[4], a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // chunks past the end read zeros
        const int64_t first = (c0 + (int64_t)G * kWavesPerBlock * j) * kChunk;
        l[j] = chunk_load_i32x4(chunk_rsrc(len + first, n - first), lane);
        a[j] = chunk_load_i32x4(chunk_rsrc(arrival + first, n - first), lane);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t first = (c0 + (int64_t)G * kWavesPerBlock * j) * kChunk;
        if (first >= n) break;  // uniform
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int b = l[j][e];
          const uint32_t key = fifo_key(__int_as_float(a[j][e]));
          if (decltype(some)::value && __ballot(b > 0 && key >= min_key) == 0ull) continue;  // uniform
          const int q = b > 0 ? route_queue(route, min(b, L)) : -1;
          const uint64_t x = make_comp(key, (uint32_t)(first + 4 * lane + e));
          int row = -1;
#pragma unroll
          for (int r = 0; r < kTacticalRows; ++r) row = q == qs[r] && x >= tau[r] ? r : row;  // the rows' queues differ
          if (__ballot(row >= 0) != 0ull) {
            for (int r = 0; r < kTacticalRows; ++r) {
              const uint64_t m = __ballot(row == r);
              if (m == 0ull) continue;
              int at = 0;
              if (lane == 0) at = atomicAdd(&nout[r], (int)__popcll(m));
              at = __builtin_amdgcn_readfirstlane(at);  // lane 0 (the whole wave is active)
              const int i = at + lanes_below(m);
              if (row == r && i < kGatherLds) out[r][i] = x;
              if (at + (int)__popcll(m) > kGatherLds) {  // uniform; most of a queue's oldest in one share
                const uint64_t past = __ballot(row == r && i >= kGatherLds);
                int to = 0;
                if (lane == 0) to = atomicAdd(&g.count[r], (int)__popcll(past));
                to = __builtin_amdgcn_readfirstlane(to) + lanes_below(past);
                if (row == r && i >= kGatherLds && to < kMergeCap) g.list[(size_t)r * kMergeCap + to] = x;
              }
            }
          }
        }
      }
    }
  };
  if (min_key != 0u) pass(std::true_type{});
  else pass(std::false_type{});
  __syncthreads();
  if (tid < kTacticalRows && nout[tid] > 0) base[tid] = atomicAdd(&g.count[tid], min(nout[tid], kGatherLds));
  __syncthreads();
  for (int r = 0; r < kTacticalRows; ++r) {
    const int c = min(nout[r], kGatherLds);
    for (int i = tid; i < c; i += kBlock)
      if (base[r] + i < kMergeCap) g.list[(size_t)r * kMergeCap + base[r] + i] = out[r][i];
  }
}

// Whether row r's listed members hold its oldest `take`: always, but for about
// one call in a million, and for pools laid out against the sample's places.
__device__ __forceinline__ bool row_listed(const Gather& g, int r, int take) {
  const int U = g.count[r];
  return U >= take && U <= kMergeCap;
}

// The oldest `take` of row r into ms.X, oldest first, by the whole block: from
// the listed members, or (exact) from the whole pool, sixteen chunks at a time,
// a load and three barriers each: 2.0 ms for 4M requests.
__device__ void oldest_of_row(MergeShared& ms, const Gather& g, int r, int queue, int take, const int32_t* len,
                              const float* arrival, int64_t n, const ewsjf_queue_table* tab) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  if (row_listed(g, r, take)) {  // uniform
    const int U = g.count[r];
    constexpr int kR = (kMergeCap + kBlock - 1) / kBlock;
    uint64_t v[kR];
#pragma unroll
    for (int i = 0; i < kR; ++i) v[i] = tid + i * kBlock < U ? g.list[(size_t)r * kMergeCap + tid + i * kBlock] : 0ull;
    uint64_t unused;
    rank_registers(ms, v, U, take, 0ull, &unused);
    return;
  }
  const int L = tab->max_len;
  const int64_t nchunks = (n + kChunk - 1) / kChunk;
  int have = 0;
  uint64_t low = 1ull;
  for (int64_t c0 = 0; c0 < nchunks; c0 += kWavesPerBlock) {
    if (tid == 0) ms.cntS = 0;
    __syncthreads();
    const int64_t first = (c0 + wv) * kChunk;
    const i32x4 l = chunk_load_i32x4(chunk_rsrc(len + first, n - first), lane);
    const i32x4 a = chunk_load_i32x4(chunk_rsrc(arrival + first, n - first), lane);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int b = l[e];
      if (b > 0 && route_queue(tab->route, min(b, L)) == queue) {
        const uint64_t x = make_comp(fifo_key(__int_as_float(a[e])), (uint32_t)(first + 4 * lane + e));
        if (x >= low) ms.S[atomicAdd(&ms.cntS, 1)] = x;  // at most kSortMax a round
      }
    }
    __syncthreads();
    have = merge_new(ms, have, ms.cntS, take);
    __syncthreads();
    low = have >= take ? ms.X[take - 1] : 1ull;
  }
}


// ---------------------------------------------------------------------------
// The batch, tombstones, and queue removal.
// ---------------------------------------------------------------------------
__device__ double eq3_utility(int64_t na, int64_t Sa, int32_t loa, int32_t hia, int64_t nb, int64_t Sb, int32_t lob,
                              int32_t hib, double eps) {
#pragma clang fp contract(off)
  const double rho_a = (double)na / (double)((int64_t)hia - (int64_t)loa + 1);
  const double rho_b = (double)nb / (double)((int64_t)hib - (int64_t)lob + 1);
  const double m_a = (double)Sa / (double)na;
  const double m_b = (double)Sb / (double)nb;
  return (rho_a + rho_b) / (fabs(m_b - m_a) + eps);
}

__global__ __launch_bounds__(kBlock) void tac_finish(const TacticalPlan* __restrict__ plan,
                                                     const int32_t* __restrict__ row_ids, int32_t B,
                                                     int32_t* tomb_len, int32_t* ids, int32_t* n_sel,
                                                     ewsjf_queue_table* tab, const uint32_t* __restrict__ cnt,
                                                     int32_t empty_threshold, int32_t* empty_cnt, double eps,
                                                     int32_t* removed, Gather g, const int32_t* len,
                                                     const float* arrival, int64_t n) {
  __shared__ MergeShared ms;
  __shared__ int64_t qn[EWSJF_MAX_QUEUES], qS[EWSJF_MAX_QUEUES];
  __shared__ int32_t qlo[EWSJF_MAX_QUEUES], qhi[EWSJF_MAX_QUEUES], qec[EWSJF_MAX_QUEUES], qorig[EWSJF_MAX_QUEUES];
  __shared__ int32_t qb[EWSJF_MAX_QUEUES];  // bounds: qb[i] separates queues i and i + 1
  __shared__ uint8_t qmark[EWSJF_MAX_QUEUES];
  __shared__ int k2s;
  const int tid = threadIdx.x;
  const TacticalPlan p = *plan;
  const int t0 = p.take[0], t1 = p.take[1], t2 = p.take[2];
  if (g.rank > 0) {
    // A workgroup per row; the first goes on.  Rows that need the whole pool are
    // all taken by the first, which rewrites the table only afterwards.
    int at = 0;
    for (int r = 0; r < kTacticalRows; ++r) {
      const int take = p.take[r];
      const int owner = r > 0 && row_listed(g, r, take) ? r : 0;
      if (take > 0 && (int)blockIdx.x == owner) {  // uniform
        oldest_of_row(ms, g, r, p.q_sel[r], take, len, arrival, n, tab);
        for (int i = tid; i < take; i += kBlock) {
          const int id = (int)comp_id(ms.X[i]);
          ids[at + i] = id;
          if (tomb_len != nullptr) tomb_len[id] = 0;  // (no member of another row's queue)
        }
        __syncthreads();
      }
      at += take;
    }
    if (blockIdx.x > 0) return;
    for (int i = at + tid; i < B; i += kBlock) ids[i] = -1;
  } else {
    for (int r = tid; r < B; r += kBlock) {
      int id = -1;
      if (r < t0) id = row_ids[r];
      else if (r < t0 + t1) id = row_ids[B + (r - t0)];
      else if (r < t0 + t1 + t2) id = row_ids[2 * B + (r - t0 - t1)];
      ids[r] = id;
      if (tomb_len != nullptr && id >= 0) tomb_len[id] = 0;
    }
  }
  if (tid == 0) *n_sel = t0 + t1 + t2;
  const int k = p.k;
  if (removed != nullptr && tid < k) removed[tid] = 0;
  if (p.n_removed == 0 || k == 1) return;  // uniform: no barrier skipped by part of the block

  // Sequential removal on an LDS copy of the queue list (k <= 256).
  if (tid < k) {
    qn[tid] = tab->count[tid];
    qS[tid] = tab->sum[tid];
    qlo[tid] = tab->lo[tid];
    qhi[tid] = tab->hi[tid];
    qec[tid] = empty_cnt[tid];
    qorig[tid] = tid;
    qmark[tid] = cnt[tid] == 0 && empty_cnt[tid] > empty_threshold;
    if (tid + 1 < k) qb[tid] = tab->bounds[tid];
  }
  __syncthreads();
  if (tid == 0) {
    int kk = k;
    for (;;) {
      int r = -1;
      for (int i = 0; i < kk; ++i)
        if (qmark[i]) {
          r = i;
          break;
        }
      if (r < 0 || kk == 1) break;
      int a;
      if (r == 0) a = 1;
      else if (r + 1 == kk) a = r - 1;
      else
        a = eq3_utility(qn[r - 1], qS[r - 1], qlo[r - 1], qhi[r - 1], qn[r], qS[r], qlo[r], qhi[r], eps) <=
                    eq3_utility(qn[r], qS[r], qlo[r], qhi[r], qn[r + 1], qS[r + 1], qlo[r + 1], qhi[r + 1], eps)
                ? r - 1
                : r + 1;
      qn[a] += qn[r];
      qS[a] += qS[r];
      qlo[a] = min(qlo[a], qlo[r]);
      qhi[a] = max(qhi[a], qhi[r]);
      if (removed != nullptr) removed[qorig[r]] = 1;
      for (int i = min(r, a); i + 2 < kk; ++i) qb[i] = qb[i + 1];  // the boundary between r and a goes
      for (int i = r; i + 1 < kk; ++i) {
        qn[i] = qn[i + 1];
        qS[i] = qS[i + 1];
        qlo[i] = qlo[i + 1];
        qhi[i] = qhi[i + 1];
        qec[i] = qec[i + 1];
        qorig[i] = qorig[i + 1];
        qmark[i] = qmark[i + 1];
      }
      --kk;
    }
    k2s = kk;
  }
  __syncthreads();
  const int k2 = k2s;
  if (tid < k2) {
    tab->count[tid] = qn[tid];
    tab->sum[tid] = qS[tid];
    tab->lo[tid] = qlo[tid];
    tab->hi[tid] = qhi[tid];
    tab->mean[tid] = (double)qS[tid] / (double)qn[tid];
    if (tid > 0) tab->bounds[tid - 1] = qb[tid - 1];
    empty_cnt[tid] = qec[tid];
  }
  if (tid == 0) tab->k = k2;
  // Routing lut of the new set, in the table's reading (contiguous bounds or
  // gapped intervals).
  const int L = tab->max_len;
  const bool gapped = tab->gapped != 0;
  lut_fill(tab->lut, tid, kBlock, L, gapped, qb, qlo, qhi, k2);
  route_fill(tab->route, tid, kBlock, L, gapped, qb, qlo, qhi, k2);
}

}  // namespace

size_t tactical_ws_bytes(int64_t n, int32_t B) { return carve_tac(n, B, nullptr, nullptr); }

hipError_t launch_tactical_step(int32_t* len, const float* arrival, int64_t n, float now, ewsjf_queue_table* table,
                                const ewsjf_theta* theta, const ewsjf_cost& cost, int32_t B, int32_t empty_threshold,
                                int32_t* empty_cnt, double eps, int32_t* tomb_len, int32_t* ids, int32_t* n_sel,
                                int32_t* q_prim, float* head_score, int32_t* removed, void* ws, hipStream_t stream) {
  TacWs w;
  carve_tac(n, B, ws, &w);
  const int G = scan_grid(n);
  hipLaunchKernelGGL(tac_scan, dim3(G), dim3(kBlock), 0, stream, len, arrival, n, table, G, w.part_cnt, w.part_head,
                     w.g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tac_reduce, dim3(EWSJF_MAX_QUEUES), dim3(w.g.rank > 0 ? kBlock : kReduceThreads), 0, stream,
                     w.part_cnt, w.part_head, G, len, arrival, now, table, theta, cost, w.cnt, w.head, w.score, w.g);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(tac_plan, dim3(1), dim3(EWSJF_MAX_QUEUES), 0, stream, table, w.cnt, w.score, B, empty_threshold,
                     empty_cnt, w.plan, q_prim, head_score, w.g);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (w.g.rank > 0) {
    hipLaunchKernelGGL(tac_gather, dim3(G), dim3(kBlock), 0, stream, len, arrival, n, table, G, w.plan, w.g);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else if ((e = launch_fifo_select(len, arrival, n, table, w.plan, B, w.row_ids, w.row_top, w.row_n, w.select_ws,
                                     stream)) != hipSuccess) {
    return e;
  }
  hipLaunchKernelGGL(tac_finish, dim3(w.g.rank > 0 ? kTacticalRows : 1), dim3(kBlock), 0, stream, w.plan, w.row_ids, B, tomb_len, ids, n_sel, table,
                     w.cnt, empty_threshold, empty_cnt, eps, removed, w.g, len, arrival, n);
  return hipGetLastError();
}

#ifdef EWSJF_STAMPS
// Instrumented build only: the sizes of a step's sample, and where its
// workspace keeps the rows' member counts.
void debug_tactical(int64_t n, int32_t B, int64_t* out) {
  char* const base = reinterpret_cast<char*>((uintptr_t)256);  // for offsets only
  TacWs w;
  carve_tac(n, B, base, &w);
  out[0] = w.g.rank;
  out[1] = w.g.lg_step;
  out[2] = w.g.n;
  out[3] = 16ll << w.g.lg_p;
  out[4] = kSampleMax;
  out[5] = reinterpret_cast<char*>(w.g.count) - base;
  out[6] = kMergeCap;
}
#endif

}  // namespace ewsjf

#ifdef EWSJF_STAMPS
extern "C" void ewsjf_debug_tactical(int64_t n, int32_t B, int64_t* out) { ewsjf::debug_tactical(n, B, out); }
#endif
