// Routing lut construction, Dynamic Queue Routing and Density-Weighted
// Scoring kernels.
#include <hip/hip_runtime.h>

#include "ewsjf_device.h"
#include "ewsjf_launch.h"
#include "ewsjf_lut.h"

namespace ewsjf {

// lut[b] = the queue holding length b under the table's reading: the number
// of bounds <= b (contiguous cover; Section 3.2 Dispatcher), or the gapped
// rule of lo/hi (Section 4.3), and the compact routing map (the words that
// route_fill writes).  Bound by latency: the launch, one read of the queue
// starts and one search of them in LDS.  One length per thread, and a wave's
// 64 lengths are two words of the map, whose rises are one ballot; a thread
// per word walked its 32 lengths one after the other.  4.7 us, 8.3-9.2 us with
// the walks.
constexpr int kLutThreads = 256;
constexpr int kLutBlocks = (4 * kLutWords + kLutThreads - 1) / kLutThreads;  // 129
static_assert(kLutBlocks * kLutThreads >= 32 * kRouteWords, "every map word has its lanes");

__global__ __launch_bounds__(kLutThreads) void build_lut_kernel(ewsjf_queue_table* tab) {
  __shared__ int32_t bounds[EWSJF_MAX_QUEUES], lo[EWSJF_MAX_QUEUES], hi[EWSJF_MAX_QUEUES];
  static_assert(kLutThreads == EWSJF_MAX_QUEUES, "one queue per thread");
  bounds[threadIdx.x] = tab->bounds[threadIdx.x];
  lo[threadIdx.x] = tab->lo[threadIdx.x];
  hi[threadIdx.x] = tab->hi[threadIdx.x];
  const int L = tab->max_len, k = tab->k;
  const bool gapped = tab->gapped != 0;
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  const int x = blockIdx.x * kLutThreads + threadIdx.x;
  const int32_t *b = bounds, *l = lo, *h = hi;
  // the map's queue of length y: 0 below 1, that of L past L
  auto queue_at = [&](int y) { return (int)lut_entry(min(y, L), L, gapped, b, l, h, k); };
  const int q = queue_at(x), before = queue_at(x - lane - 1);  // of the length before the wave's
  const int up = __shfl_up(q, 1);
  const uint64_t rise = __ballot(q != (lane == 0 ? before : up));
  const int mid = __shfl(q, 31);
  if (x < 4 * kLutWords) tab->lut[x] = x <= L ? (uint8_t)q : (uint8_t)0;
  const int w = x >> 5;
  if ((lane & 31) == 0 && w < kRouteWords)
    tab->route[w] = ((uint64_t)(uint32_t)(lane == 0 ? before : mid) << 32) | (uint32_t)(rise >> lane);
}

hipError_t launch_build_lut(ewsjf_queue_table* table, hipStream_t stream) {
  hipLaunchKernelGGL(build_lut_kernel, dim3(kLutBlocks), dim3(kLutThreads), 0, stream, table);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Routing: qid[i] = queue of len[i] (-1 for an empty slot).  Bound by the
// launch and the staging of the table at a million requests (8 bytes each),
// by HBM beyond: the compact routing map is staged (8 KiB; the byte lut takes
// 32 KiB), and each thread's first loads are issued before it.
// 1,000,003 requests: 3.9 us, 4.5 us with the lut.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void stage_route(const ewsjf_queue_table* __restrict__ tab, uint64_t* route) {
  const i32x4* src = reinterpret_cast<const i32x4*>(tab->route);
  i32x4* dst = reinterpret_cast<i32x4*>(route);
  for (int i = threadIdx.x; i < kRouteWords / 2; i += blockDim.x) dst[i] = src[i];
}

__device__ __forceinline__ int route1(int b, int L, const uint64_t* route) {
  return b <= 0 ? -1 : route_queue(route, b < L ? b : L);
}

__global__ __launch_bounds__(kBlock) void route_kernel(const int32_t* __restrict__ len, int64_t n,
                                                       const ewsjf_queue_table* __restrict__ tab,
                                                       int32_t* __restrict__ qid) {
  __shared__ uint64_t route[kRouteWords];
  const int64_t nvec = n / 4;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  i32x4 b = v < nvec ? load_i32x4(len + 4 * v) : i32x4{0, 0, 0, 0};
  stage_route(tab, route);
  const int L = tab->max_len;
  __syncthreads();
  while (v < nvec) {
    const int64_t next = v + stride;
    const i32x4 bn = next < nvec ? load_i32x4(len + 4 * next) : b;
    i32x4 q;
    q.x = route1(b.x, L, route);
    q.y = route1(b.y, L, route);
    q.z = route1(b.z, L, route);
    q.w = route1(b.w, L, route);
    *reinterpret_cast<i32x4*>(qid + 4 * v) = q;
    b = bn;
    v = next;
  }
  for (int64_t i = nvec * 4 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride)
    qid[i] = route1(len[i], L, route);
}

// ---------------------------------------------------------------------------
// Streaming pool update: new requests into consecutive ring slots and their
// lengths into the window ring.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void ring_insert_kernel(int32_t* __restrict__ ring_len,
                                                          float* __restrict__ ring_arrival, int64_t capacity,
                                                          int64_t pos, int32_t* __restrict__ window,
                                                          int64_t window_cap, int64_t wpos,
                                                          const int32_t* __restrict__ new_len,
                                                          const float* __restrict__ new_arrival, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t b = new_len[i];
  int64_t slot = pos + i;
  if (slot >= capacity) slot -= capacity;  // n <= capacity and pos < capacity
  ring_len[slot] = b;
  ring_arrival[slot] = new_arrival[i];
  if (window_cap > 0) {
    int64_t w = wpos + i;
    if (w >= window_cap) w -= window_cap;  // n <= window_cap and wpos < window_cap
    window[w] = b;
  }
}

hipError_t launch_ring_insert(int32_t* ring_len, float* ring_arrival, int64_t capacity, int64_t pos, int32_t* window,
                              int64_t window_cap, int64_t wpos, const int32_t* new_len, const float* new_arrival,
                              int64_t n, hipStream_t stream) {
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(ring_insert_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, ring_len, ring_arrival,
                     capacity, pos, window, window_cap, wpos, new_len, new_arrival, n);
  return hipGetLastError();
}

hipError_t launch_route(const int32_t* len, int64_t n, const ewsjf_queue_table* table, int32_t* qid,
                        hipStream_t stream) {
  int64_t blocks = (n / 4 + kBlock - 1) / kBlock;
  if (blocks < 1) blocks = 1;
  if (blocks > 2 * kMaxGrid) blocks = 2 * kMaxGrid;
  hipLaunchKernelGGL(route_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, stream, len, n, table, qid);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scoring: score[t][i] = Phi of request i under parameter vector t.  A
// workgroup scores its requests under kScoreRows vectors: the route, the
// reciprocal and the log are the same for all of them, so a request is read
// and prepared once, and the table staged once, per group of vectors rather
// than per vector.  Bound by the 4 bytes written per request and vector.
// 1,000,003 requests under four vectors: 7.5 us, 11.6 us with a row per
// workgroup and the byte lut.
// ---------------------------------------------------------------------------
constexpr int kScoreRows = 8;

// Rows of an odd pool size start at any multiple of 4 bytes, all that a
// 16-byte vector store needs.
typedef f32x4 f32x4_row __attribute__((aligned(4)));

__device__ __forceinline__ float score1(int b, const QParams* qp, int q, const PhiTerms& x) {
  const float phi = phi_of(qp[q], x);
  return b <= 0 ? __builtin_nanf("") : phi != phi ? -__builtin_inff() : phi;
}

__global__ __launch_bounds__(kBlock) void score_kernel(const int32_t* __restrict__ len,
                                                       const float* __restrict__ arrival, int64_t n, float now,
                                                       const ewsjf_queue_table* __restrict__ tab,
                                                       const ewsjf_theta* __restrict__ theta, int n_theta, CostF cost,
                                                       float* __restrict__ score) {
  __shared__ uint64_t route[kRouteWords];
  __shared__ QParams qp[kScoreRows][EWSJF_MAX_QUEUES];
  const int t0 = blockIdx.y * kScoreRows, rows = min(kScoreRows, n_theta - t0);
  const int64_t nvec = n / 4;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  i32x4 b = i32x4{0, 0, 0, 0};
  f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
  if (v < nvec) {
    b = load_i32x4(len + 4 * v);
    a = load_f32x4(arrival + 4 * v);
  }
  stage_route(tab, route);
  const int L = tab->max_len, k = tab->k;
  for (int i = threadIdx.x; i < rows * EWSJF_MAX_QUEUES; i += kBlock) {
    const int r = i / EWSJF_MAX_QUEUES, q = i % EWSJF_MAX_QUEUES;
    if (q < k) qp[r][q] = make_qparams(theta[t0 + r], tab->mean[q], q);
  }
  __syncthreads();
  float* const out = score + (int64_t)t0 * n;
  auto queue = [&](int len1) { return max(route1(len1, L, route), 0); };  // an empty slot's is not used
  while (v < nvec) {
    const int64_t next = v + stride;
    i32x4 bn = b;
    f32x4 an = a;
    if (next < nvec) {
      bn = load_i32x4(len + 4 * next);
      an = load_f32x4(arrival + 4 * next);
    }
    int q[4];
    PhiTerms x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      q[e] = queue(b[e]);
      x[e] = phi_terms(b[e], a[e], now, cost);
    }
    for (int r = 0; r < rows; ++r) {
      f32x4 s;
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = score1(b[e], qp[r], q[e], x[e]);
      *reinterpret_cast<f32x4_row*>(out + (int64_t)r * n + 4 * v) = s;
    }
    b = bn;
    a = an;
    v = next;
  }
  for (int64_t i = nvec * 4 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride) {
    const int b1 = len[i];
    const PhiTerms x = phi_terms(b1, arrival[i], now, cost);
    for (int r = 0; r < rows; ++r) out[(int64_t)r * n + i] = score1(b1, qp[r], queue(b1), x);
  }
}

hipError_t launch_score(const int32_t* len, const float* arrival, int64_t n, float now,
                        const ewsjf_queue_table* table, const ewsjf_theta* theta, int32_t n_theta,
                        const ewsjf_cost& cost, float* score, hipStream_t stream) {
  int64_t blocks = (n / 4 + kBlock - 1) / kBlock;
  if (blocks < 1) blocks = 1;
  if (blocks > 2 * kMaxGrid) blocks = 2 * kMaxGrid;
  const CostF c{(float)cost.c0, (float)cost.c1, (float)cost.c2};
  hipLaunchKernelGGL(score_kernel, dim3((unsigned)blocks, (n_theta + kScoreRows - 1) / kScoreRows), dim3(kBlock), 0,
                     stream, len, arrival, n, now, table, theta, n_theta, c, score);
  return hipGetLastError();
}

}  // namespace ewsjf
