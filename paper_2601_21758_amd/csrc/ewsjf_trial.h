// The statistics of a trial (Section 4.4.2) that the merge of each pool keeps.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ewsjf_device.h"
#include "ewsjf_merge.h"

namespace ewsjf {

enum {
  kAdmitted = 0,
  kTokens,
  kWaitSum,
  kWaitSqSum,
  kWaitMax,
  kPending,
  kPendingWaitMax,
  kSteps,
};
static_assert(kSteps + 1 == EWSJF_TRIAL_STATS, "statistics layout");

// Wait W = max(0, now - arrival) in binary64; a NaN arrival waits 0.
__device__ __forceinline__ double wait_of(float now, float a) {
  const double w = (double)now - (double)a;
  return w > 0.0 ? w : 0.0;
}

constexpr int kStatThreads = 256;

// The admitted requests ms.X[0..sel) of one pool (len, arrival: its slots)
// into its statistics st and its admissions per queue qa; then their slots are
// emptied.  The whole block calls it; its first kStatThreads threads sum, in a
// fixed order.  At the end of the merge it costs about 4.9 us; as a
// kernel of its own it read the admitted ids back and took 7.5 us and a launch.
__device__ __forceinline__ void trial_account(MergeShared& ms, int sel, int32_t* len, const float* arrival, float now,
                                              const ewsjf_queue_table* tab, double* st, int64_t* qa) {
  double* const rw = reinterpret_cast<double*>(ms.S);
  double* const rw2 = rw + kStatThreads;
  double* const rmax = rw2 + kStatThreads;
  int64_t* const rtok = reinterpret_cast<int64_t*>(rmax + kStatThreads);
  uint32_t* const qc = ms.cnt;
  static_assert(4 * kStatThreads * 8 <= (int)sizeof(ms.S) && EWSJF_MAX_QUEUES == kStatThreads, "room for the sums");
  const int tid = threadIdx.x;
  const bool on = tid < kStatThreads;
  const int k = tab->k, L = tab->max_len;
  const int64_t qa0 = on && tid < k ? qa[tid] : 0;
  const double st0 = tid < EWSJF_TRIAL_STATS ? st[tid] : 0.0;
  if (on) qc[tid] = 0u;
  __syncthreads();
  double w1 = 0.0, w2 = 0.0, wm = 0.0;
  int64_t tok = 0;
  if (on)
    for (int r = tid; r < sel; r += kStatThreads) {
      const uint32_t i = comp_id(ms.X[r]);
      const int b = len[i];  // admitted, so b >= 1
      const double w = wait_of(now, arrival[i]);
      w1 += w;
      w2 += w * w;
      wm = w > wm ? w : wm;
      tok += b;
      atomicAdd(&qc[tab->lut[b < L ? b : L]], 1u);
    }
  if (on) {
    rw[tid] = w1;
    rw2[tid] = w2;
    rmax[tid] = wm;
    rtok[tid] = tok;
  }
  __syncthreads();
  for (int s = kStatThreads / 2; s >= kWave; s >>= 1) {
    if (tid < s) {
      rw[tid] += rw[tid + s];
      rw2[tid] += rw2[tid + s];
      rmax[tid] = rmax[tid + s] > rmax[tid] ? rmax[tid + s] : rmax[tid];
      rtok[tid] += rtok[tid + s];
    }
    __syncthreads();
  }
  // every read of the admitted slots is done (barriers above): empty them
  for (int r = tid; r < sel; r += kBlock) len[comp_id(ms.X[r])] = 0;
  if (tid < kWave) {
    // the last wave's steps of the same tree, lane + s into lane
    w1 = rw[tid];
    w2 = rw2[tid];
    wm = rmax[tid];
    tok = rtok[tid];
    for (int s = kWave / 2; s > 0; s >>= 1) {
      w1 += __shfl_down(w1, s);
      w2 += __shfl_down(w2, s);
      const double o = __shfl_down(wm, s);
      wm = o > wm ? o : wm;
      tok += __shfl_down(tok, s);
    }
    // lane j keeps statistic j
    const double v1 = __shfl(w1, 0), v2 = __shfl(w2, 0), vm = __shfl(wm, 0), vt = (double)__shfl(tok, 0);
    const double add = tid == kAdmitted ? (double)sel : tid == kTokens ? vt : tid == kWaitSum ? v1 : tid == kWaitSqSum ? v2
                       : tid == kSteps ? 1.0 : 0.0;
    if (tid < EWSJF_TRIAL_STATS && tid != kPending && tid != kPendingWaitMax)
      st[tid] = tid == kWaitMax ? (vm > st0 ? vm : st0) : st0 + add;
  }
  if (on && tid < k && qc[tid]) qa[tid] = qa0 + (int64_t)qc[tid];
}

}  // namespace ewsjf
