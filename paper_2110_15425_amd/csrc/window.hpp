// window.hpp -- finished runs counted in LDS.
//
// A workgroup's runs are contiguous (setting-major), so they span few
// settings: their histograms and counters fit in LDS, and the global ones take
// one atomic per nonzero word and workgroup.  Counting each run straight into
// global memory is the fallback where the window does not fit (`direct`): the
// words of one setting share a few cache lines, and 64-bit atomics on those from
// all eight XCDs follow one another (about 3 ns each: 400,000 of them held a
// closed-loop sweep of 80,000 runs at 1.3 ms whatever its arithmetic).
#pragma once

#include "internal.hpp"

namespace cm {
namespace {

// One finished run -- setting s, trial t, decision step n (executed steps when
// choice is -1), target: its correct response -- into the window lds, whose first
// setting is s_lo, or into global memory; and its optional dumps.  A: the
// kernel's arguments (hist, stats, n_bins, steps_magic, trials, direct, run_*).
template <class A>
__device__ __forceinline__ void count_run(const A& a, uint32_t* lds, uint32_t s_lo, uint32_t s, uint32_t t,
                                          uint32_t steps, int c, int target, bool flag, const double* state,
                                          int width) {
  const uint64_t n = steps;
  if (a.direct) {
    uint64_t* st = a.stats + (uint64_t)s * CM_NSTAT;
    if (c >= 0) {
      const uint32_t bin = udiv_magic((steps - 1u) * a.n_bins, a.steps_magic);
      atomicAdd((unsigned long long*)&a.hist[((uint64_t)s * 2u + c) * a.n_bins + bin], 1ull);
      atomicAdd((unsigned long long*)&st[CM_ST_DEC0 + c], 1ull);
      atomicAdd((unsigned long long*)&st[CM_ST_SUMN0 + c], (unsigned long long)n);
      atomicAdd((unsigned long long*)&st[CM_ST_SUMSQ0 + c], (unsigned long long)(n * n));
      if (c == target) atomicAdd((unsigned long long*)&st[CM_ST_CORRECT], 1ull);
    } else {
      atomicAdd((unsigned long long*)&st[CM_ST_UNDEC], 1ull);
    }
    if (flag) atomicAdd((unsigned long long*)&st[CM_ST_FLAGGED], 1ull);
  } else {
    const uint32_t B = a.n_bins;
    uint32_t* rec = lds + (s - s_lo) * rec_words(B);
    uint32_t* cnt = rec + 2u * B;
    unsigned long long* sums = (unsigned long long*)(cnt + kCntWords);
    if (c >= 0) {
      const uint32_t bin = udiv_magic((steps - 1u) * B, a.steps_magic);
      atomicAdd(&rec[c * B + bin], 1u);
      atomicAdd(&cnt[kCntDec0 + c], 1u);
      if (c == target) atomicAdd(&cnt[kCntCorrect], 1u);
      atomicAdd(&sums[c], (unsigned long long)n);
      atomicAdd(&sums[2 + c], (unsigned long long)(n * n));
    } else {
      atomicAdd(&cnt[kCntUndec], 1u);
    }
    if (flag) atomicAdd(&cnt[kCntFlagged], 1u);
  }
  if (a.run_choice) {
    const uint64_t idx = (uint64_t)s * a.trials + t;
    a.run_choice[idx] = (int8_t)c;
    a.run_step[idx] = steps;
    a.run_flag[idx] = flag ? 1 : 0;
    if (a.run_state)
      for (int i = 0; i < width; ++i) a.run_state[idx * width + i] = state[i];
  }
}

// The window into the global histogram and statistics (the whole workgroup).
template <class A>
__device__ void flush_window(const A& a, const uint32_t* lds, uint32_t s_lo) {
  const uint32_t B = a.n_bins, per = 2u * B + CM_NSTAT, rw = rec_words(B);
  for (uint32_t i = threadIdx.x; i < a.window * per; i += blockDim.x) {
    const uint32_t w = i / per, j = i - w * per;
    const uint64_t sg = (uint64_t)s_lo + w;
    if (sg >= a.n_settings) continue;
    const uint32_t* rec = lds + w * rw;
    const uint32_t* cnt = rec + 2u * B;
    const unsigned long long* sums = (const unsigned long long*)(cnt + kCntWords);
    unsigned long long v;
    unsigned long long* dst;
    if (j < 2u * B) {
      v = rec[j];
      dst = (unsigned long long*)&a.hist[sg * 2u * B + j];
    } else {
      const uint32_t k = j - 2u * B;
      switch (k) {
        case CM_ST_DEC0: v = cnt[kCntDec0]; break;
        case CM_ST_DEC1: v = cnt[kCntDec1]; break;
        case CM_ST_UNDEC: v = cnt[kCntUndec]; break;
        case CM_ST_CORRECT: v = cnt[kCntCorrect]; break;
        case CM_ST_SUMN0: v = sums[0]; break;
        case CM_ST_SUMN1: v = sums[1]; break;
        case CM_ST_SUMSQ0: v = sums[2]; break;
        case CM_ST_SUMSQ1: v = sums[3]; break;
        default: v = cnt[kCntFlagged]; break;
      }
      dst = (unsigned long long*)&a.stats[sg * CM_NSTAT + k];
    }
    if (v) atomicAdd(dst, v);
  }
}

}  // namespace
}  // namespace cm
