// Accept-reject generation by waves: event i is decided by its own attempts a =
// 0, 1, ... (counter-based draws), whichever lane makes them, so a wave may try
// an event's attempts in any order and side by side as long as the first
// accepted one is kept.
//
// With one event per lane a wave runs until its unluckiest lane is done: at 5 %
// acceptance 92 rounds for 64 events that need 20 each.  Here a wave owns a
// run of events and holds up to 64 open ones in LDS (event, next attempt);
// accepted events are replaced by the next of the run, and once fewer are left
// than half the lanes, 2, 4, ... 64 lanes try consecutive attempts of one
// event.  Half a million three-body toys take 282 us a
// call instead of 1031, 1000 of them 49 instead of 405; a million mixing
// three-body ones 4.3 ms instead of 15.9, 2e5 four-body ones 14 instead of 59.
#pragma once
#include "device_common.hpp"

namespace fn {

struct AcceptLds {
  int ev[kWaves][64], at[kWaves][64];
};

// Wave w of the launch decides events [w per_wave, (w + 1) per_wave) below n.
// attempt(i, a) -> bool makes one attempt (its outcome in the caller's
// variables); keep(i) stores the accepted outcome of the lane that calls it;
// fail(i) handles an event without one among max_attempts.  All lanes of a
// wave stay together; no workgroup barrier.
template <class Attempt, class Keep, class Fail>
__device__ __forceinline__ void accept_reject(AcceptLds& lds, int64_t n, int per_wave, int max_attempts,
                                              Attempt attempt, Keep keep, Fail fail) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t first = ((int64_t)blockIdx.x * kWaves + wv) * per_wave;
  if (first >= n) return;
  const int count = (int)(n - first < per_wave ? n - first : per_wave);
  int* const pe = lds.ev[wv];
  int* const pa = lds.at[wv];
  auto order = [] {  // the wave's LDS accesses on either side stay in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  int open = count < 64 ? count : 64;  // open events (the same in all lanes), next of the run to open
  int next = open;
  pe[lane] = lane;
  pa[lane] = 0;
  while (open > 0) {
    order();
    // 2^sh lanes per open event: the most that 64 lanes give
    const int sh = open > 1 ? __builtin_clz(open - 1) - 26 : 6;
    const int slot = lane >> sh, sub = lane & ((1 << sh) - 1);
    const bool on = slot < open;
    const int e = on ? pe[slot] : 0, a0 = on ? pa[slot] : 0;
    const bool ok = on && a0 + sub < max_attempts && attempt(first + e, a0 + sub);
    const unsigned long long all = __ballot(ok);
    const unsigned long long mine = (all >> (slot << sh)) & (sh == 6 ? ~0ull : (1ull << (1 << sh)) - 1ull);
    if (ok && sub == __builtin_ctzll(mine)) keep(first + e);
    const bool head = on && sub == 0 && mine == 0;  // speaks for an event still without an accepted attempt
    const bool stays = head && a0 + (1 << sh) < max_attempts;
    if (head && !stays) fail(first + e);
    const unsigned long long left = __ballot(stays);
    const int kept = __popcll(left), place = __popcll(left & ((1ull << lane) - 1ull));
    const int room = 64 - kept, rest = count - next;
    const int add = room < rest ? room : rest;
    order();
    if (stays) {
      pe[place] = e;
      pa[place] = a0 + (1 << sh);
    }
    if (lane < add) {
      pe[kept + lane] = next + lane;
      pa[kept + lane] = 0;
    }
    next += add;
    open = kept + add;
  }
}

}  // namespace fn
