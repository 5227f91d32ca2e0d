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
// event.  2e5 four-body toys take 14 ms a call instead of 59; half a million
// three-body ones 282 us instead of 1031, a million mixing three-body ones 4.3
// ms instead of 15.9 (those two are made in two stages now, below).
#pragma once
#include "device_common.hpp"

namespace fn {

constexpr int kMaxPerWave = 128;  // events of a wave's run at most

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

// The same where an attempt is a cheap draw that often fails (a point outside
// the region) and a costly test of the points that are left: draws go on until
// 64 points wait for their test, so that its lanes are all in use.  A wave
// keeps at most 128 points, in the order of their attempts; an event whose
// attempt was accepted drops its later points when they come up, and one that
// ran out of attempts is decided by the points it still has.  draw(i, a, x, y)
// -> bool makes the point, test(i, a, x, y) -> bool decides it.
// Half a million three-body toys (half of the draws outside): 282 -> 234 us a
// call, 209 with the shorter region test, 185 with whole sets of points to a
// run's end too (its last events take draws they may not need: tests of 32 and
// then of single points there were slower); a million mixing ones 4.3 -> 3.1 ms,
// half a million 1.78 -> 1.47 ms with the latter, 1000 of the former 46 us (405
// with one event per lane).
struct StagedLds {
  int ev[kWaves][64], at[kWaves][64];       // open events and their next attempts
  int qe[kWaves][128], qa[kWaves][128];     // waiting points: event, attempt, place (a ring)
  double qx[kWaves][128], qy[kWaves][128];
  int win[kWaves][kMaxPerWave];             // accepting lane of the event, 64: none yet
};

template <class Draw, class Test, class Keep, class Fail>
__device__ __forceinline__ void accept_reject_staged(StagedLds& lds, int64_t n, int per_wave, int max_attempts,
                                                     Draw draw, Test test, Keep keep, Fail fail) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t first = ((int64_t)blockIdx.x * kWaves + wv) * per_wave;
  if (first >= n) return;
  const int count = (int)(n - first < per_wave ? n - first : per_wave);
  int* const pe = lds.ev[wv];
  int* const pa = lds.at[wv];
  int* const win = lds.win[wv];
  auto order = [] {  // the wave's LDS accesses on either side stay in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  int open = count < 64 ? count : 64;  // open events (the same in all lanes), next of the run to open
  int next = open;
  int head = 0, waiting = 0;  // the ring
  pe[lane] = lane;
  pa[lane] = 0;
  for (int e = lane; e < count; e += 64) win[e] = 64;
  // the open events that stay, packed, and new ones of the run in the free places
  auto refill = [&](bool stays, int e, int a) {
    const unsigned long long left = __ballot(stays);
    const int kept = __popcll(left), place = __popcll(left & ((1ull << lane) - 1ull));
    const int room = 64 - kept, rest = count - next;
    const int add = room < rest ? room : rest;
    order();
    if (stays) {
      pe[place] = e;
      pa[place] = a;
    }
    if (lane < add) {
      pe[kept + lane] = next + lane;
      pa[kept + lane] = 0;
    }
    next += add;
    open = kept + add;
    order();
  };
  while (open > 0 || waiting > 0) {
    // 2^sh lanes per open event: the most that 64 lanes give
    order();
    while (open > 0) {
      const int sh = open > 1 ? __builtin_clz(open - 1) - 26 : 6;
      const int slot = lane >> sh, sub = lane & ((1 << sh) - 1);
      const bool on = slot < open;
      const int e = on ? pe[slot] : 0, a = (on ? pa[slot] : 0) + sub;
      double x, y;
      const bool in = on && a < max_attempts && draw(first + e, a, x, y);
      const unsigned long long all = __ballot(in);
      const int q = (head + waiting + __popcll(all & ((1ull << lane) - 1ull))) & 127;
      if (in) {
        lds.qe[wv][q] = e;
        lds.qa[wv][q] = a;
        lds.qx[wv][q] = x;
        lds.qy[wv][q] = y;
      }
      waiting += __popcll(all);
      const bool speaks = on && sub == 0, stays = speaks && a + (1 << sh) < max_attempts;
      order();
      if (stays) pa[slot] = a + (1 << sh);
      if (__ballot(speaks != stays)) refill(stays, e, a + (1 << sh));
      order();
      if (waiting >= 64) break;
    }
    const int m = waiting < 64 ? waiting : 64;
    const int q = (head + lane) & 127;
    const int e = lane < m ? lds.qe[wv][q] : 0, a = lane < m ? lds.qa[wv][q] : 0;
    const double x = lane < m ? lds.qx[wv][q] : 0.0, y = lane < m ? lds.qy[wv][q] : 0.0;
    const bool ok = lane < m && win[e] == 64 && test(first + e, a, x, y);
    order();
    if (ok) atomicMin(&win[e], lane);
    order();
    if (ok && win[e] == lane) keep(first + e, x, y);
    head = (head + m) & 127;
    waiting -= m;
    if (__ballot(ok)) {
      const bool on = lane < open;
      const int oe = on ? pe[lane] : 0, oa = on ? pa[lane] : 0;
      refill(on && win[oe] == 64, oe, oa);
    }
  }
  for (int e = lane; e < count; e += 64)
    if (win[e] == 64) fail(first + e);
}

}  // namespace fn
