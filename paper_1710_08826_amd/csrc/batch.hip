// Many fits of one mix1d model per launch, with a device-resident minimizer.
//
// One batch step = one NLL + gradient evaluation for every running fit at its
// trial point, followed by one state-machine step of BFGS with a strong-Wolfe
// line search (Nocedal & Wright, Alg. 3.5/3.6) per fit:
//
//   batch_head    per running fit: theta_trial -> mix1d table; in one more
//                 workgroup: exclusive scan of the running fits' chunk counts
//                 -> item bases, total item count, running-fit count
//   batch_eval    persistent kernel over (fit, chunk) items; each item runs
//                 the single-fit chunk routine, so rows are bitwise those of
//                 fn_nll for the same fit
//   batch_tail    one workgroup per running fit: fixed-order level-2 sum ->
//                 NLL, gradient; then accept/reject the trial, update H, pick
//                 the next trial point, or retire (converged / failed)
//
// Launches of a few microseconds each (table 5.3, scan 4.1, level 2 3.9,
// minimizer 9.2: threads of one wave took the phases of their fits one after
// the other, from device memory) were a third of a step of 512 fits; in two
// launches, each fit's minimizer in its own workgroup on a copy in LDS, they
// take 5.6 and 7.0 (up to 12 with numerical Hessians under way, 18 before).
//
// No host synchronisation inside a step; the host polls the running-fit
// count between groups of steps.  Fits never interact, so a fit's trajectory
// (and result bits) is the same alone and inside any batch.
#include <cmath>

#include "batch.hpp"
#include "philox.hpp"

namespace fn {

// Toy events of the Gaussian + exponential mixture on [lo, hi] (theta_gen =
// mu, sigma, tau, f): component by a uniform draw, Gaussian by Box-Muller with
// redraws outside the range, exponential by the inverse CDF of the truncated
// exponential.  Event i, attempt a uses counters (i, 2a, word) and (i, 2a+1, word).
// NaN when no attempt lands in the range.
__device__ __forceinline__ double gen_mix1d_event(int64_t i, uint32_t k0, uint32_t k1, uint32_t word, double mu,
                                                  double sigma, double tau, double frac, double lo, double hi) {
  const double width = hi - lo;
  const double em = tau != 0.0 ? expm1(tau * width) : 0.0;
  for (int a = 0; a < kGenMaxAttempts; ++a) {
    double uc, u1, u2, unused;
    philox_uniforms((uint64_t)i, 2u * a, word, k0, k1, uc, u1);
    philox_uniforms((uint64_t)i, 2u * a + 1u, word, k0, k1, u2, unused);
    double t;
    if (uc < frac) {
      const double r = sqrt(-2.0 * log1p(-u1));
      t = mu + sigma * r * cos(2.0 * 3.14159265358979323846 * u2);
    } else {
      t = tau != 0.0 ? lo + log1p(u1 * em) / tau : lo + u1 * width;
      t = fmin(fmax(t, lo), hi);
    }
    if (t >= lo && t <= hi) return t;
  }
  return NAN;
}

__global__ void gen_mix1d_kernel(uint32_t k0, uint32_t k1, uint32_t word, int64_t n, double mu, double sigma,
                                 double tau, double frac, double lo, double hi, double* __restrict__ x,
                                 unsigned int* __restrict__ n_unresolved) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double v = gen_mix1d_event(i, k0, k1, word, mu, sigma, tau, frac, lo, hi);
  x[i] = v;
  if (v != v) atomicAdd(n_unresolved, 1u);
}

// ------------------------------------------------------------- admission
static_assert(sizeof(BfgsState) % sizeof(uint64_t) == 0, "state is cleared in 8-byte words");

__global__ __launch_bounds__(kBlock) void batch_admit(const AdmitRec* __restrict__ recs, int n_recs, int P,
                                                      double lo, double hi, BatchDev b,
                                                      unsigned int* __restrict__ n_unresolved) {
  const int64_t blk = blockIdx.x;
  if (blk < n_recs) {
    // a fresh fit: every field zero but the start point, the free mask, status and phase
    const AdmitRec& r = recs[blk];
    uint64_t* w = reinterpret_cast<uint64_t*>(b.st + r.slot);
    constexpr int kWords = (int)(sizeof(BfgsState) / sizeof(uint64_t));
    for (int i = threadIdx.x; i < kWords; i += blockDim.x) w[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
      BfgsState& st = b.st[r.slot];
      for (int i = 0; i < P; ++i) {
        st.xt[i] = r.theta0[i];
        st.mask[i] = 1;
      }
      st.status = kFitRunning;
      st.phase = kPhaseStart;
      b.stat[r.slot] = kFitRunning;
      b.ev[r.slot] = r.ev;
      b.nev[r.slot] = r.n;
    }
    return;
  }
  // generation workgroup g: the last record with block0 <= g owns it (records
  // without generation own no workgroups, so a later record with the same
  // block0 is the owner)
  const int64_t g = blk - n_recs;
  int a = 0, c = n_recs - 1;
  while (a < c) {
    const int mid = (a + c + 1) / 2;
    if (recs[mid].block0 <= g) a = mid;
    else c = mid - 1;
  }
  const AdmitRec& r = recs[a];
  const int64_t i = (g - r.block0) * kBlock + threadIdx.x;
  if (!r.generate || i >= r.n) return;
  const double v = gen_mix1d_event(i, r.seed, r.fit, 0u, r.theta_gen[0], r.theta_gen[1], r.theta_gen[2],
                                   r.theta_gen[3], lo, hi);
  r.ev[i] = v;
  if (v != v) atomicAdd(n_unresolved, 1u);
}

// fn_batch_set: workgroup f resets slot f -- a fresh fit at theta0[f] (all
// parameters free) for f < n_fits, idle beyond; its event pointer and count come
// from the host's staging arrays (pinned, read in place: 16 bytes a slot).
__global__ __launch_bounds__(kBlock) void batch_set_kernel(const double* __restrict__ theta0,
                                                           const double* const* __restrict__ h_ev,
                                                           const int64_t* __restrict__ h_nev, int n_fits, int P,
                                                           BatchDev b) {
  const int f = blockIdx.x;
  uint64_t* w = reinterpret_cast<uint64_t*>(b.st + f);
  constexpr int kWords = (int)(sizeof(BfgsState) / sizeof(uint64_t));
  for (int i = threadIdx.x; i < kWords; i += blockDim.x) w[i] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    if (f < n_fits) {
      BfgsState& st = b.st[f];
      for (int i = 0; i < P; ++i) {
        st.xt[i] = theta0[(int64_t)f * P + i];
        st.mask[i] = 1;
      }
      st.status = kFitRunning;
      st.phase = kPhaseStart;
    }
    b.stat[f] = f < n_fits ? kFitRunning : kFitIdle;
    b.ev[f] = h_ev[f];
    b.nev[f] = h_nev[f];
  }
}

void batch_launch_set(const BatchDev& b, const double* theta0, const double* const* h_ev, const int64_t* h_nev,
                      int n_fits, int max_fits, int P, hipStream_t s) {
  hipLaunchKernelGGL(batch_set_kernel, dim3((unsigned)max_fits), dim3(kBlock), 0, s, theta0, h_ev, h_nev, n_fits, P,
                     b);
}

__global__ void batch_gather_rows(const double* __restrict__ rres, const int* __restrict__ slots, int n, int w,
                                  double* __restrict__ rows) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)n * w) return;
  const int i = (int)(t / w), j = (int)(t - (int64_t)i * w);
  rows[t] = rres[(int64_t)slots[i] * w + j];
}

// ------------------------------------------------------------------ steps
__device__ __forceinline__ int64_t chunks_of(const ChunkRule& rule, int64_t n) {
  const int c = rule(n);
  return (n + c - 1) / c;
}

// One workgroup: item_base[f] = sum of chunk counts of running fits < f;
// item_base[n_fits] = total; *n_running = number of running fits (in host
// memory, where the host reads it once the stream is idle).  Thread t
// takes a contiguous run of fits; the exclusive scan of the per-thread sums
// (thread order) is a shuffle scan within each wave plus the totals of the
// preceding waves: exact integer sums, the same as a serial loop.
__device__ inline void batch_scan(const int* __restrict__ stat, const int64_t* __restrict__ nev, int n_fits,
                                  const ChunkRule& rule, int64_t* __restrict__ item_base, int* __restrict__ n_running) {
  constexpr int kWaves = kBlock / 64;
  __shared__ int64_t wsum[kWaves];
  __shared__ int wcnt[kWaves];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int per = (n_fits + kBlock - 1) / kBlock;
  const int f0 = min(t * per, n_fits), f1 = min(f0 + per, n_fits);
  int64_t s = 0;
  int c = 0;
#pragma unroll 4
  for (int f = f0; f < f1; ++f) {
    if (stat[f] == kFitRunning) {
      s += chunks_of(rule, nev[f]);
      ++c;
    }
  }
  int64_t x = s;
  int cx = c;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t y = __shfl_up(x, d, 64);
    const int cy = __shfl_up(cx, d, 64);
    if (lane >= d) {
      x += y;
      cx += cy;
    }
  }
  if (lane == 63) {
    wsum[w] = x;
    wcnt[w] = cx;
  }
  __syncthreads();
  int64_t before = 0;
  for (int u = 0; u < w; ++u) before += wsum[u];
  if (t == kBlock - 1) {
    int total = 0;
    for (int u = 0; u < kWaves; ++u) total += wcnt[u];
    item_base[n_fits] = before + x;
    *n_running = total;
  }
  int64_t b = before + x - s;
#pragma unroll 4
  for (int f = f0; f < f1; ++f) {
    item_base[f] = b;
    if (stat[f] == kFitRunning) b += chunks_of(rule, nev[f]);
  }
}

// Workgroup 0 scans; the others make the tables of 64 fits each, component k
// in wave k % 4 (different shapes in one wave would run one after the other).
__global__ __launch_bounds__(kBlock) void batch_head(Mix1dConst mc, const BfgsState* __restrict__ st,
                                                     const int* __restrict__ stat, const int64_t* __restrict__ nev,
                                                     int n_fits, ChunkRule rule, Mix1dTable* __restrict__ tabs,
                                                     int64_t* __restrict__ item_base, int* __restrict__ n_running) {
  if (blockIdx.x == 0) {
    batch_scan(stat, nev, n_fits, rule, item_base, n_running);
    return;
  }
  __shared__ int bad[64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int f = ((int)blockIdx.x - 1) * 64 + lane;
  const bool run = f < n_fits && stat[f] == kFitRunning;
  if (w == 0) bad[lane] = 0;
  __syncthreads();
  if (run) {
    for (int k = w; k < mc.K; k += kBlock / 64)
      if (!mix1d_component(mc, st[f].xt, k, tabs[f])) bad[lane] = 1;
  }
  __syncthreads();
  if (run && w == 0) mix1d_table_rest(mc, st[f].xt, bad[lane] == 0, tabs[f]);
}

// The fit f >= lo with item_base[f] <= it < item_base[f+1] (fits that don't run
// have empty ranges, so the search lands on a running one).  The wave looks at
// 64 entries per round: two dependent loads for 4096 fits.
__device__ __forceinline__ int fit_of_item(const int64_t* __restrict__ item_base, int64_t it, int lo, int n_fits) {
  const int lane = threadIdx.x & 63;
  int hi = n_fits;  // invariant: item_base[lo] <= it < item_base[hi]
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6;
    const int i = lo + lane * step;
    const int below = __popcll(__ballot(i < hi && item_base[i < hi ? i : lo] <= it));
    lo += (below - 1) * step;
    hi = min(lo + step, hi);
  }
  return lo;
}

// Each workgroup takes one contiguous run of items (sizes differ by one at
// most), so it looks for its fit once and then walks on.  One item at a time,
// each with its own binary search, left the workgroups waiting: a step of 512
// fits of 1e3 to 2e5 events (19M in all), 74 -> 62 us.  Bound by a chunk's
// fixed part (four events per thread, then the row's sum): handing runs out
// from a counter (2.13 -> 2.60 ms for the whole set of fits: the counter's
// atomics), requesting the next chunk's events ahead and shorter sums of the
// row were no faster.
template <bool GRAD, int KMAX, int SIG>
__global__ __launch_bounds__(kBlock) void batch_eval(Mix1dConst mc, const Mix1dTable* __restrict__ tabs,
                                                     const double* const* __restrict__ ev,
                                                     const int64_t* __restrict__ nev,
                                                     const int64_t* __restrict__ item_base,
                                                     const int64_t* __restrict__ part_base, int n_fits, ChunkRule rule,
                                                     double* __restrict__ part) {
  constexpr int NV = GRAD ? mix_nv(KMAX) : 1;
  __shared__ double lds[block_sum_lds(NV)];
  const int64_t total = item_base[n_fits];
  const int64_t each = total / gridDim.x;
  const int more = (int)(total - each * gridDim.x);  // workgroups with one item more
  const int b = blockIdx.x;
  int64_t it = b * each + min(b, more);
  const int64_t last = it + each + (b < more ? 1 : 0);
  int f = 0;
  while (it < last) {
    f = fit_of_item(item_base, it, f, n_fits);
    const int64_t base = item_base[f], stop = min(last, item_base[f + 1]);
    const int64_t n = nev[f];
    const int chunk = rule(n);
    const double* x = ev[f];
    double* rows = part + part_base[f] * NV;
    for (; it < stop; ++it) {
      mix1d_chunk<GRAD, KMAX, SIG>(mc, tabs + f, x, n, it - base, chunk, rows + (it - base) * NV, lds);
      __syncthreads();
    }
    ++f;
  }
}

// Level 2 and the minimizer step of fit blockIdx.x.  The state's words are
// requested before the rows, so that both come back together; thread 0 works on
// them in LDS and registers.
template <int PC>
__global__ __launch_bounds__(kBlock) void batch_tail(Mix1dConst mc, const Mix1dTable* __restrict__ tabs,
                                                     const int64_t* __restrict__ nev,
                                                     const int64_t* __restrict__ part_base,
                                                     const double* __restrict__ part, ChunkRule rule, int nv, int kmax,
                                                     double tol, int max_iter, BfgsState* __restrict__ st,
                                                     int* __restrict__ stat, double* __restrict__ rres) {
  __shared__ double scratch[kBlock], res[kBlock], out[2 + 2 * kBatchMaxP];
  __shared__ BfgsState m;
  const int f = blockIdx.x, t = threadIdx.x;
  if (stat[f] != kFitRunning) return;
  const int P = PC > 0 ? PC : mc.n_params;
  const int W = bfgs_words<kBatchMaxP>(P);
  double word = 0.0;
  int num = 0;
  if (t < W) word = *bfgs_word(st[f], P, t);
  if (t < P + 8) num = *bfgs_int(st[f], P, t);
  mix1d_finalize_one(mc, tabs[f], part + part_base[f] * nv, chunks_of(rule, nev[f]), nv, kmax, 1, (double)nev[f], out,
                     nullptr, scratch, res);
  if (t < W) *bfgs_word(m, P, t) = word;
  if (t < P + 8) *bfgs_int(m, P, t) = num;
  for (int w = t + kBlock; w < W; w += kBlock) *bfgs_word(m, P, w) = *bfgs_word(st[f], P, w);
  __syncthreads();
  if (t == 0) {
    bfgs_step_one<kBatchMaxP, PC>(m, out, P, tol, max_iter);
    if (m.status != kFitRunning) {
      write_result(m, P, rres + (int64_t)f * (3 + 2 * P));
      stat[f] = m.status;
    }
  }
  __syncthreads();
  for (int w = t; w < W; w += kBlock) *bfgs_word(st[f], P, w) = *bfgs_word(m, P, w);
  if (t < P + 8) *bfgs_int(st[f], P, t) = *bfgs_int(m, P, t);
}

// Every slot's [status, NLL, iterations, evaluations, theta(P), sqrt|H_ii|(P)].
__global__ __launch_bounds__(kBlock) void batch_collect(const BfgsState* __restrict__ st, int n, int P,
                                                        double* __restrict__ rows) {
  const int w = 4 + 2 * P;
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (t >= (int64_t)n * w) return;
  const int f = (int)(t / w), j = (int)(t - (int64_t)f * w);
  const BfgsState& s = st[f];
  double v;
  if (j == 0) v = s.status;
  else if (j == 1) v = s.f;
  else if (j == 2) v = s.iter;
  else if (j == 3) v = s.n_eval;
  else if (j < 4 + P) v = s.x[j - 4];
  else {
    const int i = j - 4 - P;
    v = s.mask[i] ? sqrt(fabs(s.Hm(i, i))) : 0.0;
  }
  rows[t] = v;
}

// ---------------------------------------------------------------- launchers
void batch_launch_gen_mix1d(uint32_t k0, uint32_t k1, uint32_t word, int64_t n, const double* theta_gen, double lo,
                            double hi, double* x, unsigned int* n_unresolved, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(gen_mix1d_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, k0, k1, word, n,
                     theta_gen[0], theta_gen[1], theta_gen[2], theta_gen[3], lo, hi, x, n_unresolved);
}

void batch_launch_admit(const BatchDev& b, const AdmitRec* recs, int n_recs, int64_t gen_blocks, int P, double lo,
                        double hi, unsigned int* n_unresolved, hipStream_t s) {
  if (n_recs == 0) return;
  hipLaunchKernelGGL(batch_admit, dim3((unsigned)(n_recs + gen_blocks)), dim3(kBlock), 0, s, recs, n_recs, P, lo, hi,
                     b, n_unresolved);
}

void batch_launch_gather_rows(const BatchDev& b, const int* slots, int n, int P, double* rows_out, hipStream_t s) {
  if (n == 0) return;
  const int w = 3 + 2 * P;
  const int64_t total = (int64_t)n * w;
  hipLaunchKernelGGL(batch_gather_rows, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, b.rres, slots, n, w,
                     rows_out);
}

void batch_launch_step(const BatchDev& b, const Mix1dConst& mc, int n_fits, int P, ChunkRule rule, int eval_grid,
                       double tol, int max_iter, hipStream_t s) {
  const int kmax = mix1d_kmax(mc.K);
  const int nv = mix1d_nv(kmax, true);
  hipLaunchKernelGGL(batch_head, dim3(1 + (n_fits + 63) / 64), dim3(kBlock), 0, s, mc, b.st, b.stat, b.nev, n_fits,
                     rule, b.tabs, b.item_base, b.n_running);
#define FN_EVAL(K, SIG)                                                                               \
  hipLaunchKernelGGL((batch_eval<true, K, SIG>), dim3(eval_grid), dim3(kBlock), 0, s, mc, b.tabs, b.ev, b.nev, \
                     b.item_base, b.part_base, n_fits, rule, b.part)
#define FN_EVAL_SIG(SIG) \
  case SIG:              \
    FN_EVAL(2, SIG);     \
    break;
  switch (mix1d_sig(mc)) {
    FN_MIX_SIGS(FN_EVAL_SIG)
    default:
      if (kmax == 4) FN_EVAL(4, 0);
      else FN_EVAL(8, 0);
  }
#undef FN_EVAL_SIG
#undef FN_EVAL
#define FN_TAIL_P(PC)                                                                                        \
  case PC:                                                                                                  \
    hipLaunchKernelGGL((batch_tail<PC>), dim3(n_fits), dim3(kBlock), 0, s, mc, b.tabs, b.nev, b.part_base,  \
                       b.part, rule, nv, kmax, tol, max_iter, b.st, b.stat, b.rres);                        \
    break;
  switch (P <= 8 ? P : 0) {
    FN_TAIL_P(1)
    FN_TAIL_P(2)
    FN_TAIL_P(3)
    FN_TAIL_P(4)
    FN_TAIL_P(5)
    FN_TAIL_P(6)
    FN_TAIL_P(7)
    FN_TAIL_P(8)
    FN_TAIL_P(0)
  }
#undef FN_TAIL_P
}

void batch_launch_collect(const BatchDev& b, int n, int P, double* rows, hipStream_t s) {
  const int64_t total = (int64_t)n * (4 + 2 * P);
  hipLaunchKernelGGL(batch_collect, dim3((unsigned)((total + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, b.st, n, P,
                     rows);
}

int batch_eval_blocks_per_cu(const Mix1dConst& mc) {
  int nb = 0;
#define FN_OCC_SIG(SIG)                                                                     \
  case SIG:                                                                                 \
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_eval<true, 2, SIG>, kBlock, 0); \
    break;
  switch (mix1d_sig(mc)) {
    FN_MIX_SIGS(FN_OCC_SIG)
    default:
      if (mix1d_kmax(mc.K) == 4)
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_eval<true, 4, 0>, kBlock, 0);
      else
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_eval<true, 8, 0>, kBlock, 0);
  }
#undef FN_OCC_SIG
  return nb > 0 ? nb : 1;
}

}  // namespace fn
