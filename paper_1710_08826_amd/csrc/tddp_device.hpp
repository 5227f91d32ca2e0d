// Device code of the time-dependent three-body Dalitz-plot model with mixing
// (the paper's pi+ pi- pi0 time-dependent amplitude fit, Sec. 1 Table 2 and
// Fig. 2), compiled at run time for each model structure like the
// time-integrated three-body passes.
//
// Daughters 2 and 3 are charge conjugates (m2 = m3), so the Dbar0 amplitude
// at (s12, s13) is the D0 one at (s13, s12):
//   A = sum_k c_k A_k(s12, s13),  Abar = sum_k cbar_k A_k(s13, s12),
// with A_k the isobar amplitudes of dalitz_device.hpp (fixed lineshapes), and
// the rate is the mixing and resolution form of td4_device.hpp:
//   R = 1/2 [(|A|^2+|Abar|^2) Hc + (|A|^2-|Abar|^2) Hcos - 2 Re(A* Abar) Hs - 2 Im(A* Abar) Hsin].
// The normalization is the grid integral of the t-integrated rate, a
// quadratic form in (c, cbar) through three K x K matrices of grid sums,
//   MAA_ij = dA sum A_i conj(A_j),  MBB_ij = dA sum B_i conj(B_j),
//   MAB_ij = dA sum conj(A_i) B_j,  B_k(s12, s13) = A_k(s13, s12),
// built once per model (the lineshapes are fixed).
#pragma once
#include "dalitz_device.hpp"
#include "td4_device.hpp"

namespace fn {

// Decay-time constants of a model: 1/tau, the resolution width, the time
// functions' constants and the coefficients of the resolution functions (wa of
// the complex form, then we of the real one: time_fns takes both at wa).
struct TddpTime {
  double gamma;
  double sigma;
  TimeConst tk;
  double wL;
  double wa[kWeidN];
  double we[kErfcN];
};
static_assert(__builtin_offsetof(TddpTime, we) == __builtin_offsetof(TddpTime, wa) + kWeidN * sizeof(double), "we follows wa");

// One point's lineshapes and barrier-and-angular factors, from which both
// amplitude sets A_k(s12, s13) and B_k = A_k(s13, s12) follow as products.
// With m2 = m3 (the model requires it) the pair terms at the mirrored point
// are those at (s12, s13) with pairs "12" and "13" exchanged, and for pair
// "23" only the spin-1 angular factor changes, by its sign (Z_1 = s_ac - s_bc
// with s_ac and s_bc exchanged; its mass term vanishes for equal masses), so
// each pair's terms are formed once per point.  A lineshape Ka T depends on the
// pair mass alone: resonances of pairs "12" and "13" are evaluated at both
// masses, once for all of the same spin, mass and width (as charged pairs of
// charge-conjugate daughters come; S::REP: the first of them), and those of
// "23" once for both sets: 16 lineshapes per event instead of 22 for the
// sixteen-resonance model, and 16 complex values held instead of 32 (NLL and
// gradient, 1M events: 88.9 -> 83.4 us).
template <class S>
struct TddpPoint {
  double H[3][3];              // factor of pair and spin
  double tr[S::K][2], ti[S::K][2];  // Ka T at s12, s13 (pairs 12, 13) or [0]: at s23
};
// Index of resonance k's lineshape in set SIDE (0: A, 1: B).
template <class S>
__host__ __device__ constexpr int tddp_at(int side, int k) {
  return S::chan[k] == 2 ? 0 : (S::chan[k] ^ side);
}
// Factor of pair C and spin L in set SIDE.
template <class S>
__device__ __forceinline__ double tddp_h(const TddpPoint<S>& p, int side, int C, int L) {
  if (L == 0) return 1.0;
  if (C == 2) return side && L == 1 ? -p.H[2][1] : p.H[2][L];
  return p.H[C ^ side][L];
}

__device__ __forceinline__ void tddp_bw(const double* __restrict__ rk, int L, double s, double G, double& tr,
                                        double& ti) {
  double a, b, D;
  bw_denominator(rk, s, G, a, b, D);
  const double d = L == 0 ? rcp_fast(D) : rk[dKA] * rcp_fast(D);  // Ka = 1 for L = 0
  tr = d * a;
  ti = d * b;
}

template <class S>
__device__ __forceinline__ void tddp_point(const DalitzConst& dc, const double* __restrict__ r, double s12,
                                           double s13, TddpPoint<S>& p) {
  constexpr int K = S::K;
  constexpr bool u1_01 = shape_uses<S>(0, 1) || shape_uses<S>(1, 1);
  constexpr bool u2_01 = shape_uses<S>(0, 2) || shape_uses<S>(1, 2);
  constexpr bool any01 = u1_01 || u2_01 || shape_uses<S>(0, 0) || shape_uses<S>(1, 0);
  constexpr bool any2 = shape_uses<S>(2, 0) || shape_uses<S>(2, 1) || shape_uses<S>(2, 2);
  const double s23 = dc.msum - s12 - s13;
  PairTerms q[3];
  if (any01) {
    pair_terms_t<u1_01, u2_01>(dc.ch[0], s12, s13, s23, dc.r2, dc.rD2, q[0]);
    pair_terms_t<u1_01, u2_01>(dc.ch[1], s13, s12, s23, dc.r2, dc.rD2, q[1]);
  }
  if (any2) pair_terms_t<shape_uses<S>(2, 1), shape_uses<S>(2, 2)>(dc.ch[2], s23, s12, s13, dc.r2, dc.rD2, q[2]);
#pragma unroll
  for (int C = 0; C < 3; ++C)
#pragma unroll
    for (int L = 1; L < 3; ++L) p.H[C][L] = (C == 2 ? any2 : any01) ? q[C].H[L] : 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (S::REP[k] != k) continue;
    const int C = S::chan[k], L = S::L[k];
    const double* rk = r + k * kDalFields;
    if (C == 2) {
      tddp_bw(rk, L, q[2].s, q[2].G[L], p.tr[k][0], p.ti[k][0]);
    } else {
      tddp_bw(rk, L, q[0].s, q[0].G[L], p.tr[k][0], p.ti[k][0]);
      tddp_bw(rk, L, q[1].s, q[1].G[L], p.tr[k][1], p.ti[k][1]);
    }
  }
}

// The coherent sum of set SIDE, sum_k c_k H T_k, the factor H applied once per
// pair and spin.
template <class S, int SIDE>
__device__ __forceinline__ cplx tddp_sum(const TddpPoint<S>& p, cdouble* __restrict__ c) {
  cplx A = {0.0, 0.0};
#pragma unroll
  for (int C = 0; C < 3; ++C)
#pragma unroll
    for (int L = 0; L < 3; ++L) {
      if (!shape_uses<S>(C, L)) continue;
      cplx in = {0.0, 0.0};
#pragma unroll
      for (int k = 0; k < S::K; ++k) {
        if (S::chan[k] != C || S::L[k] != L) continue;
        const int u = S::REP[k], v = tddp_at<S>(SIDE, k);
        in = cfma({c[2 * k], c[2 * k + 1]}, {p.tr[u][v], p.ti[u][v]}, in);
      }
      const double h = tddp_h<S>(p, SIDE, C, L);
      A = L == 0 ? cplx{A.re + in.re, A.im + in.im}
                 : cplx{__builtin_fma(h, in.re, A.re), __builtin_fma(h, in.im, A.im)};
    }
  return A;
}

// Adds Re(l H T_k) and -Im(l H T_k) of set SIDE to acc[2k], acc[2k + 1].
template <class S, int SIDE>
__device__ __forceinline__ void tddp_sum_grad(const TddpPoint<S>& p, cplx l, double* acc) {
#pragma unroll
  for (int C = 0; C < 3; ++C)
#pragma unroll
    for (int L = 0; L < 3; ++L) {
      if (!shape_uses<S>(C, L)) continue;
      const double h = tddp_h<S>(p, SIDE, C, L);
      const cplx lh = L == 0 ? l : cplx{l.re * h, l.im * h};
#pragma unroll
      for (int k = 0; k < S::K; ++k) {
        if (S::chan[k] != C || S::L[k] != L) continue;
        const int u = S::REP[k], v = tddp_at<S>(SIDE, k);
        grad_acc(lh, {p.tr[u][v], p.ti[u][v]}, acc[2 * k], acc[2 * k + 1]);
      }
    }
}

// Both amplitude sets themselves.
template <class S>
__device__ __forceinline__ void tddp_basis2(const DalitzConst& dc, const double* __restrict__ r, double s12,
                                            double s13, double (&are)[S::K], double (&aim)[S::K],
                                            double (&bre)[S::K], double (&bim)[S::K]) {
  TddpPoint<S> p;
  tddp_point<S>(dc, r, s12, s13, p);
#pragma unroll
  for (int k = 0; k < S::K; ++k) {
    const int u = S::REP[k], a = tddp_at<S>(0, k), b = tddp_at<S>(1, k);
    const double ha = tddp_h<S>(p, 0, S::chan[k], S::L[k]), hb = tddp_h<S>(p, 1, S::chan[k], S::L[k]);
    are[k] = ha * p.tr[u][a];
    aim[k] = ha * p.ti[u][a];
    bre[k] = hb * p.tr[u][b];
    bim[k] = hb * p.ti[u][b];
  }
}

// Events pass: one workgroup per chunk of events (s12, s13, t rows at
// ev, ev + ld, ev + 2 ld), one row of partial sums each:
// [-sum ln R, d/dRe c_k, d/dIm c_k (k), d/dRe cbar_k, d/dIm cbar_k (k), d/dx, d/dy].
// coef: theta on the device, (c, cbar, x, y).
template <class S, bool GRAD>
__device__ inline void tddp_events_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab,
                                        const TddpTime& tt, cdouble* __restrict__ coef0,
                                        const double* __restrict__ ev, int64_t ld, int64_t n, int chunk,
                                        double* __restrict__ part) {
  constexpr int K = S::K;
  constexpr int NV = GRAD ? 3 + 4 * K : 1;
  __shared__ double lds[block_sum_lds(NV)];
  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  const int64_t base = (int64_t)blockIdx.x * chunk;
  const int64_t end = base + chunk < n ? base + chunk : n;
  const double* const r0 = &tab->r[0][0];
  LogProd lp;  // -sum ln R enters acc[0] once per thread, at the end
  // an event's three values are loaded one iteration ahead (at a clamped
  // index): with one or two waves per SIMD nothing else hides the latency
  const int64_t i0 = base + threadIdx.x;
  const int64_t f0 = i0 < end ? i0 : base;
  double n12 = ev[f0], n13 = ev[ld + f0], nt = ev[2 * ld + f0];
  for (int64_t i = i0; i < end; i += kBlock) {
    const double s12 = n12, s13 = n13, t = nt;
    const int64_t in = i + kBlock < end ? i + kBlock : i;
    n12 = ev[in];
    n13 = ev[ld + in];
    nt = ev[2 * ld + in];
    // constants re-read through the scalar cache per event (an opaque zero
    // offset keeps them out of SGPRs that would overflow into VGPR lanes)
    int zero = 0;
    asm volatile("" : "+s"(zero));
    const double* r = r0 + zero;
    cdouble* coef = coef0 + zero;
    TimeFns T;
    time_fns<GRAD>((&tt.tk)[zero], tt.wa + zero, tt.wL, coef[4 * K], coef[4 * K + 1], t, T);
    TddpPoint<S> pt;
    tddp_point<S>(dc, r, s12, s13, pt);
    const cplx A = tddp_sum<S, 0>(pt, coef), Ab = tddp_sum<S, 1>(pt, coef + 2 * K);
    const double Hc = T.Hc, Hs = T.Hs;
    const cplx hc = {T.hr, T.hi};
    const double a2 = A.re * A.re + A.im * A.im, b2 = Ab.re * Ab.re + Ab.im * Ab.im;
    const double zr = A.re * Ab.re + A.im * Ab.im, zi = A.re * Ab.im - A.im * Ab.re;  // conj(A) Abar
    const double R = 0.5 * ((a2 + b2) * Hc + (a2 - b2) * hc.re - 2.0 * zr * Hs - 2.0 * zi * hc.im);
    lp.mul(R);
    if (GRAD) {
      const double w = -rcp_fast(R);
      const double hpc = Hc + hc.re, hmc = Hc - hc.re;
      // dR/dRe c_k - i dR/dIm c_k = lc A_k, and with lb and B_k for cbar:
      // lc = hpc conj(A) - (Hs + i Hsin) conj(Abar), lb = hmc conj(Abar) - (Hs - i Hsin) conj(A)
      // (the event's factor w = -1/R included)
      const cplx lc = {w * (hpc * A.re - Hs * Ab.re - hc.im * Ab.im), w * (-hpc * A.im + Hs * Ab.im - hc.im * Ab.re)};
      const cplx lb = {w * (hmc * Ab.re - Hs * A.re + hc.im * A.im), w * (-hmc * Ab.im + Hs * A.im + hc.im * A.re)};
      tddp_sum_grad<S, 0>(pt, lc, acc + 1);
      tddp_sum_grad<S, 1>(pt, lb, acc + 1 + 2 * K);
      acc[1 + 4 * K] += w * 0.5 * ((a2 - b2) * T.dr - 2.0 * zi * T.di);
      acc[2 + 4 * K] += w * 0.5 * ((a2 + b2) * T.dHc - 2.0 * zr * T.dHs);
    }
  }
  acc[0] = -lp.log();
  block_sum_row<NV>(acc, lds, part + (int64_t)blockIdx.x * NV);
}

// The normalization matrices over one chunk of grid cells: the Gram sums of
// the 2K vector (A, B), whose blocks are MAA, MBB and (B_j conj(A_i)) MAB_ij.
template <class S>
__device__ inline void tddp_gram_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab, int chunk,
                                      double* __restrict__ part) {
  constexpr int K = S::K;
  using G = Gram<2 * K>;
  __shared__ double lds[G::LDS];
  G g;
  g.init(lds);
  const uint32_t ncell = (uint32_t)dc.nx * (uint32_t)dc.ny;
  const uint32_t base = blockIdx.x * (uint32_t)chunk;
  const uint32_t end = base + chunk < ncell ? base + chunk : ncell;
  const double* const r0 = &tab->r[0][0];
  for (uint32_t i = base + (threadIdx.x & ~63u); i < end; i += kBlock) {
    const uint32_t c = i + (threadIdx.x & 63u);
    double s12, s13;
    const bool in = dalitz_cell(dc, c < end ? c : i, s12, s13) && c < end;
    if (!__any(in)) continue;
    int zero = 0;
    asm volatile("" : "+s"(zero));
    double are[K], aim[K], bre[K], bim[K], re[2 * K], im[2 * K];
    tddp_basis2<S>(dc, r0 + zero, s12, s13, are, aim, bre, bim);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      re[k] = are[k];
      im[k] = aim[k];
      re[K + k] = bre[k];
      im[K + k] = bim[k];
    }
    if (!in) {
#pragma unroll
      for (int k = 0; k < 2 * K; ++k) re[k] = im[k] = 0.0;
    }
    g.add(re, im, lds);
  }
  g.reduce(lds, part + (int64_t)blockIdx.x * 2 * gram_count(2 * K));
}

// ---------------------------------------------------------------- toy events
// A and Abar at one point.
template <class S>
__device__ __forceinline__ void tddp_amps(const DalitzConst& dc, const double* __restrict__ r,
                                          cdouble* __restrict__ coef, double s12, double s13, cplx& A,
                                          cplx& Ab) {
  TddpPoint<S> p;
  tddp_point<S>(dc, r, s12, s13, p);
  A = tddp_sum<S, 0>(p, coef);
  Ab = tddp_sum<S, 1>(p, coef + 2 * S::K);
}

// Largest (|A| + |Abar|)^2 over the grid-cell centres inside the region (bits
// of a non-negative double, ordered like the value) in *vmax.
template <class S>
__device__ inline void tddp_gridmax_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab,
                                         const double* __restrict__ coef, unsigned long long* __restrict__ vmax) {
  const uint32_t ncell = (uint32_t)dc.nx * (uint32_t)dc.ny;
  const double* r = &tab->r[0][0];
  double m = 0.0;
  for (uint32_t c = blockIdx.x * kBlock + threadIdx.x; c < ncell; c += gridDim.x * kBlock) {
    double s12, s13;
    if (!dalitz_cell(dc, c, s12, s13)) continue;
    cplx A, Ab;
    tddp_amps<S>(dc, r, (cdouble*)coef, s12, s13, A, Ab);
    const double e = sqrt(A.re * A.re + A.im * A.im) + sqrt(Ab.re * Ab.re + Ab.im * Ab.im);
    m = fmax(m, e * e);
  }
  block_max(m, vmax);
}

// Accept-reject toy events: R(s12, s13, t) <= e^{-lam t} (|A| + |Abar|)^2 with
// lam = G (1 - |y|), so event i, attempt a takes (u1, u2) from counter
// (i, 2a, 2) and (u3, u4) from (i, 2a + 1, 2) under key (k0, k1): the
// candidate (lo12 + u1 (hi12 - lo12), lo13 + u2 (hi13 - lo13), t = -ln(1 - u3)/lam)
// is kept when it lies in the region and u4 W e^{-lam t} < R; the measured
// time adds sigma_t times a Box-Muller normal from counter (i, 0, 3).  bad[0]
// counts kept events with (|A| + |Abar|)^2 > W, bad[1] events left NaN after
// max_attempts.
template <class S>
__device__ inline void tddp_gen_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab,
                                     const double* __restrict__ coef, const TddpTime& tt, uint32_t k0, uint32_t k1,
                                     int64_t n, const double* __restrict__ Wp, double lo12, double hi12, double lo13,
                                     double hi13, int per_wave, int max_attempts, double* __restrict__ ev, int64_t ld,
                                     unsigned long long* __restrict__ bad) {
#pragma clang fp contract(off)
  __shared__ StagedLds lds;
  const double W = *Wp;
  if (!(W > 0.0 && W < __builtin_inf())) return;  // the host reports it
  const double* r = &tab->r[0][0];
  constexpr int K = S::K;
  const double x = coef[4 * K], y = coef[4 * K + 1];
  const double G = tt.gamma;
  const double lam = G * (1.0 - fabs(y));
  const double w12 = hi12 - lo12, w13 = hi13 - lo13;
  double t, env;
  accept_reject_staged(
      lds, n, per_wave, max_attempts,
      [&](int64_t i, int a, double& s12, double& s13) {
#pragma clang fp contract(off)
        double u1, u2;
        philox_uniforms((uint64_t)i, 2u * a, 2u, k0, k1, u1, u2);
        s12 = lo12 + u1 * w12;
        s13 = lo13 + u2 * w13;
        return dalitz_inside_quick(dc, s12, s13);
      },
      [&](int64_t i, int a, double s12, double s13) {
#pragma clang fp contract(off)
        double u3, u4;
        philox_uniforms((uint64_t)i, 2u * a + 1u, 2u, k0, k1, u3, u4);
        t = -log1p(-u3) / lam;
        cplx A, Ab;
        tddp_amps<S>(dc, r, (cdouble*)coef, s12, s13, A, Ab);
        const double a2 = A.re * A.re + A.im * A.im, b2 = Ab.re * Ab.re + Ab.im * Ab.im;
        const double zr = A.re * Ab.re + A.im * Ab.im, zi = A.re * Ab.im - A.im * Ab.re;
        const double gt = G * t;
        const double ep = exp(y * gt), em = exp(-y * gt);
        double sx, cx;
        sincos(x * gt, &sx, &cx);
        const double R = 0.5 * exp(-gt) *
                         ((a2 + b2) * (0.5 * (ep + em)) + (a2 - b2) * cx - 2.0 * zr * (0.5 * (ep - em)) -
                          2.0 * zi * sx);
        const double e = sqrt(a2) + sqrt(b2);
        env = e * e;
        return u4 * W * exp(-lam * t) < R;
      },
      [&](int64_t i, double s12, double s13) {
#pragma clang fp contract(off)
        double v1, v2;
        philox_uniforms((uint64_t)i, 0u, 3u, k0, k1, v1, v2);
        ev[i] = s12;
        ev[ld + i] = s13;
        ev[2 * ld + i] = t + tt.sigma * (sqrt(-2.0 * log1p(-v1)) * cos(2.0 * 3.14159265358979323846 * v2));
        if (env > W) atomicAdd(bad, 1ull);
      },
      [&](int64_t i) {
        for (int j = 0; j < 3; ++j) ev[j * ld + i] = __builtin_nan("");
        atomicAdd(bad + 1, 1ull);
      });
}

}  // namespace fn

// Kernels for shape S (used by the generated source).
// (coef null: theta is the launch's argument)
#define FN_TDDP_EVENTS(NAME, S, GRAD)                                                                          \
  extern "C" __global__ __launch_bounds__(fn::kBlock) __attribute__((amdgpu_waves_per_eu(2))) void NAME(       \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, fn::TddpTime tt,                            \
      const double* __restrict__ coef, fn::TddpArg ca, const double* __restrict__ ev, int64_t ld, int64_t n,   \
      int chunk, double* __restrict__ part) {                                                                  \
    fn::cdouble* c = coef ? (fn::cdouble*)coef : (fn::cdouble*)&ca.v[0];                                       \
    fn::tddp_events_body<S, GRAD>(dc, tab, tt, c, ev, ld, n, chunk, part);                                    \
  }
#define FN_TDDP_GRAM(NAME, S)                                                                                  \
  extern "C" __global__ __launch_bounds__(fn::kBlock) __attribute__((amdgpu_waves_per_eu(2))) void NAME(       \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, int chunk, double* __restrict__ part) {    \
    fn::tddp_gram_body<S>(dc, tab, chunk, part);                                                               \
  }
#define FN_TDDP_GEN(GRIDMAX, GEN, S)                                                                           \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void GRIDMAX(                                            \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, const double* __restrict__ coef,            \
      unsigned long long* __restrict__ vmax) {                                                                 \
    fn::tddp_gridmax_body<S>(dc, tab, coef, vmax);                                                             \
  }                                                                                                            \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void GEN(                                                \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, const double* __restrict__ coef,            \
      fn::TddpTime tt, uint32_t k0, uint32_t k1, int64_t n, const double* __restrict__ W, double lo12,         \
      double hi12, double lo13, double hi13, int per_wave, int max_attempts, double* __restrict__ ev,          \
      int64_t ld, unsigned long long* __restrict__ bad) {                                                      \
    fn::tddp_gen_body<S>(dc, tab, coef, tt, k0, k1, n, W, lo12, hi12, lo13, hi13, per_wave, max_attempts, ev,  \
                         ld, bad);                                                                              \
  }
