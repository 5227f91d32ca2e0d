// Device code of the time-dependent four-body model (the paper's four-body
// time-dependent amplitude analyses, Abstract and Sec. 5).  The per-event and
// normalization-matrix passes are compiled at run time for each model shape
// (which pair entries are resonant and with which spin, which entries and
// angular factor every basis amplitude takes) as compile-time constants; the
// time functions are shared with the library's own kernels.
//
// Per event (m12, m34, c12, c34, phi, t) and fit:
//   a12[r], a34[r]   pair lineshapes: 1 (non-resonant) or Ka F_L(q r) T with
//                    T = (a + i b)/(a^2 + b^2), a = m0^2 - s, b = Kw G_L(s),
//                    G_L = q^(2L+1) F_L(q r)^2 / sqrt(s) (as in the three-body kernel)
//   B_k = a12[r1_k] a34[r2_k] Omega_k(c12, c34, phi), A = sum c_k B_k, Abar = sum cbar_k B_k
//   R = 1/2 [(|A|^2+|Abar|^2) Hc + (|A|^2-|Abar|^2) Hcos - 2 Re(A* Abar) Hs - 2 Im(A* Abar) Hsin]
// with Hc, Hs = (h(G(1-y)) +- h(G(1+y)))/2 and Hcos + i Hsin = h(G(1 - i x)), where
// h(a; t) = exp(a^2 s^2/2 - a t) erfc((a s^2 - t)/(s sqrt2)) / 2 is the exponential
// convolved with the Gaussian resolution of width s, evaluated through the
// Faddeeva function w (Weideman, SIAM J. Numer. Anal. 31 (1994) 1497:
// w(z) = [2 p(Z)/(L - i z) + 1/sqrt(pi)] / (L - i z), Z = (L + i z)/(L - i z),
// p a polynomial of degree N-1 whose coefficients are the Fourier
// coefficients of exp(-t^2)(L^2 + t^2), t = L tan(theta/2); N = 40, L = sqrt(N/sqrt 2)).
// dh/da = (a s^2 - t) h - s/sqrt(2 pi) exp(-t^2/(2 s^2)) gives the x, y derivatives.
// I is the phase-space average of the t-integrated rate, a quadratic form in the
// coefficients through the per-fit matrix M_ij = <B_i conj(B_j)>.
#pragma once
#include "accept_device.hpp"
#include "device_common.hpp"
#include "fastmath.hpp"
#include "gram_device.hpp"
#include "philox.hpp"
#include "td4_types.hpp"

namespace fn {

struct cplx {
  double re, im;
};
__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// c + a b as four chained FMAs
__device__ __forceinline__ cplx cfma(cplx a, cplx b, cplx c) {
  return {__builtin_fma(a.re, b.re, __builtin_fma(-a.im, b.im, c.re)),
          __builtin_fma(a.re, b.im, __builtin_fma(a.im, b.re, c.im))};
}
// (gr, gi) += (Re(l b), -Im(l b)): a gradient pair d/dRe, d/dIm from l b
__device__ __forceinline__ void grad_acc(cplx l, cplx b, double& gr, double& gi) {
  gr = __builtin_fma(l.re, b.re, __builtin_fma(-l.im, b.im, gr));
  gi = __builtin_fma(-l.re, b.im, __builtin_fma(-l.im, b.re, gi));
}
__device__ __forceinline__ cplx crcp(cplx a) {
  const double d = rcp_fast(__builtin_fma(a.re, a.re, a.im * a.im));
  return {a.re * d, -a.im * d};
}

constexpr double kInvSqrtPi = 0.56418958354775628695;
constexpr double kInvSqrt2Pi = 0.39894228040143267794;
constexpr double kInvSqrt2 = 0.70710678118654752440;

// The rational approximation: scale L and coefficients wa[0..N-1] = a_1..a_N.

// w(z) for Im z >= 0.
__device__ inline cplx faddeeva(const double* __restrict__ wa, double L, cplx z) {
  const cplx d = {L + z.im, -z.re};           // L - i z
  const cplx id = crcp(d);
  const cplx Z = cmul({L - z.im, z.re}, id);  // (L + i z)/(L - i z)
  const double nZi = -Z.im;
  cplx p = {wa[kWeidN - 1], 0.0};
#pragma unroll
  for (int n = kWeidN - 2; n >= 0; --n)
    p = {__builtin_fma(p.re, Z.re, fma_sc(p.im, nZi, wa[n])), __builtin_fma(p.re, Z.im, p.im * Z.re)};
  const cplx t = cmul({2.0 * p.re, 2.0 * p.im}, id);
  return cmul({t.re + kInvSqrtPi, t.im}, id);
}

// w(i y) = exp(y^2) erfc(y), y >= 0: (K + y) w(i y) as a polynomial in Z =
// (K - y)/(K + y), which maps [0, inf) to (-1, 1] (the Chebyshev expansion of
// Schonfelder, Math. Comp. 32 (1978) 1232, in powers of Z; we: its kErfcN
// coefficients, td4_types.hpp).  Relative error at most 7.2e-16 over y in
// [1e-6, 1e3] (host emulation; the 40-term form of w(z) on this axis: 1.0e-15).
__device__ inline double erfcx_pos(const double* __restrict__ we, double y) {
  const double id = rcp_acc(kErfcK + y);  // its error enters twice, through Z and the last product
  const double Z = (kErfcK - y) * id;
  double p = we[kErfcN - 1];
#pragma unroll
  for (int n = kErfcN - 2; n >= 0; --n) p = fma_sc(p, Z, we[n]);
  return p * id;
}

// h(a; t) and dh/da for real a.  g = exp(-t^2/(2 s^2)).
__device__ inline void h_real(const double* __restrict__ we, double a, double t, double s, double s2, double g,
                              double& h, double& dh) {
  const double u = a * s2 - t;
  const double z = u * (kInvSqrt2 / s);
  const double w = erfcx_pos(we, fabs(z));
  h = z >= 0.0 ? 0.5 * g * w : exp_fast(0.5 * a * a * s2 - a * t) - 0.5 * g * w;
  dh = u * h - s * kInvSqrt2Pi * g;
}

// h(a; t) and dh/da for complex a (ALONE: time_fns).
template <bool ALONE>
__device__ inline void h_cplx(const double* __restrict__ wa, double L, cplx a, double t, double s, double s2, double g,
                              cplx& h, cplx& dh) {
  const cplx u = {a.re * s2 - t, a.im * s2};
  const cplx z = {u.re * (kInvSqrt2 / s), u.im * (kInvSqrt2 / s)};
  const bool up = z.re >= 0.0;
  const cplx arg = up ? cplx{-z.im, z.re} : cplx{z.im, -z.re};  // i z or -i z, Im >= 0
  const cplx w = faddeeva(wa, L, arg);
  if (up) {
    h = {0.5 * g * w.re, 0.5 * g * w.im};
  } else {
    const double er = 0.5 * (a.re * a.re - a.im * a.im) * s2 - a.re * t;
    const double ei = a.re * a.im * s2 - a.im * t;
    double sn, cs;
    sincos_fast<ALONE>(ei, sn, cs);
    const double e = exp_fast(er);
    h = {e * cs - 0.5 * g * w.re, e * sn - 0.5 * g * w.im};
  }
  const cplx uh = cmul(u, h);
  dh = {uh.re - s * kInvSqrt2Pi * g, uh.im};
}

// The time functions of one event and their derivatives: Hc, Hs and dHc/dy,
// dHs/dy; hr + i hi = Hcos + i Hsin and dhr/dx, dhi/dx.
struct TimeFns {
  double Hc, Hs, hr, hi, dHc, dHs, dr, di;
};

// The resolution constants of one fit (G = 1/tau, s = sigma_t).
__host__ __device__ inline TimeConst time_const(double G, double s) {
  TimeConst k;
  const double s2 = s * s;
  k.g = G;
  k.s = s;
  k.s2 = s2;
  k.gs2 = G * s2;
  k.hg2s2 = 0.5 * G * G * s2;
  k.iz = kInvSqrt2 / s;
  k.ni2s2 = -0.5 / s2;
  k.kg = G * s * kInvSqrt2Pi;
  k.g2s2 = G * G * s2;
  k.s3 = s * fmax(3.0, G * s);
  return k;
}

// Terms 2 k0 + 1 .. 2 k1 of the series of time_fns: c_n = G^n h_n / n! and
// e_n = n c_n = v c_{n-1} + w c_{n-2} (v = G u, w = G^2 s^2) added to the
// four sums and, for gradients, their derivatives' sums; qy, qx: y^2k, (-x^2)^k.
struct TimeSeries {
  double ce, co;           // c_{2k}, c_{2k-1}
  double qy, qx;
  double ey, oy, ex, ox;   // even terms past c_0 and odd terms / y, / x
  double dey, doy, dex, dox;
};
template <bool GRAD>
__device__ __forceinline__ void time_terms(TimeSeries& a, double v, double w, double y2, double nx2, int k0, int k1) {
#pragma unroll
  for (int k = k0; k < k1; ++k) {
    const double eo = __builtin_fma(v, a.ce, w * a.co);
    a.co = eo * (1.0 / (2 * k + 1));
    const double ee = __builtin_fma(v, a.co, w * a.ce);
    a.ce = ee * (1.0 / (2 * k + 2));
    a.oy = __builtin_fma(a.co, a.qy, a.oy);
    a.ox = __builtin_fma(a.co, a.qx, a.ox);
    if (GRAD) {
      a.doy = __builtin_fma(eo, a.qy, a.doy);
      a.dox = __builtin_fma(eo, a.qx, a.dox);
      a.dey = __builtin_fma(ee, a.qy, a.dey);
      a.dex = __builtin_fma(ee, a.qx, a.dex);
    }
    a.qy *= y2;
    a.qx *= nx2;
    a.ey = __builtin_fma(a.ce, a.qy, a.ey);
    a.ex = __builtin_fma(a.ce, a.qx, a.ex);
  }
}

// The time functions at decay time t.  All four are h(a; t) at points a = G +
// d, d = +-G y and -i G x, near a = G, and h's derivatives follow from h itself:
// h_0 = h(G; t), h_1 = u h_0 - s g / sqrt(2 pi), h_{n+1} = u h_n + n s^2 h_{n-1}
// (u = G s^2 - t, g = exp(-t^2 / 2 s^2); for u < 0 the terms of each step have
// one sign).  So one real h and a Taylor series give what otherwise takes two
// real and one complex h.  |h_n d^n / n!| <= h_0 r^n / n! with r = max(|x|,
// |y|) G (|t| + s max(3, G s)) for n <= 20, which puts the rest after ten terms
// below 3e-18 h_0 (3e-16 in the derivatives' sums) for r <= 1/8 and after twenty
// below 2e-18 (4e-17) for r <= 5/4.  For u > 0 the recurrence cancels and each
// step multiplies its rounding error by u, which r bounds as well: G s in place
// of 3 for resolutions above three lifetimes, where u reaches G s^2 (with 3 s
// there, the error grew to 7e-11 of h_0 at thirty lifetimes).  A wave takes ten
// terms, twenty when one of its events needs them, and the three functions
// evaluated one by one beyond that (the line lies where twenty terms, 160
// multiply-adds, stop sufficing; the three evaluations take about 460
// instructions).  The events are few there: mixing parameters of the size fits
// meet (below 0.01) keep r <= 1/8 up to twelve lifetimes.
// One NLL and gradient: four-body, 10M events, twenty amplitudes 456 -> 349 us;
// three-body, 1M events, sixteen resonances 105.8 -> 94.5 us.  The rare forms are
// kept out of the registers of the common one: their branches are marked
// unlikely, and they use the written-out exponential, sine and cosine (with the
// library's inlined, its coefficients filled some sixty vector registers over
// the whole event loop: four-body pass 227 -> 185 registers, 290 -> 281 us;
// three-body 296 -> 256 and two waves per SIMD instead of one, 83.4 -> 77.4 us).
//
// ALONE: each event takes the form its own r asks for, and its sine and cosine
// likewise, so that its value does not depend on the others of its wave (the
// density, which is handed out per event).  A wave with events of two forms then
// takes both: 1M events, ten amplitudes, 43 us a call either way for mixing
// parameters below 0.01, 57 instead of 53 at x = 0.8, whose events fall on both
// sides of the line.
template <bool GRAD, bool ALONE = false>
__device__ __forceinline__ void time_fns(const TimeConst& k, const double* __restrict__ wt, double wL, double x,
                                         double y, double t, TimeFns& o) {
  const double g = exp_fast(t * t * k.ni2s2);
  const double r = fmax(fabs(x), fabs(y)) * k.g * (fabs(t) + k.s3);
  const bool beyond = !(r <= kTimeSeriesMax), more = r > kTimeSeriesTen;
  if (__builtin_expect(ALONE ? beyond : __any(beyond), 0)) {
    double hp, dhp, hm, dhm;
    cplx hc, dhc;
    const double* we = wt + kWeidN;
    h_real(we, k.g * (1.0 - y), t, k.s, k.s2, g, hp, dhp);
    h_real(we, k.g * (1.0 + y), t, k.s, k.s2, g, hm, dhm);
    h_cplx<ALONE>(wt, wL, {k.g, -k.g * x}, t, k.s, k.s2, g, hc, dhc);
    o.Hc = 0.5 * (hp + hm);
    o.Hs = 0.5 * (hp - hm);
    o.hr = hc.re;
    o.hi = hc.im;
    // d hp/dy = -G dh(G(1-y)), d hm/dy = +G dh(G(1+y)), d hc/dx = -i G dh(G(1-ix))
    o.dHc = 0.5 * k.g * (dhm - dhp);
    o.dHs = -0.5 * k.g * (dhp + dhm);
    o.dr = k.g * dhc.im;
    o.di = -k.g * dhc.re;
    return;
  }
  const double u = k.gs2 - t;
  const double z = u * k.iz;
  double eg = exp_fast(__builtin_fma(-k.g, t, k.hg2s2));
  asm volatile("" : "+v"(eg));  // formed in line with the rest, not behind a branch on z
  const double e = 0.5 * g * erfcx_pos(wt + kWeidN, fabs(z));
  const double c0 = z >= 0.0 ? e : eg - e;
  const double v = k.g * u, w = k.g2s2;
  const double y2 = y * y, nx2 = -x * x;
  // n = 1, 2
  const double c1 = __builtin_fma(v, c0, -k.kg * g);
  const double e2 = __builtin_fma(v, c1, w * c0);
  TimeSeries a;
  a.ce = 0.5 * e2;
  a.co = c1;
  a.qy = y2;
  a.qx = nx2;
  a.oy = a.ox = a.doy = a.dox = c1;
  a.dey = a.dex = e2;
  a.ey = a.ce * y2;
  a.ex = a.ce * nx2;
  time_terms<GRAD>(a, v, w, y2, nx2, 1, 5);
  if (__builtin_expect(ALONE ? more : __any(more), 0)) time_terms<GRAD>(a, v, w, y2, nx2, 5, 10);
  o.Hc = c0 + a.ey;
  o.Hs = -y * a.oy;
  o.hr = c0 + a.ex;
  o.hi = -x * a.ox;
  o.dHc = y * a.dey;
  o.dHs = -a.doy;
  o.dr = -x * a.dex;
  o.di = -a.dox;
}

// ------------------------------------------------------- shape-specialized
// A shape S gives, as compile-time constants: K, N12, N34, L12[], NR12[],
// L34[], NR34[] (NR = 1 marks a flat entry), A1[], A2[] (pair entries of
// every basis amplitude) and T[] (angular factor).

// Entry r of pair 12 or 34 of shape S, read as a constant expression: a
// template parameter bound to the array itself left the compiler with a load
// and a branch per entry and event.
template <class S, bool P34>
struct Td4Pair {
  static constexpr int N = P34 ? S::N34 : S::N12;
  static __device__ __forceinline__ constexpr int L(int r) { return P34 ? S::L34[r] : S::L12[r]; }
  static __device__ __forceinline__ constexpr bool flat(int r) { return (P34 ? S::NR34[r] : S::NR12[r]) != 0; }
  static constexpr bool any_l1() {
    bool u = false;
    for (int r = 0; r < N; ++r) u = u || ((P34 ? S::L34[r] : S::L12[r]) == 1 && !(P34 ? S::NR34[r] : S::NR12[r]));
    return u;
  }
};

// m^2 rounded by itself, as the reference evaluation in 64 bits has it: formed
// inside an FMA, m0^2 - m^2 keeps the square's rounding, which next to a narrow
// peak is a difference of 1e-14 in the density.
__device__ __forceinline__ double sq_rn(double m) {
#pragma clang fp contract(off)
  const double s = m * m;
  return s;
}

// Lineshapes of one pair from its invariant mass m (rt: the fit's m0^2, Kw, Ka).
template <class S, bool P34>
__device__ __forceinline__ void pair_amps_s(double m, double sum2, double dif2, double r2,
                                            const double (*__restrict__ rt)[3], cplx (&amp)[Td4Pair<S, P34>::N]) {
  using T = Td4Pair<S, P34>;
  const double s = sq_rn(m);
  const double im = rcp_fast(m);
  const double lq = fmax((s - sum2) * (s - dif2), 0.0);
  const double q2 = 0.25 * lq * im * im;
  const double G0 = sqrt_fast(q2) * im;
  double F1 = 1.0, G1 = 0.0;
  constexpr bool l1 = T::any_l1();
  if (l1) {
    F1 = rsqrt_fast(1.0 + q2 * r2);
    G1 = G0 * q2 * F1 * F1;
  }
#pragma unroll
  for (int r = 0; r < T::N; ++r) {
    amp[r] = {1.0, 0.0};
    if (!T::flat(r)) {
      const double G = T::L(r) == 1 ? G1 : G0;
      const double a = rt[r][0] - s;
      const double b = rt[r][1] * G;
      const double d = rcp_fast(__builtin_fma(a, a, b * b));
      const double k = T::L(r) == 1 ? rt[r][2] * F1 * d : d;  // Ka = 1 for L = 0
      amp[r] = {k * a, k * b};
    }
  }
}

// One kinematic point under one fit's lineshapes: the lineshapes of both
// pairs and the angular values every basis function is formed from.
template <class S>
struct Td4Point {
  cplx a12[S::N12], a34[S::N34];
  double c12, c34;
  double ssc, sss;  // 1/2 sin theta12 sin theta34 (cos phi, sin phi)
};

template <class S, bool ALONE = false>
__device__ __forceinline__ void td4_point_s(const Td4Const& tc, const Td4Table& tb, double m12, double m34, double c12,
                                            double c34, double phi, Td4Point<S>& p) {
  pair_amps_s<S, false>(m12, tc.sum12, tc.dif12, tc.r2, tb.r12, p.a12);
  pair_amps_s<S, true>(m34, tc.sum34, tc.dif34, tc.r2, tb.r34, p.a34);
  constexpr bool has_sc = [] {
    bool u = false;
    for (int k = 0; k < S::K; ++k) u = u || S::T[k] >= 4;
    return u;
  }();
  p.c12 = c12;
  p.c34 = c34;
  p.ssc = 0.0;
  p.sss = 0.0;
  if (has_sc) {
    const double ss = 0.5 * sqrt_fast(fmax(1.0 - c12 * c12, 0.0)) * sqrt_fast(fmax(1.0 - c34 * c34, 0.0));
    double sp, cp;
    sincos_fast<ALONE>(phi, sp, cp);
    p.ssc = ss * cp;
    p.sss = ss * sp;
  }
}

// Basis function B_k of a point (k a constant after unrolling); products
// with flat entries and real angular factors are formed as such.
template <class S>
__device__ __forceinline__ cplx td4_bk(const Td4Point<S>& p, int k) {
  const int r1 = S::A1[k], r2 = S::A2[k];
  cplx xy;
  if (S::NR12[r1] && S::NR34[r2]) xy = {1.0, 0.0};
  else if (S::NR12[r1]) xy = p.a34[r2];
  else if (S::NR34[r2]) xy = p.a12[r1];
  else xy = cmul(p.a12[r1], p.a34[r2]);
  switch (S::T[k]) {
    case 0: return xy;
    case 1: return {xy.re * p.c34, xy.im * p.c34};
    case 2: return {xy.re * p.c12, xy.im * p.c12};
    case 3: { const double cc = p.c12 * p.c34; return {xy.re * cc, xy.im * cc}; }
    case 4: return cmul(xy, {p.ssc, p.sss});
    default: return cmul(xy, {p.ssc, -p.sss});
  }
}

// Whether any basis function of shape S in sum SIDE (0: A, 1: Abar) has pair
// entries r1 and r2 (r2 < 0: any).
template <class S>
__host__ __device__ constexpr bool td4_has(int side, int r1, int r2) {
  bool u = false;
  for (int k = 0; k < S::K; ++k)
    u = u || (S::A1[k] == r1 && (r2 < 0 || S::A2[k] == r2) && (side ? S::PB[k] : S::PA[k]) >= 0);
  return u;
}

// w += c Omega_T, the angular factor of type T (first: w = c Omega_T).
template <class S>
__device__ __forceinline__ void td4_add_omega(const Td4Point<S>& p, int T, double cr, double ci, bool first, cplx& w) {
  if (first && T == 0) {
    w = {cr, ci};
    return;
  }
  if (first) w = {0.0, 0.0};
  if (T == 0) {
    w = {w.re + cr, w.im + ci};
  } else if (T <= 3) {
    const double om = T == 1 ? p.c34 : (T == 2 ? p.c12 : p.c12 * p.c34);
    w = {__builtin_fma(cr, om, w.re), __builtin_fma(ci, om, w.im)};
  } else {
    const double sn = T == 4 ? p.sss : -p.sss;
    w = {__builtin_fma(cr, p.ssc, __builtin_fma(-ci, sn, w.re)), __builtin_fma(cr, sn, __builtin_fma(ci, p.ssc, w.im))};
  }
}

// The coherent sum SIDE of a point, sum_k c_k B_k with B_k = a12 a34 Omega_k,
// factored by pair entries: sum_r1 a12[r1] sum_r2 a34[r2] sum_k c_k Omega_k.
// The products of lineshapes are taken once per pair of entries and sum, not
// once per basis function, and no basis function is formed.
template <class S, int SIDE>
__device__ __forceinline__ cplx td4_sum(const Td4Point<S>& p, const double (*__restrict__ c)[2]) {
  cplx A = {0.0, 0.0};
#pragma unroll
  for (int r1 = 0; r1 < S::N12; ++r1) {
    if (!td4_has<S>(SIDE, r1, -1)) continue;
    cplx in = {0.0, 0.0};
    bool none = true;
#pragma unroll
    for (int r2 = 0; r2 < S::N34; ++r2) {
      if (!td4_has<S>(SIDE, r1, r2)) continue;
      cplx w = {0.0, 0.0};
      bool first = true;
#pragma unroll
      for (int k = 0; k < S::K; ++k)
        if (S::A1[k] == r1 && S::A2[k] == r2 && (SIDE ? S::PB[k] : S::PA[k]) >= 0) {
          td4_add_omega<S>(p, S::T[k], c[k][0], c[k][1], first, w);
          first = false;
        }
      if (S::NR34[r2]) in = none ? w : cplx{in.re + w.re, in.im + w.im};
      else in = cfma(p.a34[r2], w, in);
      none = false;
    }
    if (S::NR12[r1]) A = {A.re + in.re, A.im + in.im};
    else A = cfma(p.a12[r1], in, A);
  }
  return A;
}

// Adds the event's gradient terms of sum SIDE, Re(l B_k) and -Im(l B_k), to
// the accumulators of its coefficients (acc: their slots in theta order), with
// the products l a12 and l a12 a34 shared in the same way.
template <class S, int SIDE>
__device__ __forceinline__ void td4_sum_grad(const Td4Point<S>& p, cplx l, double* acc) {
#pragma unroll
  for (int r1 = 0; r1 < S::N12; ++r1) {
    if (!td4_has<S>(SIDE, r1, -1)) continue;
    const cplx u = S::NR12[r1] ? l : cmul(l, p.a12[r1]);
#pragma unroll
    for (int r2 = 0; r2 < S::N34; ++r2) {
      if (!td4_has<S>(SIDE, r1, r2)) continue;
      const cplx v = S::NR34[r2] ? u : cmul(u, p.a34[r2]);
#pragma unroll
      for (int k = 0; k < S::K; ++k) {
        const int i = SIDE ? S::PB[k] : S::PA[k];
        if (S::A1[k] != r1 || S::A2[k] != r2 || i < 0) continue;
        const int T = S::T[k];
        if (T == 0) {
          acc[i] += v.re;
          acc[i + 1] -= v.im;
        } else if (T <= 3) {
          const double om = T == 1 ? p.c34 : (T == 2 ? p.c12 : p.c12 * p.c34);
          acc[i] = __builtin_fma(v.re, om, acc[i]);
          acc[i + 1] = __builtin_fma(-v.im, om, acc[i + 1]);
        } else {
          grad_acc(v, {p.ssc, T == 4 ? p.sss : -p.sss}, acc[i], acc[i + 1]);
        }
      }
    }
  }
}

// All basis amplitudes B_k of one kinematic point under one fit's lineshapes.
template <class S>
__device__ __forceinline__ void td4_basis_s(const Td4Const& tc, const Td4Table& tb, double m12, double m34, double c12,
                                            double c34, double phi, cplx (&B)[S::K]) {
  Td4Point<S> p;
  td4_point_s<S>(tc, tb, m12, m34, c12, c34, phi, p);
#pragma unroll
  for (int k = 0; k < S::K; ++k) B[k] = td4_bk<S>(p, k);
}

// Workgroup -> (chunk, fit) of a pass over a sample shared by n_fits fits.
// Workgroups are handed to the eight XCDs round robin by index, and each XCD
// has its own L2: the n_fits workgroups of one chunk are given indices that
// are equal modulo 8, so that the chunk is fetched into one L2 only.  The
// launch has td4_blocks(nch, n_fits) workgroups; false for padding ones.
constexpr int kXcds = 8;
__host__ __device__ inline int64_t td4_blocks(int64_t nch, int n_fits) {
  return n_fits == 1 ? nch : (nch + kXcds - 1) / kXcds * kXcds * n_fits;
}
__device__ __forceinline__ bool td4_block_item(int64_t nch, int n_fits, int64_t& ch, int& f) {
  const int64_t b = blockIdx.x;
  if (n_fits == 1) {
    ch = b;
    f = 0;
    return true;
  }
  const int64_t x = b % kXcds, j = b / kXcds;
  f = (int)(j % n_fits);
  ch = (j / n_fits) * kXcds + x;
  return ch < nch;
}

// Events pass for n_fits fits sharing one sample: one workgroup per (chunk,
// fit), the fits of a chunk on one XCD so that they share it through its L2;
// a fit whose status entry is not running is skipped (status may be null).
template <class S, bool GRAD>
__device__ inline void td4_events_body(const Td4Const& tc, const Td4Table* __restrict__ tabs,
                                       const int* __restrict__ status, const double* __restrict__ ev, int64_t ld,
                                       int64_t n, int chunk, int64_t nch, int n_fits, double* __restrict__ part) {
  constexpr int K = S::K;
  constexpr int P = S::P;
  // partial row: NLL, then the gradient in theta order (A's coefficients,
  // Abar's, x, y)
  constexpr int NV = GRAD ? 1 + P : 1;
  __shared__ double lds[block_sum_lds(NV)];
  int64_t ch;
  int f;
  if (!td4_block_item(nch, n_fits, ch, f)) return;
  if (status && status[f] != 1) return;
  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  const int64_t base = ch * chunk;
  const int64_t end = base + chunk < n ? base + chunk : n;
  LogProd lp;  // -sum ln R enters acc[0] once per thread, at the end
  // an event's six values are loaded one iteration ahead (at a clamped index):
  // with two waves per SIMD nothing else hides the latency
  const int64_t i0 = base + threadIdx.x;
  double nx[6];
#pragma unroll
  for (int j = 0; j < 6; ++j) nx[j] = ev[j * ld + (i0 < end ? i0 : base)];
  for (int64_t i = i0; i < end; i += kBlock) {
    double e[6];
    const int64_t in = i + kBlock < end ? i + kBlock : i;
#pragma unroll
    for (int j = 0; j < 6; ++j) e[j] = nx[j];
#pragma unroll
    for (int j = 0; j < 6; ++j) nx[j] = ev[j * ld + in];
    // the fit's constants are re-read through the scalar cache on every event
    // (an opaque zero offset keeps them from being hoisted into SGPRs that
    // would overflow into VGPR lanes)
    int zero = 0;
    asm volatile("" : "+s"(zero));
    const Td4Table& tb = tabs[f + zero];
    // time functions first: the lineshapes are not live across them
    TimeFns T;
    time_fns<GRAD>(tb.tk, tc.wa + zero, tc.wL, tb.x, tb.y, e[5], T);
    Td4Point<S> pt;
    td4_point_s<S>(tc, tb, e[0], e[1], e[2], e[3], e[4], pt);
    const cplx A = td4_sum<S, 0>(pt, tb.c), Ab = td4_sum<S, 1>(pt, tb.cb);
    const double Hc = T.Hc, Hs = T.Hs;
    const cplx hc = {T.hr, T.hi};
    const double a2 = A.re * A.re + A.im * A.im, b2 = Ab.re * Ab.re + Ab.im * Ab.im;
    const double zr = A.re * Ab.re + A.im * Ab.im, zi = A.re * Ab.im - A.im * Ab.re;  // conj(A) Abar
    const double R = 0.5 * ((a2 + b2) * Hc + (a2 - b2) * hc.re - 2.0 * zr * Hs - 2.0 * zi * hc.im);
    lp.mul(R);
    if (GRAD) {
      const double w = -rcp_fast(R);
      const double hpc = Hc + hc.re, hmc = Hc - hc.re;
      // dR/dRe c_k - i dR/dIm c_k = lc B_k and the same for cbar with lb, where
      // lc = hpc conj(A) - (Hs + i Hsin) conj(Abar), lb = hmc conj(Abar) - (Hs - i Hsin) conj(A)
      // (the event's factor w = -1/R included)
      const cplx lc = {w * (hpc * A.re - Hs * Ab.re - hc.im * Ab.im), w * (-hpc * A.im + Hs * Ab.im - hc.im * Ab.re)};
      const cplx lb = {w * (hmc * Ab.re - Hs * A.re + hc.im * A.im), w * (-hmc * Ab.im + Hs * A.im + hc.im * A.re)};
      td4_sum_grad<S, 0>(pt, lc, acc + 1);
      td4_sum_grad<S, 1>(pt, lb, acc + 1);
      acc[P - 1] += w * 0.5 * ((a2 - b2) * T.dr - 2.0 * zi * T.di);
      acc[P] += w * 0.5 * ((a2 + b2) * T.dHc - 2.0 * zr * T.dHs);
    }
  }
  acc[0] = -lp.log();
  block_sum_row<NV>(acc, lds, part + ((int64_t)f * nch + ch) * NV);
}

// R(x_i, t_i) / I per event (I: the level-2 step's output): the events pass's
// own point, sums and time functions, one event per thread.  A generic kernel
// with the structure at run time kept its amplitude arrays in scratch memory:
// 1M events, ten amplitudes and their ten mirror images, 172 us a call
// against 45 here, both with the 9 us of the normalization's level-2 step.
template <class S>
__device__ inline void td4_eval_body(const Td4Const& tc, const Td4Table* __restrict__ tab,
                                     const double* __restrict__ ev, int64_t ld, int64_t n,
                                     const double* __restrict__ norm, double* __restrict__ p) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const Td4Table& tb = *tab;
  TimeFns T;
  time_fns<false, true>(tb.tk, tc.wa, tc.wL, tb.x, tb.y, ev[5 * ld + i], T);
  Td4Point<S> pt;
  td4_point_s<S, true>(tc, tb, ev[i], ev[ld + i], ev[2 * ld + i], ev[3 * ld + i], ev[4 * ld + i], pt);
  const cplx A = td4_sum<S, 0>(pt, tb.c), Ab = td4_sum<S, 1>(pt, tb.cb);
  const double a2 = A.re * A.re + A.im * A.im, b2 = Ab.re * Ab.re + Ab.im * Ab.im;
  const double zr = A.re * Ab.re + A.im * Ab.im, zi = A.re * Ab.im - A.im * Ab.re;
  const double R = 0.5 * ((a2 + b2) * T.Hc + (a2 - b2) * T.hr - 2.0 * zr * T.Hs - 2.0 * zi * T.hi);
  p[i] = R / *norm;
}

// ------------------------------------------------------ four-body phase space
// Two-body momentum q(m; ma, mb) and the phase-space weight of (m12, m34)
// with the angles uniform: q(M; m12, m34) q(m12; m1, m2) q(m34; m3, m4).
// Contraction is off: the weight decides accept-reject draws and is the same
// plain IEEE evaluation on the host and the device.
__host__ __device__ inline double td4_q(double m, double ma, double mb) {
#pragma clang fp contract(off)
  const double l = (m * m - (ma + mb) * (ma + mb)) * (m * m - (ma - mb) * (ma - mb));
  return sqrt(l > 0.0 ? l : 0.0) / (2.0 * m);
}
__host__ __device__ inline double td4_ps_weight(const Td4Const& tc, double m12, double m34) {
#pragma clang fp contract(off)
  return td4_q(tc.M, m12, m34) * td4_q(m12, tc.m1, tc.m2) * td4_q(m34, tc.m3, tc.m4);
}

// Unweighted phase-space point i (m12, m34, cos theta12, cos theta34, phi):
// attempt a takes (u1, u2) from counter (i, s0 + 3a, 2), (u3, u4) from
// (i, s0 + 3a + 1, 2) and (u5, u6) from (i, s0 + 3a + 2, 2); (m12, m34)
// uniform in [m1 + m2, M - m3 - m4] x [m3 + m4, M - m1 - m2] is kept when
// m12 + m34 < M and u3 wmax < weight; then c12 = 2 u4 - 1, c34 = 2 u5 - 1,
// phi = (2 u6 - 1) pi.  false when no attempt is kept.
__device__ inline bool td4_ps_point(const Td4Const& tc, int64_t i, uint32_t k0, uint32_t k1, uint32_t s0,
                                    int max_attempts, double (&x)[5]) {
#pragma clang fp contract(off)
  const double lo12 = tc.m1 + tc.m2, hi12 = tc.M - tc.m3 - tc.m4;
  const double lo34 = tc.m3 + tc.m4, hi34 = tc.M - tc.m1 - tc.m2;
  for (int a = 0; a < max_attempts; ++a) {
    double u1, u2, u3, u4, u5, u6;
    philox_uniforms((uint64_t)i, s0 + 3u * a, 2u, k0, k1, u1, u2);
    philox_uniforms((uint64_t)i, s0 + 3u * a + 1u, 2u, k0, k1, u3, u4);
    philox_uniforms((uint64_t)i, s0 + 3u * a + 2u, 2u, k0, k1, u5, u6);
    const double m12 = lo12 + u1 * (hi12 - lo12);
    const double m34 = lo34 + u2 * (hi34 - lo34);
    if (m12 + m34 < tc.M && u3 * tc.ps_wmax < td4_ps_weight(tc, m12, m34)) {
      x[0] = m12;
      x[1] = m34;
      x[2] = 2.0 * u4 - 1.0;
      x[3] = 2.0 * u5 - 1.0;
      x[4] = (2.0 * u6 - 1.0) * 3.14159265358979323846;
      return true;
    }
  }
  return false;
}

// (|A| + |Abar|)^2 at one point of the model (the bound of the rate at t = 0).
template <class S>
__device__ inline double td4_env(const Td4Const& tc, const Td4Table& tb, double m12, double m34, double c12,
                                 double c34, double phi) {
  constexpr int K = S::K;
  cplx B[K];
  td4_basis_s<S>(tc, tb, m12, m34, c12, c34, phi, B);
  cplx A = {0.0, 0.0}, Ab = {0.0, 0.0};
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const cplx p = cmul({tb.c[k][0], tb.c[k][1]}, B[k]);
    const cplx q = cmul({tb.cb[k][0], tb.cb[k][1]}, B[k]);
    A = {A.re + p.re, A.im + p.im};
    Ab = {Ab.re + q.re, Ab.im + q.im};
  }
  const double e = sqrt(A.re * A.re + A.im * A.im) + sqrt(Ab.re * Ab.re + Ab.im * Ab.im);
  return e * e;
}

// Toy events of the model by accept-reject with importance sampling of the
// pair masses: event i, attempt a takes (u1, u2) ... (u9, u10) from Philox
// counters (i, 5a + j, word 4), j = 0..4, key (k0, k1): m12 from the r12
// proposal with selector u1 and position u3, m34 from the r34 proposal with
// u2 and u4 (Td4Proposal), c12 = 2 u5 - 1, c34 = 2 u6 - 1, phi = (2 u7 - 1) pi,
// t = -ln(1 - u8)/lam with lam = G (1 - |y|); kept when
// u9 W q12(m12) q34(m34) e^{-lam t} < w(m12, m34) R, w the phase-space weight
// and R the unconvolved rate (at most e^{-lam t} (|A| + |Abar|)^2), so W
// must bound w (|A| + |Abar|)^2 / (q12 q34).  The measured time adds sigma
// times a Box-Muller normal from counter (i, 0, 5).  bad[0] counts kept
// events above the bound, bad[1] events left NaN.
template <class S>
__device__ inline void td4_gen_body(const Td4Const& tc, const Td4Table* __restrict__ tab, const Td4Proposal& pr,
                                    uint32_t k0, uint32_t k1, int64_t n, const double* __restrict__ Wp, int per_wave,
                                    int max_attempts, double* __restrict__ ev, int64_t ld,
                                    unsigned long long* __restrict__ bad) {
#pragma clang fp contract(off)
  constexpr int K = S::K;
  __shared__ AcceptLds lds;
  const double W = *Wp;
  if (!(W > 0.0 && W < __builtin_inf())) return;  // the host reports it
  const Td4Table& tb = *tab;
  const double G = tc.gamma, x = tb.x, y = tb.y;
  const double lam = G * (1.0 - fabs(y));
  double m12, m34, c12, c34, phi, t, ratio;
  accept_reject(
      lds, n, per_wave, max_attempts,
      [&](int64_t i, int a) {
#pragma clang fp contract(off)
        double u1, u2, u3, u4, u5, u6, u7, u8, u9, u10;
        philox_uniforms((uint64_t)i, 5u * a, 4u, k0, k1, u1, u2);
        philox_uniforms((uint64_t)i, 5u * a + 1u, 4u, k0, k1, u3, u4);
        m12 = td4_prop_draw(pr.p12, u1, u3);
        m34 = td4_prop_draw(pr.p34, u2, u4);
        if (!(m12 + m34 < tc.M)) return false;
        const double w = td4_ps_weight(tc, m12, m34);
        if (!(w > 0.0)) return false;
        philox_uniforms((uint64_t)i, 5u * a + 2u, 4u, k0, k1, u5, u6);
        philox_uniforms((uint64_t)i, 5u * a + 3u, 4u, k0, k1, u7, u8);
        philox_uniforms((uint64_t)i, 5u * a + 4u, 4u, k0, k1, u9, u10);
        c12 = 2.0 * u5 - 1.0;
        c34 = 2.0 * u6 - 1.0;
        phi = (2.0 * u7 - 1.0) * 3.14159265358979323846;
        t = -log1p(-u8) / lam;
        cplx B[K];
        td4_basis_s<S>(tc, tb, m12, m34, c12, c34, phi, B);
        cplx A = {0.0, 0.0}, Ab = {0.0, 0.0};
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const cplx p = cmul({tb.c[k][0], tb.c[k][1]}, B[k]);
          const cplx q = cmul({tb.cb[k][0], tb.cb[k][1]}, B[k]);
          A = {A.re + p.re, A.im + p.im};
          Ab = {Ab.re + q.re, Ab.im + q.im};
        }
        const double a2 = A.re * A.re + A.im * A.im, b2 = Ab.re * Ab.re + Ab.im * Ab.im;
        const double zr = A.re * Ab.re + A.im * Ab.im, zi = A.re * Ab.im - A.im * Ab.re;
        const double gt = G * t;
        const double ep = exp(y * gt), em = exp(-y * gt);
        double sx, cx;
        sincos(x * gt, &sx, &cx);
        const double R = 0.5 * exp(-gt) *
                         ((a2 + b2) * (0.5 * (ep + em)) + (a2 - b2) * cx - 2.0 * zr * (0.5 * (ep - em)) -
                          2.0 * zi * sx);
        const double q12 = td4_prop_density(pr.p12, m12), q34 = td4_prop_density(pr.p34, m34);
        const double e = sqrt(a2) + sqrt(b2);
        ratio = w * (e * e) / (q12 * q34);
        return u9 * W * q12 * q34 * exp(-lam * t) < w * R;
      },
      [&](int64_t i) {
#pragma clang fp contract(off)
        double v1, v2;
        philox_uniforms((uint64_t)i, 0u, 5u, k0, k1, v1, v2);
        ev[i] = m12;
        ev[ld + i] = m34;
        ev[2 * ld + i] = c12;
        ev[3 * ld + i] = c34;
        ev[4 * ld + i] = phi;
        ev[5 * ld + i] = t + tb.sigma * (sqrt(-2.0 * log1p(-v1)) * cos(2.0 * 3.14159265358979323846 * v2));
        if (ratio > W) atomicAdd(bad, 1ull);
      },
      [&](int64_t i) {
        for (int j = 0; j < 6; ++j) ev[j * ld + i] = __builtin_nan("");
        atomicAdd(bad + 1, 1ull);
      });
}

// Largest w (|A| + |Abar|)^2 / (q12 q34) over the points of a phase-space
// sample (the generator's bound; bits of a non-negative double) in *vmax.
template <class S>
__device__ inline void td4_envmax_body(const Td4Const& tc, const Td4Table* __restrict__ tab, const Td4Proposal& pr,
                                       const double* __restrict__ mc, int64_t ld, int64_t n,
                                       unsigned long long* __restrict__ vmax) {
  const Td4Table& tb = *tab;
  double m = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
    const double m12 = mc[i], m34 = mc[ld + i];
    const double e = td4_env<S>(tc, tb, m12, m34, mc[2 * ld + i], mc[3 * ld + i], mc[4 * ld + i]);
    const double r = td4_ps_weight(tc, m12, m34) * e / (td4_prop_density(pr.p12, m12) * td4_prop_density(pr.p34, m34));
    m = fmax(m, r);
  }
  block_max(m, vmax);
}

// M = sum over the phase-space sample of B_i conj(B_j) (Gram), one row per
// workgroup and fit (fits with sel[f] == 0 are skipped, sel may be null).
template <class S>
__device__ inline void td4_gram_body(const Td4Const& tc, const Td4Table* __restrict__ tabs,
                                     const int* __restrict__ sel, const double* __restrict__ mc, int64_t ld,
                                     int64_t n, int chunk, int64_t nch, int n_fits, double* __restrict__ part) {
  constexpr int K = S::K;
  using G = Gram<K>;
  __shared__ double lds[G::LDS];
  int64_t ch;
  int f;
  if (!td4_block_item(nch, n_fits, ch, f)) return;
  if (sel && !sel[f]) return;
  G g;
  g.init(lds);
  const int64_t base = ch * chunk;
  const int64_t end = base + chunk < n ? base + chunk : n;
  for (int64_t i = base + (threadIdx.x & ~63); i < end; i += kBlock) {
    const int64_t p = i + (threadIdx.x & 63);
    const int64_t q = p < end ? p : i;
    int zero = 0;
    asm volatile("" : "+s"(zero));
    cplx B[K];
    td4_basis_s<S>(tc, tabs[f + zero], mc[q], mc[ld + q], mc[2 * ld + q], mc[3 * ld + q], mc[4 * ld + q], B);
    double re[K], im[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      re[k] = B[k].re;
      im[k] = B[k].im;
    }
    if (p >= end) {
#pragma unroll
      for (int k = 0; k < K; ++k) re[k] = im[k] = 0.0;
    }
    g.add(re, im, lds);
  }
  g.reduce(lds, part + ((int64_t)f * nch + ch) * 2 * gram_count(K));
}

}  // namespace fn

// Kernels for shape S (used by the generated source).
#define FN_TD4_EVENTS(NAME, S, GRAD)                                                                           \
  extern "C" __global__ __launch_bounds__(fn::kBlock) __attribute__((amdgpu_waves_per_eu(2))) void NAME(        \
      fn::Td4Const tc, const fn::Td4Table* __restrict__ tabs, const int* __restrict__ status,                  \
      const double* __restrict__ ev, int64_t ld, int64_t n, int chunk, int64_t nch, int n_fits,                \
      double* __restrict__ part) {                                                                              \
    fn::td4_events_body<S, GRAD>(tc, tabs, status, ev, ld, n, chunk, nch, n_fits, part);                       \
  }
#define FN_TD4_EVAL(NAME, S)                                                                                   \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void NAME(                                                \
      fn::Td4Const tc, const fn::Td4Table* __restrict__ tab, const double* __restrict__ ev, int64_t ld,        \
      int64_t n, const double* __restrict__ norm, double* __restrict__ p) {                                     \
    fn::td4_eval_body<S>(tc, tab, ev, ld, n, norm, p);                                                          \
  }
#define FN_TD4_GRAM(NAME, S)                                                                                   \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void NAME(                                                \
      fn::Td4Const tc, const fn::Td4Table* __restrict__ tabs, const int* __restrict__ sel,                     \
      const double* __restrict__ mc, int64_t ld, int64_t n, int chunk, int64_t nch, int n_fits,                \
      double* __restrict__ part) {                                                                              \
    fn::td4_gram_body<S>(tc, tabs, sel, mc, ld, n, chunk, nch, n_fits, part);                                  \
  }
#define FN_TD4_GEN(ENVMAX, GEN, S)                                                                             \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void ENVMAX(                                             \
      fn::Td4Const tc, const fn::Td4Table* __restrict__ tab, fn::Td4Proposal pr, const double* __restrict__ mc, \
      int64_t ld, int64_t n, unsigned long long* __restrict__ vmax) {                                          \
    fn::td4_envmax_body<S>(tc, tab, pr, mc, ld, n, vmax);                                                      \
  }                                                                                                            \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void GEN(                                                \
      fn::Td4Const tc, const fn::Td4Table* __restrict__ tab, fn::Td4Proposal pr, uint32_t k0, uint32_t k1,     \
      int64_t n, const double* __restrict__ W, int per_wave, int max_attempts, double* __restrict__ ev,        \
      int64_t ld, unsigned long long* __restrict__ bad) {                                                      \
    fn::td4_gen_body<S>(tc, tab, pr, k0, k1, n, W, per_wave, max_attempts, ev, ld, bad);                       \
  }
