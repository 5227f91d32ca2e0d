// Device code of the one-observable mixture shared by the single-fit kernels
// (mix1d.hip) and the batched ones (batch.hip): the prologue table, the
// component shapes, the per-chunk evaluation and the level-2 step.
#pragma once
#include <type_traits>

#include <cmath>

#include "device_common.hpp"
#include "fastmath.hpp"

namespace fn {

// Lower incomplete gamma function gamma(a, y), y >= 0, for a = 3/2 and 5/2.
// Series y^a e^-y sum_n y^n / (a (a+1) ... (a+n)) below y = 1, closed forms
// through erf above (gamma(3/2,y) = sqrt(pi)/2 erf(sqrt y) - sqrt(y) e^-y and
// gamma(5/2,y) = 3/2 gamma(3/2,y) - y^(3/2) e^-y).
__device__ inline double lower_gamma_half(int twice_a, double y) {
  const double a = 0.5 * twice_a;
  if (y <= 0.0) return 0.0;
  if (y < 1.0) {
    double term = 1.0 / a, sum = term;
    for (int n = 1; n < 60; ++n) {
      term *= y / (a + n);
      sum += term;
      if (term < 1e-18 * sum) break;
    }
    return pow(y, a) * exp(-y) * sum;
  }
  const double ry = sqrt(y);
  const double g32 = 0.88622692545275801365 * erf(ry) - ry * exp(-y);
  if (twice_a == 3) return g32;
  return 1.5 * g32 - y * ry * exp(-y);
}

// theta -> component k of the per-fit table: its fraction, 1/N_k and
// d ln N_k / d(its parameters) from its closed-form integral on [lo, hi], and
// its shape constants (written in place).  Returns false when the parameters
// do not define a density.
__device__ inline bool mix1d_component(const Mix1dConst& mc, const double* __restrict__ th, int k, Mix1dTable& t) {
  bool ok = true;
  const double lo = mc.lo, hi = mc.hi;
  t.a[k] = 0.0; t.b[k] = 0.0; t.c[k] = 0.0;
  if (k < mc.K - 1) {
    t.frac[k] = th[mc.fidx[k]];
  } else {
    // the last component takes 1 - sum of the others, subtracted in order
    double rest = 1.0;
    for (int j = 0; j < mc.K - 1; ++j) rest -= th[mc.fidx[j]];
    t.frac[k] = rest;
  }
  const double p0 = th[mc.pidx[k][0]];
  const double p1 = mc.npar[k] > 1 ? th[mc.pidx[k][1]] : 0.0;
  double N = 0.0, d0 = 0.0, d1 = 0.0;
  switch (mc.type[k]) {
    case kGauss: {
      const double mu = p0, sg = p1;
      if (!(sg > 0.0)) { ok = false; break; }
      const double s2 = sg * 1.41421356237309504880;
      const double A = (lo - mu) / s2, B = (hi - mu) / s2;
      double D;
      if (A > 0.0) D = erfc(A) - erfc(B);
      else if (B < 0.0) D = erfc(-B) - erfc(-A);
      else D = erf(B) - erf(A);
      N = sg * 1.25331413731550025121 * D;  // sqrt(pi/2)
      const double eA = exp(-A * A), eB = exp(-B * B);
      d0 = (eA - eB) / N;
      d1 = 1.0 / sg + 1.41421356237309504880 * (A * eA - B * eB) / N;
      t.a[k] = mu; t.b[k] = 1.0 / sg;
      break;
    }
    case kExp: {
      const double tau = p0, D = hi - lo;
      const double td = tau * D;
      const double up = expm1(td), dn = -expm1(-td);
      if (fabs(tau) < 1e-12) N = D * (1.0 + 0.5 * tau * (hi + lo));
      else N = exp(tau * lo) * up / tau;
      if (fabs(td) < 1e-3) d0 = 0.5 * (hi + lo) + tau * D * D / 12.0 - td * td * td * D / 720.0;
      else d0 = lo + D / dn - 1.0 / tau;
      t.a[k] = tau;
      // the events passes' form, relative to the value at the mean d0 (mix_term):
      // 1 over the integral relative to the end of the range where the shape is
      // largest, taken to the mean by a factor between 1/e and 1
      const bool flat = fabs(tau) < 1e-12;
      t.b[k] = (flat ? 1.0 : tau) / (flat ? D * (1.0 - 0.5 * fabs(td)) : (tau > 0.0 ? dn : up)) *
               exp_fast(tau * (d0 - (tau > 0.0 ? hi : lo)));
      break;
    }
    case kArgus: {
      const double m0 = p0, c = p1;
      if (!(m0 > 0.0) || !(c < 0.0)) { ok = false; break; }
      const double kk = -c, im2 = 1.0 / (m0 * m0);
      const double wlo = fmax(0.0, 1.0 - lo * lo * im2), whi = fmax(0.0, 1.0 - hi * hi * im2);
      const double k32 = pow(kk, -1.5), k52 = pow(kk, -2.5), h = 0.5 * m0 * m0;
      N = h * k32 * (lower_gamma_half(3, kk * wlo) - lower_gamma_half(3, kk * whi));
      const double dNc = h * k52 * (lower_gamma_half(5, kk * wlo) - lower_gamma_half(5, kk * whi));
      const double im3 = im2 / m0;
      const double flo = wlo > 0.0 ? sqrt(wlo) * exp(-kk * wlo) * 2.0 * lo * lo * im3 : 0.0;
      const double fhi = whi > 0.0 ? sqrt(whi) * exp(-kk * whi) * 2.0 * hi * hi * im3 : 0.0;
      const double dNm = 2.0 * N / m0 + h * (flo - fhi);
      d0 = dNm / N;
      d1 = dNc / N;
      t.a[k] = im2; t.b[k] = c; t.c[k] = 1.0 / m0;
      break;
    }
    case kBW: {
      const double m0 = p0, g = p1;
      if (!(g > 0.0)) { ok = false; break; }
      const double hg = 0.5 * g, uh = (hi - m0) / hg, ul = (lo - m0) / hg;
      N = (atan(uh) - atan(ul)) / hg;
      const double ih = 1.0 / (1.0 + uh * uh), il = 1.0 / (1.0 + ul * ul);
      const double dNm = (il - ih) / (hg * hg);
      const double dNg = -N / g + (-uh * ih + ul * il) / (g * hg);
      d0 = dNm / N;
      d1 = dNg / N;
      t.a[k] = m0; t.b[k] = hg * hg; t.c[k] = g;
      break;
    }
    default:
      ok = false;
  }
  if (!(N > 0.0) || !isfinite(N)) ok = false;
  t.invN[k] = 1.0 / N;
  t.dlnN[k][0] = d0;
  t.dlnN[k][1] = d1;
  return ok;
}

// The table entries past the components, the yield (extended likelihood) and
// the validity flag, by one thread once the components are in (the single-fit
// prologue and batch_head give each component its own); ok: every component's check.
__device__ inline void mix1d_table_rest(const Mix1dConst& mc, const double* __restrict__ th, bool ok, Mix1dTable& t) {
  for (int k = mc.K; k < kMixMaxComp; ++k) {
    t.frac[k] = 0.0; t.invN[k] = 0.0; t.a[k] = 0.0; t.b[k] = 0.0; t.c[k] = 0.0;
    t.dlnN[k][0] = 0.0; t.dlnN[k][1] = 0.0;
  }
  t.yield = mc.yidx >= 0 ? th[mc.yidx] : 0.0;
  if (mc.yidx >= 0 && !(t.yield > 0.0 && isfinite(t.yield))) ok = false;
  t.valid = ok ? 1.0 : 0.0;
}

// Component shape s(x) and d ln s / d(its parameters).
template <bool GRAD>
__device__ inline double mix_shape(int type, const Mix1dTable& t, int k, double x,
                                   double& dl0, double& dl1) {
  switch (type) {
    case kGauss: {
      const double z = (x - t.a[k]) * t.b[k];
      if (GRAD) { dl0 = z * t.b[k]; dl1 = z * z * t.b[k]; }
      return exp(-0.5 * z * z);
    }
    case kExp: {
      if (GRAD) { dl0 = x; dl1 = 0.0; }
      return exp(t.a[k] * x);
    }
    case kArgus: {
      const double w = 1.0 - x * x * t.a[k];
      if (!(w > 0.0)) { if (GRAD) { dl0 = 0.0; dl1 = 0.0; } return 0.0; }
      if (GRAD) { dl0 = (0.5 / w + t.b[k]) * 2.0 * x * x * t.a[k] * t.c[k]; dl1 = w; }
      return x * sqrt(w) * exp(t.b[k] * w);
    }
    default: {  // kBW
      const double d = x - t.a[k];
      const double s = rcp_fast(__builtin_fma(d, d, t.b[k]));
      if (GRAD) { dl0 = 2.0 * d * s; dl1 = -0.5 * t.c[k] * s; }
      return s;
    }
  }
}

// Type signature of a mixture compiled for its component types: 0 for the
// generic passes (types read at run time), 1 + t0 for one component of type
// t0, 5 + 4 t0 + t1 for two (types in MixType order).  The per-event passes of
// mixtures of one or two components are instantiated for each signature, so
// that each component's shape code is selected at compile time.
constexpr int kMixSigCount = 21;
__host__ __device__ constexpr int mix_sig_K(int sig) { return sig == 0 ? 0 : (sig < 5 ? 1 : 2); }
__host__ __device__ constexpr int mix_sig_type(int sig, int k) {
  return sig < 5 ? sig - 1 : (k == 0 ? (sig - 5) / 4 : (sig - 5) % 4);
}

// The component of a two-component signature whose exponential the other's is
// divided by (mix1d_typed_chunk), or -1: an exponential next to a Gaussian, an
// Argus shape or another exponential.
__host__ __device__ constexpr int mix_sig_pivot(int sig) {
  if (mix_sig_K(sig) != 2) return -1;
  const int t0 = mix_sig_type(sig, 0), t1 = mix_sig_type(sig, 1);
  if (t1 == kExp && t0 != kBW) return 1;
  if (t0 == kExp && t1 != kBW) return 0;
  return -1;
}

// A component's shape at x as pre e^arg, and its derivatives' factors:
// d ln s / d(its parameters) are alpha0 m0 and alpha1 m1, alpha constants of
// the fit (mix_alpha).  An exponential is taken relative to its value at its
// mean d ln N / d tau, e^(tau (x - mean)), which is at most e times that on the
// range whatever the slope (mix_invn: its weight in these units), and its
// derivative's sum needs no second term (mix_dlnn).  Relative to x = 0 it reaches
// e^709 on legal ranges, where sums weighted by it overflow and its weight is
// subnormal, and both parts of the derivative grow with the range's distance
// from zero.
struct MixTerm {
  double pre, arg, m0, m1;
};
template <int TYPE>
__device__ __forceinline__ MixTerm mix_term(const Mix1dTable& t, int k, double x) {
  MixTerm r;
  if (TYPE == kGauss) {
    const double z = (x - t.a[k]) * t.b[k];
    r = {1.0, -0.5 * z * z, z, z * z};
  } else if (TYPE == kExp) {
    const double d = x - t.dlnN[k][0];
    r = {1.0, t.a[k] * d, d, 0.0};
  } else if (TYPE == kArgus) {
    const double xx = x * x, w = 1.0 - xx * t.a[k];
    const bool in = w > 0.0;
    const double wi = in ? w : 1.0;
    r.pre = in ? x * sqrt(wi) : 0.0;
    r.arg = in ? t.b[k] * wi : -__builtin_inf();  // e^-inf: the pivot's own argument is the larger one
    r.m0 = in ? (0.5 * rcp_acc(wi) + t.b[k]) * xx : 0.0;
    r.m1 = in ? w : 0.0;
  } else {
    const double d = x - t.a[k];
    const double s = rcp_fast(__builtin_fma(d, d, t.b[k]));
    r = {s, 0.0, d * s, s};
  }
  return r;
}
template <int TYPE>
__device__ __forceinline__ double mix_alpha(const Mix1dTable& t, int k, int j) {
  if (TYPE == kGauss) return t.b[k];
  if (TYPE == kArgus) return j == 0 ? 2.0 * t.a[k] * t.c[k] : 1.0;
  if (TYPE == kBW) return j == 0 ? 2.0 : -0.5 * t.c[k];
  return 1.0;
}

// 1 / N_k and d ln N_k / d(parameter j) in mix_term's units.
__device__ __forceinline__ double mix_invn(int type, const Mix1dTable& t, int k) {
  return type == kExp ? t.b[k] : t.invN[k];
}
__device__ __forceinline__ double mix_dlnn(int type, const Mix1dTable& t, int k, int j) {
  return type == kExp ? 0.0 : t.dlnN[k][j];
}

// slot[s] += w * dP/d(slot s) at one point: shape parameters of component k at
// 2k, 2k + 1 (dP = f_k u_k (d ln s_k - d ln N_k)), fraction k < K-1 at
// 2 KMAX + k (dP = u_k - u_{K-1}, the last component taking 1 - sum f).
template <int KMAX>
__device__ __forceinline__ void mix1d_add_dp(int K, const Mix1dTable& t, const double (&u)[KMAX],
                                             const double (&dl)[KMAX][2], double w, double* slot) {
  double ul = 0.0;
#pragma unroll
  for (int k = 0; k < KMAX; ++k)
    if (k == K - 1) ul = u[k];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    if (k < K) {
      const double wu = w * t.frac[k] * u[k];
      slot[2 * k] += wu * (dl[k][0] - t.dlnN[k][0]);
      slot[2 * k + 1] += wu * (dl[k][1] - t.dlnN[k][1]);
      if (k < K - 1) slot[2 * KMAX + k] += w * (u[k] - ul);
    }
  }
}

// One chunk of events of a mixture of one or two components of known types ->
// one partial row.  P = sum_k g_k s_k with g_k = f_k / N_k; per event the sums
// are V_k = sum v, sum v m0 and sum v m1 with v = -s_k / P, and the slots
// follow from them once per thread: shape slots f_k/N_k (alpha sum v m - V d ln
// N), fraction slot V_0/N_0 - V_1/N_1.  With a pivot p (mix_sig_pivot) the
// density is e^arg_p (g_p + g_o pre_o e^d), d = arg_o - arg_p: one exponential
// serves both components, and sum arg_p is the pivot's parameter times sum (x -
// mean).  d is at most |tau| times the range's length, and where that exceeds
// kPivotMax the larger of the two arguments is taken out instead, so that no
// factor of the two exceeds 1: e^d overflows from 709 on, and d's rounding error
// grows with it before that.  Events that overflow nevertheless lie outside the
// range, and the wave takes its chunk again in that form.
// The Gaussian and exponential mixture takes 43 VALU instructions per event (52
// relative to the larger argument) instead of 112 with an exponential for each:
// NLL and gradient of 2^26 events 207 -> 149 us, 130 with the loads below (their
// bytes alone take 88 at 6.1 TB/s) and a tenth more at slopes past the line; 512
// toy fits to convergence 3.87 -> 3.23 ms.
constexpr double kPivotMax = 16.0;
template <bool GRAD, int SIG>
__device__ inline void mix1d_typed_chunk(const Mix1dConst& mc, const Mix1dTable* __restrict__ tabp,
                                         const double* __restrict__ x, int64_t n, int64_t chunk_idx, int chunk,
                                         double* __restrict__ out_row, double* lds) {
  constexpr int KMAX = 2;
  constexpr int NV = GRAD ? mix_nv(KMAX) : 1;
  constexpr int K = mix_sig_K(SIG), PV = mix_sig_pivot(SIG);
  constexpr int T0 = mix_sig_type(SIG, 0), T1 = K == 2 ? mix_sig_type(SIG, 1) : T0;
  const Mix1dTable& t = *tabp;
  const double i0 = mix_invn(T0, t, 0), i1 = K == 2 ? mix_invn(T1, t, 1) : 0.0;
  const double g0 = t.frac[0] * i0, g1 = K == 2 ? t.frac[1] * i1 : 0.0;
  double V0, A0, B0, V1, A1, B1, X, M;
  const int64_t base = chunk_idx * chunk;
  const int64_t end = base + chunk < n ? base + chunk : n;
  LogProd lp;  // -sum ln P enters acc[0] once per thread, at the end
  // the chunk's events; larger: relative to the larger argument (std::true_type) or to the pivot's
  auto pass = [&](auto larger) {
    V0 = A0 = B0 = V1 = A1 = B1 = X = M = 0.0;
    lp = LogProd{};
    auto event = [&](double xv) {
      const MixTerm a = mix_term<T0>(t, 0, xv), b = mix_term<T1>(t, 1, xv);
      double s0, s1 = 0.0;
      if constexpr (PV >= 0) {
        const MixTerm &p = PV == 1 ? b : a, &o = PV == 1 ? a : b;
        const double d = o.arg - p.arg;
        double so, sp = 1.0;
        X += p.m0;
        if constexpr (decltype(larger)::value) {
          const double e = exp_fast(-fabs(d));
          const bool up = d > 0.0;
          so = (PV == 1 ? T0 : T1) == kArgus ? (up ? o.pre : o.pre * e) : (up ? 1.0 : e);
          sp = up ? e : 1.0;
          M += up ? d : 0.0;
        } else {
          so = o.pre * exp_fast(d);
        }
        s0 = PV == 1 ? so : sp;
        s1 = PV == 1 ? sp : so;
      } else {
        s0 = T0 == kBW ? a.pre : a.pre * exp_fast(a.arg);
        if (K == 2) s1 = T1 == kBW ? b.pre : b.pre * exp_fast(b.arg);
      }
      const double P = K == 2 ? __builtin_fma(g1, s1, g0 * s0) : g0 * s0;
      lp.mul(P);
      if (GRAD) {
        const double w = -rcp_fast(P);
        const double v0 = w * s0, v1 = w * s1;
        V0 += v0;
        A0 = __builtin_fma(v0, a.m0, A0);
        if (T0 != kExp) B0 = __builtin_fma(v0, a.m1, B0);
        if (K == 2) {
          V1 += v1;
          A1 = __builtin_fma(v1, b.m0, A1);
          if (T1 != kExp) B1 = __builtin_fma(v1, b.m1, B1);
        }
      }
    };
    // groups of four events per thread, the next group's loads in flight while
    // one is worked on (one load at a time left the pass waiting for memory),
    // then the rest one by one
    constexpr int U = 4;
    const int64_t full = (end - base) / (U * kBlock);
    const double* xp = x + base + threadIdx.x;
    double nx[U];
    if (full > 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) nx[u] = xp[u * kBlock];
    }
    for (int64_t g = 0; g < full; ++g) {
      double cur[U];
#pragma unroll
      for (int u = 0; u < U; ++u) cur[u] = nx[u];
      xp += U * kBlock;
      if (g + 1 < full) {
#pragma unroll
        for (int u = 0; u < U; ++u) nx[u] = xp[u * kBlock];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) event(cur[u]);
    }
    for (int64_t i = base + full * (U * kBlock) + threadIdx.x; i < end; i += kBlock) event(x[i]);
  };
  bool steep = false;
  if constexpr (PV >= 0) steep = fabs(t.a[PV]) * (mc.hi - mc.lo) > kPivotMax;
  if (__builtin_expect(!steep, 1)) {
    pass(std::false_type{});
    if constexpr (PV >= 0) steep = __any(!(lp.m < __builtin_inf()));
  }
  if constexpr (PV >= 0) {
    if (__builtin_expect(steep, 0)) pass(std::true_type{});
  }
  double acc[NV];
  acc[0] = -lp.log();
  if (PV >= 0) acc[0] -= __builtin_fma(t.a[PV >= 0 ? PV : 0], X, M);
  if (GRAD) {
    acc[1] = g0 * __builtin_fma(-V0, mix_dlnn(T0, t, 0, 0), mix_alpha<T0>(t, 0, 0) * A0);
    acc[2] = T0 == kExp ? 0.0 : g0 * __builtin_fma(-V0, t.dlnN[0][1], mix_alpha<T0>(t, 0, 1) * B0);
    acc[3] = acc[4] = acc[5] = acc[6] = 0.0;
    if (K == 2) {
      acc[3] = g1 * __builtin_fma(-V1, mix_dlnn(T1, t, 1, 0), mix_alpha<T1>(t, 1, 0) * A1);
      acc[4] = T1 == kExp ? 0.0 : g1 * __builtin_fma(-V1, t.dlnN[1][1], mix_alpha<T1>(t, 1, 1) * B1);
      acc[5] = V0 * i0 - V1 * i1;
    }
  }
  block_sum_row<NV>(acc, lds, out_row);
}

// d ln s / d(parameter j) of component k is this constant of the fit times m_j
// of its MixTerm (types at run time).
__device__ __forceinline__ double mix_alpha_of(int type, const Mix1dTable& t, int k, int j) {
  if (type == kGauss) return mix_alpha<kGauss>(t, k, j);
  if (type == kArgus) return mix_alpha<kArgus>(t, k, j);
  if (type == kBW) return mix_alpha<kBW>(t, k, j);
  return 1.0;
}

// The same for three components or more (KMAX at most), whose types are read at
// run time, by branches that all lanes take alike: the sums V_k, sum v m0 and
// sum v m1 as above, U events per thread and round for each branch taken, the
// next round's events loaded ahead.  With the library's exponential, arrays for
// eight components and the slots formed per event, 2^25 events of two Gaussians
// and an exponential took 335 us; 187 now (1e6: 30.4 -> 22.1, 3001: 30.8 -> 28.1
// with the result on the host).
template <bool GRAD, int KMAX>
__device__ inline void mix1d_generic_chunk(const Mix1dConst& mc, const Mix1dTable* __restrict__ tabp,
                                           const double* __restrict__ x, int64_t n, int64_t chunk_idx, int chunk,
                                           double* __restrict__ out_row, double* lds) {
  constexpr int NV = GRAD ? mix_nv(KMAX) : 1;
  constexpr int U = GRAD ? (KMAX <= 4 ? 2 : 1) : 4;
  const int K = mc.K;
  const Mix1dTable& t = *tabp;
  double g[KMAX], V[KMAX], A[KMAX], B[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    g[k] = k < K ? t.frac[k] * mix_invn(mc.type[k], t, k) : 0.0;
    V[k] = A[k] = B[k] = 0.0;
  }
  const int64_t base = chunk_idx * chunk;
  const int64_t end = base + chunk < n ? base + chunk : n;
  LogProd lp;  // -sum ln P enters acc[0] once per thread, at the end
  double nx[U];
  auto load = [&](int64_t i) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = i + u * kBlock;
      nx[u] = x[j < end ? j : end - 1];
    }
  };
  if (base < end) load(base + threadIdx.x);
  for (int64_t i = base + threadIdx.x; i < end; i += U * kBlock) {
    double xv[U], P[U], s[U][KMAX], m0[U][KMAX], m1[U][KMAX];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      xv[u] = nx[u];
      P[u] = 0.0;
    }
    load(i + U * kBlock);
    // component k at the U events, its terms kept at column j
    auto component = [&](int k, int j, double gk) {
      auto shape = [&](auto type) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const MixTerm a = mix_term<decltype(type)::value>(t, k, xv[u]);
          s[u][j] = decltype(type)::value == kBW ? a.pre : a.pre * exp_fast(a.arg);
          m0[u][j] = a.m0;
          m1[u][j] = a.m1;
        }
      };
      const int type = mc.type[k];
      if (type == kGauss) shape(std::integral_constant<int, kGauss>{});
      else if (type == kExp) shape(std::integral_constant<int, kExp>{});
      else if (type == kArgus) shape(std::integral_constant<int, kArgus>{});
      else shape(std::integral_constant<int, kBW>{});
#pragma unroll
      for (int u = 0; u < U; ++u) P[u] = __builtin_fma(gk, s[u][j], P[u]);
    };
    if constexpr (GRAD) {
#pragma unroll
      for (int k = 0; k < KMAX; ++k)
        if (k < K) component(k, k, g[k]);
    } else {
      // nothing is kept per component: one copy of the shapes' code (unrolled,
      // its first pass through the instruction cache cost small samples 1.5 us)
#pragma unroll 1
      for (int k = 0; k < K; ++k) component(k, 0, t.frac[k] * mix_invn(mc.type[k], t, k));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool valid = u == 0 || i + u * kBlock < end;
      lp.mul(valid ? P[u] : 1.0);
      if (GRAD) {
        const double w = valid ? -rcp_fast(P[u]) : 0.0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
          if (k < K) {
            const double v = w * s[u][k];
            V[k] += v;
            A[k] = __builtin_fma(v, m0[u][k], A[k]);
            B[k] = __builtin_fma(v, m1[u][k], B[k]);
          }
        }
      }
    }
  }
  double acc[NV];
  acc[0] = -lp.log();
  if (GRAD) {
    double last = 0.0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
      if (k == K - 1) last = V[k] * mix_invn(mc.type[k], t, k);
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      const bool on = k < K;
      const int type = on ? mc.type[k] : kExp;
      acc[1 + 2 * k] = on ? g[k] * __builtin_fma(-V[k], mix_dlnn(type, t, k, 0), mix_alpha_of(type, t, k, 0) * A[k]) : 0.0;
      acc[2 + 2 * k] = type != kExp ? g[k] * __builtin_fma(-V[k], t.dlnN[k][1], mix_alpha_of(type, t, k, 1) * B[k]) : 0.0;
      acc[1 + 2 * KMAX + k] = k < K - 1 ? V[k] * mix_invn(type, t, k) - last : 0.0;
    }
  }
  block_sum_row<NV>(acc, lds, out_row);
}

// One chunk of events -> one partial row (shared by the single-fit and the
// batched launches so that both produce the same bits).  SIG: the type
// signature the code is compiled for (0: generic, KMAX components at most).
template <bool GRAD, int KMAX, int SIG = 0>
__device__ inline void mix1d_chunk(const Mix1dConst& mc, const Mix1dTable* __restrict__ tabp,
                                   const double* __restrict__ x, int64_t n, int64_t chunk_idx,
                                   int chunk, double* __restrict__ out_row, double* lds) {
  static_assert(SIG == 0 || KMAX == 2, "typed passes hold two components");
  if constexpr (SIG != 0) mix1d_typed_chunk<GRAD, SIG>(mc, tabp, x, n, chunk_idx, chunk, out_row, lds);
  else mix1d_generic_chunk<GRAD, KMAX>(mc, tabp, x, n, chunk_idx, chunk, out_row, lds);
}

// Binned data: bin b of nb uniform bins on [lo, hi] holds n_b events, and the
// density at its centre x_b = lo + (b + 1/2) Delta gives the expected count
// nu_b = N Delta P(x_b).  One chunk of bins -> one partial row:
//   STAT 0 (Poisson): [W, X, Y, dX slots, dY slots], W = sum n_b,
//                     X = sum_b P_b, Y = sum_b n_b ln P_b (N enters at the end)
//   STAT 1 (chi^2 over the bins with n_b > 0, N = *nptr):
//                     [W, C, D, dC slots], C = sum (n_b - nu_b)^2 / n_b,
//                     D = dC/dN = -2 Delta sum (n_b - nu_b) P_b / n_b
//   STAT 2:           [W] (the total count, when N = W for chi^2)
template <int KMAX, int STAT, bool GRAD>
__host__ __device__ constexpr int mix1d_binned_nv() {
  return STAT == 2 ? 1 : (GRAD ? 3 + (STAT == 0 ? 2 : 1) * (mix_nv(KMAX) - 1) : 3);
}

template <bool GRAD, int KMAX, int STAT>
__device__ inline void mix1d_binned_chunk(const Mix1dConst& mc, const Mix1dTable* __restrict__ tabp,
                                          const double* __restrict__ counts, int64_t nb, const double* nptr,
                                          int64_t chunk_idx, int chunk, double* __restrict__ out_row, double* lds) {
  constexpr int G = mix_nv(KMAX) - 1;
  constexpr int NV = mix1d_binned_nv<KMAX, STAT, GRAD>();
  const Mix1dTable& t = *tabp;
  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  const double delta = (mc.hi - mc.lo) / (double)nb;
  const double N = STAT == 1 ? (nptr ? *nptr : t.yield) : 0.0;
  const int64_t base = chunk_idx * chunk;
  const int64_t end = base + chunk < nb ? base + chunk : nb;
  for (int64_t b = base + threadIdx.x; b < end; b += kBlock) {
    const double n = counts[b];
    acc[0] += n;
    if (STAT == 2) continue;
    const double xv = mc.lo + ((double)b + 0.5) * delta;
    double u[KMAX], dl[KMAX][2];
    double P = 0.0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      u[k] = 0.0; dl[k][0] = 0.0; dl[k][1] = 0.0;
      if (k < mc.K) {
        u[k] = mix_shape<GRAD>(mc.type[k], t, k, xv, dl[k][0], dl[k][1]) * t.invN[k];
        P += t.frac[k] * u[k];
      }
    }
    if (STAT == 0) {
      acc[1] += P;
      const double cy = n != 0.0 ? n * rcp_fast(P) : 0.0;
      if (n != 0.0) acc[2] += n * log_fast(P);
      if (GRAD) {
        mix1d_add_dp<KMAX>(mc.K, t, u, dl, 1.0, acc + 3);
        mix1d_add_dp<KMAX>(mc.K, t, u, dl, cy, acc + 3 + G);
      }
    } else if (n > 0.0) {
      const double in = 1.0 / n;
      const double r = n - N * delta * P;  // n_b - nu_b
      acc[1] += r * r * in;
      acc[2] -= 2.0 * delta * r * P * in;
      if (GRAD) mix1d_add_dp<KMAX>(mc.K, t, u, dl, -2.0 * N * delta * r * in, acc + 3);
    }
  }
  block_sum_row<NV>(acc, lds, out_row);
}

// Gradient of parameter p from gradient slots (slots sharing a parameter are
// added in slot order).
__device__ inline double mix1d_param_grad(const Mix1dConst& mc, int kmax, const double* slots, int p) {
  double g = 0.0;
  for (int k = 0; k < mc.K; ++k) {
    for (int j = 0; j < mc.npar[k]; ++j)
      if (mc.pidx[k][j] == p) g += slots[2 * k + j];
    if (k < mc.K - 1 && mc.fidx[k] == p) g += slots[2 * kmax + k];
  }
  return g;
}

// Level 2 and the slot -> parameter map; with an expected yield nu (extended
// likelihood) NLL gains nu - N ln nu and d/dnu = 1 - N/nu.
// out: [NLL, grad(P), I = 1, dI = 0]; out_user: [NLL, grad(P)].
__device__ inline void mix1d_finalize_one(const Mix1dConst& mc, const Mix1dTable& t,
                                          const double* part, int64_t nrows, int nv, int kmax,
                                          int with_grad, double n_events, double* out, double* out_user,
                                          double* scratch, double* res) {
  // the validity flag and the yield as vector loads issued before the row
  // sums (a lane-varying zero offset: scalar loads would be waited for with
  // the first kernel argument, before the rows are requested)
  int zero = 0;
  asm volatile("" : "+v"(zero));
  const double valid = (&t.valid)[zero], yield = (&t.yield)[zero];
  sum_rows(part, nrows, nv, scratch, res);
  const int P = mc.n_params;
  const int p = threadIdx.x;
  const bool ok = valid != 0.0;
  const bool ext = mc.yidx >= 0;
  if (p == 0) {
    double v = res[0];
    if (ext) v += yield - n_events * log(yield);
    out[0] = ok ? v : INFINITY;
    out[1 + P] = 1.0;
    if (out_user) out_user[0] = out[0];
  }
  if (p < P) {
    out[2 + P + p] = 0.0;
    if (with_grad) {
      double g = mix1d_param_grad(mc, kmax, res + 1, p);
      if (ext && p == mc.yidx) g += 1.0 - n_events / yield;
      if (!ok) g = NAN;
      out[1 + p] = g;
      if (out_user) out_user[1 + p] = g;
    }
  }
}

// Level 2 of binned data and the statistic, N the yield parameter (extended)
// or the total count W:
//   Poisson  F = sum_b (nu_b - n_b ln nu_b) = N Delta X - W ln(N Delta) - Y
//   chi^2    F = C
// out: [F, grad(P)].
__device__ inline void mix1d_binned_finalize_one(const Mix1dConst& mc, const Mix1dTable& t, const double* part,
                                                 int64_t nrows, int nv, int kmax, int stat, int64_t nb,
                                                 int with_grad, double* out, double* scratch, double* res) {
  sum_rows(part, nrows, nv, scratch, res);
  const int P = mc.n_params;
  const int G = 3 * kmax;
  const int p = threadIdx.x;
  const bool ok = t.valid != 0.0;
  const bool ext = mc.yidx >= 0;
  const double W = res[0];
  const double delta = (mc.hi - mc.lo) / (double)nb;
  const double N = ext ? t.yield : W;
  const double nd = N * delta;
  if (p == 0) {
    const double v = stat == 0 ? nd * res[1] - W * log(nd) - res[2] : res[1];
    out[0] = ok ? v : INFINITY;
  }
  if (with_grad && p < P) {
    double g;
    if (stat == 0) {
      g = nd * mix1d_param_grad(mc, kmax, res + 3, p) - mix1d_param_grad(mc, kmax, res + 3 + G, p);
      if (ext && p == mc.yidx) g += delta * res[1] - W / N;
    } else {
      g = mix1d_param_grad(mc, kmax, res + 3, p);
      if (ext && p == mc.yidx) g += res[2];
    }
    out[1 + p] = ok ? g : NAN;
  }
}

// Total of the rows' first entries into *total (one workgroup).
__device__ inline void mix1d_binned_total_one(const double* part, int64_t nrows, double* total, double* scratch,
                                              double* res) {
  sum_rows(part, nrows, 1, scratch, res);
  if (threadIdx.x == 0) *total = res[0];
}

}  // namespace fn
