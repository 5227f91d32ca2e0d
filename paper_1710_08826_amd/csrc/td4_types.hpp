// Time-dependent four-body model: constants and per-fit tables shared by the
// host, the library's kernels and the kernels compiled at run time.
#pragma once
#include "model.hpp"

namespace fn {

constexpr int kTd4MaxAmp = 20;   // basis amplitudes
constexpr int kTd4MaxRes = 6;    // resonances per pair
constexpr int kWeidN = 40;       // terms of the Faddeeva rational approximation

// w(i y) = exp(y^2) erfc(y) on y >= 0: kErfcK and the coefficients in Z =
// (K - y)/(K + y) of (K + y) w(i y), rising powers (Chebyshev expansion of
// degree 23 computed with 50 digits, rounded once).
constexpr int kErfcN = 24;
constexpr double kErfcK = 3.75;
#define FN_ERFC_COEFFS                                                                             \
  0x1.178842825349dp+0, 0x1.eae02d0a1456bp-1, 0x1.78fecb4e81b0dp-1, 0x1.f63dd81196191p-2, \
  0x1.1dc271189e1d8p-2, 0x1.0e3ea224bc968p-3, 0x1.92618b78faeb3p-5, 0x1.9ac6956772b07p-7, \
  0x1.029006d608353p-10, -0x1.a0b75a1ed9a23p-11, -0x1.6d95256e626cep-12, -0x1.63793f07b8761p-17, \
  0x1.3a550343ac142p-15, 0x1.2ac332d500810p-17, -0x1.b9620425f3497p-19, -0x1.bc81305359091p-20, \
  0x1.2b30aeec1a69fp-22, 0x1.1b2f3e2d5daa8p-22, -0x1.bd29fda663e3ap-26, -0x1.5b8e3892d117dp-25, \
  0x1.7cbe65b7d4a0bp-29, 0x1.77e18f2629084p-28, -0x1.f7c249888c033p-33, -0x1.f79317cac1c2fp-32

// Largest r (td4_device.hpp: time_fns) the time functions' series take with
// ten terms and with twenty.
constexpr double kTimeSeriesTen = 0.125;
constexpr double kTimeSeriesMax = 1.25;

// Constants of the time functions for one decay constant G = 1/tau and one
// resolution width s: products that do not depend on the event.
struct TimeConst {
  double g, s, s2;
  double gs2, hg2s2, g2s2;  // G s^2, G^2 s^2 / 2, G^2 s^2
  double iz, ni2s2;         // 1/(s sqrt 2), -1/(2 s^2)
  double kg, s3;            // G s / sqrt(2 pi), s max(3, G s)
};

struct Td4Const {
  double M;                            // parent mass
  double m1s, m2s, m3s, m4s;           // squared daughter masses
  double sum12, dif12, sum34, dif34;   // (m1 +- m2)^2, (m3 +- m4)^2
  double r2;                           // squared barrier radius
  double m1, m2, m3, m4;               // daughter masses
  double ps_wmax;                      // phase-space weight bound of the generators
  double gamma;                        // 1 / tau
  double wL;                           // Faddeeva approximation scale L
  double wa[kWeidN];                   // its polynomial coefficients a_1..a_N
  double we[kErfcN];                   // real form's coefficients (time_fns takes both at wa)
  int K, n12, n34, n_params;
  int L12[kTd4MaxRes], L34[kTd4MaxRes];
  int nr12[kTd4MaxRes], nr34[kTd4MaxRes];  // 1 = non-resonant (flat) entry
  int amp1[kTd4MaxAmp], amp2[kTd4MaxAmp], atype[kTd4MaxAmp];
  // theta index of Re c_k (in A) and of Re cbar_k (in Abar); -1 when the
  // basis function is not a member of that sum
  int pa[kTd4MaxAmp], pb[kTd4MaxAmp];
};

static_assert(__builtin_offsetof(Td4Const, we) == __builtin_offsetof(Td4Const, wa) + kWeidN * sizeof(double),
              "we follows wa");

// Fixed constants of one fit (systematic variations change them per fit).
struct Td4FitConst {
  double m0_12[kTd4MaxRes], w0_12[kTd4MaxRes], m0_34[kTd4MaxRes], w0_34[kTd4MaxRes];
  double sigma;
};

// Proposal density of one pair mass in the toy generator: with probability
// wu uniform on [lo, hi]; otherwise resonance r (probability (1 - wu)/n each)
// through a Student-t density of two degrees of freedom, g(x) = (1 + x^2)^(-3/2)
// / 2, x = (m - m_r)/s_r, truncated to [lo, hi].  Its distribution function is
// (1 + v)/2 with v = x / sqrt(1 + x^2), so a truncated draw is v uniform in
// [vlo_r, vhi_r] and x = v / sqrt(1 - v^2): additions, products, quotients and
// square roots only, which the host reference reproduces bit for bit.  Its
// tails fall as |x|^-3, past the |x|^-2 of a Breit-Wigner intensity, so the
// uniform part carries the proposal away from the peaks.
struct Td4PairProposal {
  int n;                               // resonant entries (0: uniform only)
  double lo, hi, wu;
  double m[kTd4MaxRes], s[kTd4MaxRes], vlo[kTd4MaxRes], vhi[kTd4MaxRes];
};
struct Td4Proposal {
  Td4PairProposal p12, p34;
};

// Draw from the pair proposal with the component selector usel and the
// position upos (both uniform in [0, 1)).
__host__ __device__ inline double td4_prop_draw(const Td4PairProposal& p, double usel, double upos) {
#pragma clang fp contract(off)
  if (p.n == 0 || usel < p.wu) return p.lo + upos * (p.hi - p.lo);
  int r = (int)((usel - p.wu) / (1.0 - p.wu) * p.n);
  r = r < p.n ? r : p.n - 1;
  const double v = p.vlo[r] + upos * (p.vhi[r] - p.vlo[r]);
  return p.m[r] + p.s[r] * (v / sqrt(1.0 - v * v));
}

// The pair proposal's density at m (on [lo, hi]).
__host__ __device__ inline double td4_prop_density(const Td4PairProposal& p, double m) {
#pragma clang fp contract(off)
  double q = (p.n == 0 ? 1.0 : p.wu) / (p.hi - p.lo);
  const double wr = p.n == 0 ? 0.0 : (1.0 - p.wu) / p.n;
  for (int r = 0; r < p.n; ++r) {
    const double x = (m - p.m[r]) / p.s[r];
    const double t = 1.0 + x * x;
    q = q + wr / ((p.s[r] * (p.vhi[r] - p.vlo[r])) * (t * sqrt(t)));
  }
  return q;
}

// Per-fit table (prologue output).
struct Td4Table {
  double r12[kTd4MaxRes][3];  // m0^2, Kw, Ka  (resonant entries)
  double r34[kTd4MaxRes][3];
  double c[kTd4MaxAmp][2], cb[kTd4MaxAmp][2];
  double x, y, sigma;
  TimeConst tk;                 // time functions' constants (sigma's)
  double valid;
};

}  // namespace fn
