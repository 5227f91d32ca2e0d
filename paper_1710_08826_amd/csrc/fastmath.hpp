// FP64 reciprocal, square root and logarithm for the per-event loops.
//
// rcp/rsqrt start from the hardware approximations (v_rcp_f64, v_rsq_f64,
// relative error below 2^-24 on gfx950: at most 2.5e8 units in the last place
// over 2^20 arguments, half log-uniform in [2^-60, 2^60], half mantissas in
// [1, 2) at exponents -20..20) and apply one Newton-Raphson step on the
// residual e, computed with an FMA: 1/x = r / (1 - e) with e = 1 - x r, taken
// as r (1 + e); 1/sqrt(x) = y (1 - e)^(-1/2) with e = 1 - x y^2, taken as
// y (1 + e/2).  The truncation error is of order e^2 < 2^-48: measured at most
// 10.6 units in the last place for rcp and 19.3 for rsqrt on that sample
// (2.4e-15 and 4.3e-15 relative).  The amplitudes that use them enter sums
// whose tolerance is 1e-12 relative, and one term less each (19 per event of
// the eight-resonance Dalitz pass) measured 3% off its step.  rcp_acc adds the
// second-order term, r (1 + e + e^2), for a result within half a unit in the
// last place on the same sample (for the logarithm's argument reduction).
// They take finite, positive, normal arguments; callers clamp where a zero
// can occur.
//
// log_fast: argument reduction x = 2^e m with m in [sqrt(1/2), sqrt(2))
// (Cody & Waite, Software Manual for the Elementary Functions, 1980), then
// ln m = 2 atanh(f) = 2 (f + f^3/3 + f^5/5 + ...), f = (m-1)/(m+1), |f| <=
// 0.1716 (Abramowitz & Stegun 4.1.27); eleven terms bring the truncation
// below 3e-17 relative.  ln 2 is split into a 32-bit head and a tail so that
// e ln 2 is formed without rounding error in the head.
#pragma once
#if !defined(__HIPCC_RTC__)
#include <hip/hip_runtime.h>
#endif

namespace fn {

__device__ __forceinline__ double rcp_fast(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}

__device__ __forceinline__ double rcp_acc(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, __builtin_fma(e, e, e), r);
}

__device__ __forceinline__ double rsqrt_fast(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(y * 0.5, e, y);
}

// In place, D[j] <- 1 / D[j] for the first n (1..4) entries, from one
// reciprocal of their product (simultaneous inversion: with p_j = D_0 ... D_j
// and r = 1 / p_{n-1}, 1/D_j = r p_{j-1} D_{j+1} ... D_{n-1}, peeled from the
// top down): 3 (n - 1) multiplies in place of n - 1 reciprocals and their
// Newton steps (a stream of v_rcp_f64 alone issues at about a third of the
// FMA rate on gfx950).  The products form a serial chain, which pays where
// the waves hide its latency: the three-body Dalitz passes (eight
// resonances, 1M events: step 18.5 -> 17.9 us); the four-body pass, at two
// waves per SIMD, measured 5% slower and the time-dependent three-body pass
// even, and they keep one reciprocal per denominator.  A product of four denominators stays a normal
// number for denominators in [2^-250, 2^250]; the result carries a few more
// roundings (about 2 n) than a reciprocal each.  n is a compile-time constant
// where this is inlined into unrolled code.
__device__ __forceinline__ void rcp_group(double (&D)[4], int n) {
  double p[4];
  p[0] = D[0];
#pragma unroll
  for (int j = 1; j < 4; ++j) p[j] = j < n ? p[j - 1] * D[j] : p[j - 1];
  double pn = p[0];
#pragma unroll
  for (int j = 1; j < 4; ++j) pn = j < n ? p[j] : pn;
  double r = rcp_fast(pn);
#pragma unroll
  for (int j = 3; j > 0; --j) {
    if (j < n) {
      const double dj = r * p[j - 1];
      r = r * D[j];
      D[j] = dj;
    }
  }
  D[0] = r;
}

// a b + c with c the same in all lanes (a coefficient), c read from scalar
// registers by the instruction itself.  From the plain expression the compiler
// forms the two-operand v_fmac, whose addend has to be copied into vector
// registers first, and a 32-bit move takes as long as an FP64 FMA here: a
// polynomial step then cost three instructions (two in v_mov_b64 form).
__device__ __forceinline__ double fma_sc(double a, double b, double c) {
#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC_RTC__)
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
#else
  return __builtin_fma(a, b, c);
#endif
}

// e^x: x = n ln 2 + r with |r| <= ln 2 / 2 (Cody & Waite), e^r = 1 + r + r^2
// q(r), q the degree-9 interpolant of (e^r - 1 - r)/r^2 at the Chebyshev nodes
// of that interval (relative error of e^r 1.6e-17), 2^n by ldexp.  Twenty
// instructions against 34 of the library's, whose addends are moved (fma_sc).
// Zero below -750 (to -infinity); above 709.8 infinity by ldexp, NaN at
// +infinity and beyond 1e44; NaN for NaN.
__device__ __forceinline__ double exp_fast(double x) {
  constexpr double kLog2e = 1.44269504088896340736;
  constexpr double kLn2Hi = 0x1.62e42fefa39efp-1, kLn2Lo = 0x1.abc9e3b39803fp-56;
  const double n = __builtin_rint(x * kLog2e);
  const double r = __builtin_fma(-n, kLn2Lo, __builtin_fma(-n, kLn2Hi, x));
  double p = 0x1.af389eea54156p-26;
  p = fma_sc(p, r, 0x1.28917c9f3a495p-22);
  p = fma_sc(p, r, 0x1.71de0db2eb873p-19);
  p = fma_sc(p, r, 0x1.a019b914881bap-16);
  p = fma_sc(p, r, 0x1.a01a01a7c2f2cp-13);
  p = fma_sc(p, r, 0x1.6c16c17889f3cp-10);
  p = fma_sc(p, r, 0x1.11111111109b5p-7);
  p = fma_sc(p, r, 0x1.5555555553d68p-5);
  p = fma_sc(p, r, 0x1.5555555555556p-3);
  p = fma_sc(p, r, 0x1.0000000000001p-1);
  p = __builtin_fma(__builtin_fma(p, r, 1.0), r, 1.0);
  const double e = __builtin_amdgcn_ldexp(p, (int)n);
  return x < -750.0 ? 0.0 : e;
}

// The library's sine and cosine as a call: inlined, its coefficients would sit
// in some forty vector registers of the caller's event loop.
__device__ __attribute__((noinline)) inline void sincos_any(double x, double* sn, double* cs) { sincos(x, sn, cs); }

// sin x and cos x: x = k pi/2 + r with |r| <= pi/4 (Cody & Waite, pi/2 in two
// parts), the two functions of r by polynomials in r^2 at the Chebyshev nodes
// of [0, pi^2/16] (errors 2.0e-17 relative and 9e-19), exchanged and signed by
// k's quadrant.  Absolute error below 2e-16 for |x| < 1e5; a wave with a
// larger (or not finite) argument takes the library's function (ALONE: only the
// lanes that have one).
template <bool ALONE = false>
__device__ __forceinline__ void sincos_fast(double x, double& sn, double& cs) {
  const bool far = !(fabs(x) < 1e5);
  if (__builtin_expect(ALONE ? far : __any(far), 0)) {
    double a, b;
    sincos_any(x, &a, &b);
    sn = a;
    cs = b;
    return;
  }
  const double k = __builtin_rint(x * 0.63661977236758134308);
  const double r = __builtin_fma(-k, 0x1.1a62633145c07p-54, __builtin_fma(-k, 0x1.921fb54442d18p+0, x));
  const double z = r * r;
  double s = 0x1.5e0b13ccdcb64p-33;
  s = fma_sc(s, z, -0x1.ae600af19478ap-26);
  s = fma_sc(s, z, 0x1.71de3796799f6p-19);
  s = fma_sc(s, z, -0x1.a01a019e839e3p-13);
  s = fma_sc(s, z, 0x1.1111111110bb2p-7);
  s = fma_sc(s, z, -0x1.5555555555555p-3);
  s = __builtin_fma(r * z, s, r);
  double c = -0x1.907d9d3a50522p-37;
  c = fma_sc(c, z, 0x1.1eeb68e0a87edp-29);
  c = fma_sc(c, z, -0x1.27e4fa17d1cf9p-22);
  c = fma_sc(c, z, 0x1.a01a019f4ea9bp-16);
  c = fma_sc(c, z, -0x1.6c16c16c16967p-10);
  c = fma_sc(c, z, 0x1.5555555555555p-5);
  c = __builtin_fma(z * z, c, __builtin_fma(z, -0.5, 1.0));
  const int q = (int)k;
  const bool odd = q & 1;
  const double a = odd ? c : s, b = odd ? s : c;
  // sin takes the sign of bit 1 of k, cos that of bit 1 of k + 1
  sn = __longlong_as_double(__double_as_longlong(a) ^ ((long long)(q & 2) << 62));
  cs = __longlong_as_double(__double_as_longlong(b) ^ ((long long)((q + 1) & 2) << 62));
}

// sqrt for x >= 0; arguments below 1e-300 are treated as 1e-300.
__device__ __forceinline__ double sqrt_fast(double x) {
  const double xc = __builtin_fmax(x, 1e-300);
  return xc * rsqrt_fast(xc);
}

__device__ __forceinline__ double log_fast(double x) {
  double m = __builtin_amdgcn_frexp_mant(x);  // [0.5, 1)
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool lo = m < 0.70710678118654752440;
  m = lo ? 2.0 * m : m;
  e = lo ? e - 1 : e;
  const double f = (m - 1.0) * rcp_acc(m + 1.0);
  const double f2 = f * f;
  double p = 1.0 / 23.0;
  p = __builtin_fma(p, f2, 1.0 / 21.0);
  p = __builtin_fma(p, f2, 1.0 / 19.0);
  p = __builtin_fma(p, f2, 1.0 / 17.0);
  p = __builtin_fma(p, f2, 1.0 / 15.0);
  p = __builtin_fma(p, f2, 1.0 / 13.0);
  p = __builtin_fma(p, f2, 1.0 / 11.0);
  p = __builtin_fma(p, f2, 1.0 / 9.0);
  p = __builtin_fma(p, f2, 1.0 / 7.0);
  p = __builtin_fma(p, f2, 1.0 / 5.0);
  p = __builtin_fma(p, f2, 1.0 / 3.0);
  const double f2x = 2.0 * f;
  const double lm = __builtin_fma(f2x * f2, p, f2x);
  const double de = (double)e;
  // ln 2 rounded to 32 significant bits, and the remainder
  constexpr double kLn2Hi = 0x1.62e42ff000000p-1;
  constexpr double kLn2Lo = -0x1.718432a1b0e26p-35;
  const double r = __builtin_fma(de, kLn2Hi, __builtin_fma(de, kLn2Lo, lm));
  // IEEE results outside (0, inf): -inf at 0, +inf at inf, NaN below 0 or NaN
  const bool finite_pos = x > 0.0 && x <= 1.7976931348623157e308;
  return finite_pos ? r : (x == 0.0 ? -__builtin_inf() : (x > 0.0 ? x : __builtin_nan("")));
}

// Sum of logarithms through a running product: sum_i ln x_i = ln m + e ln 2,
// the product of the factors kept as m in [0.5, 1) times 2^e (split again
// after every factor, so that it neither overflows nor underflows), and one
// logarithm at the end serves all the factors: one multiply and two
// mantissa/exponent splits per factor instead of a logarithm each.  Each
// multiply rounds once, so after n factors the product's relative error is
// below n 2^-53 and the sum's absolute error below n 2^-53 plus the final
// logarithm's.  A zero factor gives -inf, a negative or NaN factor NaN and an
// infinite one +inf, as the sum of the factors' logarithms would.
struct LogProd {
  double m = 1.0;
  int e = 0;
  __device__ __forceinline__ void mul(double x) {
    const double p = m * x;
    e += __builtin_amdgcn_frexp_exp(p);
    m = __builtin_amdgcn_frexp_mant(p);
  }
  __device__ __forceinline__ double log() const {
    // ln 2 rounded to 32 significant bits, and the remainder (e ln 2 formed
    // without rounding error in the head for |e| < 2^21)
    constexpr double kLn2Hi = 0x1.62e42ff000000p-1;
    constexpr double kLn2Lo = -0x1.718432a1b0e26p-35;
    const double de = (double)e;
    return __builtin_fma(de, kLn2Hi, __builtin_fma(de, kLn2Lo, log_fast(m)));
  }
};

}  // namespace fn
