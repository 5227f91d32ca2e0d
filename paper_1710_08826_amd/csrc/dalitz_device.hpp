// Device code of the three-body Dalitz-plot model, compiled at run time for
// each model structure (the resonances' pairs and spins become compile-time
// constants; see jit.hpp) and, for the structure-generic helpers, into the
// library.
//
//   P~(s12, s13) = |sum_k c_k A_k|^2,
//   A_k = [F_L(q r)/F_L(q0 r)] F_L(p r_D) Z_L(s) T_k(s_AB)
//   T_k = 1 / (m0^2 - s_AB - i m0 Gamma_k(s_AB))
//   Gamma_k(s) = Gamma0 (q/q0)^(2L+1) (m0/sqrt s) [F_L(q r)/F_L(q0 r)]^2
//
// with Blatt-Weisskopf factors F_0 = 1, F_1 = (1+z)^-1/2,
// F_2 = (z^2+3z+9)^-1/2 (z = (q r)^2) and Zemach spin factors Z_0 = 1,
// Z_1 = s_AC - s_BC + (M^2 - mC^2)(mB^2 - mA^2)/s_AB, Z_2 = Z_1^2 - X Y / 3,
// X = lambda(s_AB, M^2, mC^2)/s_AB, Y = lambda(s_AB, mA^2, mB^2)/s_AB.
//
// Per event, all in registers:
//  * every quantity that depends only on the pair (s_AB, q, p, the barrier
//    polynomials, Zemach factors) is computed once per pair and shared by all
//    resonances of that pair;
//  * per resonance the lineshape reduces to T = (a + i b)/(a^2 + b^2) with
//    a = m0^2 - s and b = m0 Gamma(s) = Kw * G_{pair,L}(s), where
//    G = q^(2L+1) F_L(q r)^2 / sqrt(s) is per pair and
//    Kw = Gamma0 m0^2 / (q0^(2L+1) F_L(q0 r)^2) comes from the prologue;
//  * the amplitude is A = Ka * H_{pair,L} * T with H = F_L(q r) F_L(p r_D) Z_L
//    per pair and Ka = 1/F_L(q0 r) per resonance.
//
// Modes of the chunk routine:
//   kEvents  -ln P~ over an event chunk (+ adjoint gradient)          -> NLL
//   kGrid    P~ over a chunk of grid cells inside the region (+ dP~)  -> I
// and a matrix pass: sum over the cells inside the region of A_i conj(A_j)
// (gram_device.hpp), the cached M of fixed lineshapes.
#pragma once
#include "accept_device.hpp"
#include "device_common.hpp"
#include "fastmath.hpp"
#include "gram_device.hpp"
#include "model.hpp"
#include "philox.hpp"

namespace fn {

enum DalMode : int { kEvents = 0, kGrid = 1 };

__host__ __device__ constexpr int dal_nv(int mode, int grad, int k) {
  return 1 + (grad == 0 ? 0 : (grad == 1 ? 2 * k : 4 * k));
}

struct PairTerms {
  double s;         // s_AB
  double G[3];      // q^(2L+1) F_L(q r)^2 / sqrt(s)
  double H[3];      // F_L(q r) F_L(p r_D) Z_L
};

// G and H of one pair from (s_AB, s_AC, s_BC), for the spins U1 (L = 1) and
// U2 (L = 2) the pair needs (L = 0 is always formed):
//   q/sqrt(s) = sqrt(lambda_q) / (2 s),  q^2 = lambda_q / (4 s),  p^2 = lambda_p / (4 s)
//   G_1 = (q/sqrt s) q^2 / (1 + z_q),          H_1 = Z_1 / sqrt((1 + z_q)(1 + z_p))
//   G_2 = (q/sqrt s) q^4 / (z_q^2 + 3 z_q + 9), H_2 = Z_2 / sqrt(poly(z_q) poly(z_p))
template <bool U1, bool U2>
__device__ __forceinline__ void pair_terms_is(const DalitzChan& ch, double s_ab, double is, double s_ac, double s_bc,
                                              double r2, double rD2, PairTerms& o) {
  const double lq = fmax((s_ab - ch.sum2) * (s_ab - ch.dif2), 0.0);
  const double q2 = 0.25 * lq * is;
  const double qirs = 0.5 * sqrt_fast(lq) * is;
  o.s = s_ab;
  o.G[0] = qirs;
  o.H[0] = 1.0;
  o.G[1] = o.G[2] = o.H[1] = o.H[2] = 0.0;
  if (U1 || U2) {
    const double lp = fmax((s_ab - ch.Psum2) * (s_ab - ch.Pdif2), 0.0);
    const double p2 = 0.25 * lp * is;
    const double zq = q2 * r2, zp = p2 * rD2;
    const double z1 = __builtin_fma(ch.zc, is, s_ac - s_bc);
    // 1/u_q = (1/sqrt(u_q u_p))^2 u_p: one reciprocal square root serves both
    if (U1) {
      const double uq = 1.0 + zq, up = 1.0 + zp;
      const double r = rsqrt_fast(uq * up);
      o.G[1] = qirs * q2 * (r * r * up);
      o.H[1] = z1 * r;
    }
    if (U2) {
      const double vq = __builtin_fma(zq, zq + 3.0, 9.0), vp = __builtin_fma(zp, zp + 3.0, 9.0);
      const double r = rsqrt_fast(vq * vp);
      o.G[2] = qirs * q2 * q2 * (r * r * vp);
      const double z2 = z1 * z1 - (lp * is) * (lq * is) * (1.0 / 3.0);
      o.H[2] = z2 * r;
    }
  }
}

// The same, forming 1/s_AB itself.
template <bool U1, bool U2>
__device__ __forceinline__ void pair_terms_t(const DalitzChan& ch, double s_ab, double s_ac, double s_bc, double r2,
                                             double rD2, PairTerms& o) {
  pair_terms_is<U1, U2>(ch, s_ab, rcp_fast(s_ab), s_ac, s_bc, r2, rD2, o);
}

// Centre of cell i along a grid axis that starts at a with cells of size d,
// as the plain IEEE evaluation (no contraction), so that every pass and the
// cell list see the same bits.
__device__ inline double grid_centre(double a, int64_t i, double d) {
#pragma clang fp contract(off)
  return a + (i + 0.5) * d;
}

// Physical-region bounds of the grid row at s12: s23 between lo and hi, from
// the energies of daughters 2 and 3 in the (12) rest frame.  Contraction is
// off so that the decision is the plain IEEE evaluation.
__device__ inline void dalitz_row_bounds(const DalitzConst& dc, double s12, double& lo, double& hi) {
#pragma clang fp contract(off)
  const double rs = sqrt(s12);
  const double e2 = (s12 - dc.m1s + dc.m2s) / (2.0 * rs);
  const double e3 = (dc.M2 - s12 - dc.m3s) / (2.0 * rs);
  const double p2 = sqrt(fmax(e2 * e2 - dc.m2s, 0.0));
  const double p3 = sqrt(fmax(e3 * e3 - dc.m3s, 0.0));
  const double es = e2 + e3;
  lo = es * es - (p2 + p3) * (p2 + p3);
  hi = es * es - (p2 - p3) * (p2 - p3);
}

// Physical-region predicate at a grid-cell centre, given its row's bounds.
__device__ inline bool dalitz_in_row(const DalitzConst& dc, double s12, double s13, double lo, double hi) {
#pragma clang fp contract(off)
  const double s23 = dc.msum - s12 - s13;
  return s23 >= lo && s23 <= hi;
}

__device__ inline bool dalitz_inside(const DalitzConst& dc, double s12, double s13) {
  double lo, hi;
  dalitz_row_bounds(dc, s12, lo, hi);
  return dalitz_in_row(dc, s12, s13, lo, hi);
}

// The same decision, most often without its square roots and divisions: with
// A = 2 sqrt(s12) e2, B = 2 sqrt(s12) e3 and the squared momenta's a = A^2 - 4
// s12 m2^2, b likewise, s23 lies between lo and hi where
//   F = (4 s12 (s23 - m2^2 - m3^2) - 2 A B)^2 - 4 a b <= 0,
// the physical region's boundary polynomial.  The rounding errors of F, and
// those of lo and hi carried over to it, stay below 100 2^-53 T^2 with T = 4
// s12 (|s23| + m2^2 + m3^2) + (|A| + |B|)^2; a point within 4500 2^-52 T^2 of
// the boundary (one in 1e10), or NaN, is left to the predicate itself.  22
// operations instead of 100 per draw of the event generators (263 with the
// draw's own): half a million toys 234 -> 209 us.
__device__ __forceinline__ bool dalitz_inside_quick(const DalitzConst& dc, double s12, double s13) {
  const double s23 = dc.msum - s12 - s13;
  const double A = s12 - dc.m1s + dc.m2s, B = dc.M2 - s12 - dc.m3s, f = 4.0 * s12;
  const double a = __builtin_fma(A, A, -f * dc.m2s), b = __builtin_fma(B, B, -f * dc.m3s);
  const double D = __builtin_fma(f, s23 - dc.m2s - dc.m3s, -2.0 * A * B);
  const double F = __builtin_fma(D, D, -4.0 * a * b);
  const double ab = fabs(A) + fabs(B);
  const double T = __builtin_fma(f, fabs(s23) + dc.m2s + dc.m3s, ab * ab);
  bool in = F < 0.0;
  if (__builtin_expect(!(a > 0.0 && b > 0.0 && fabs(F) > 1e-12 * T * T), 0)) in = dalitz_inside(dc, s12, s13);
  return in;
}

// Compile-time structure queries on a shape S (S::K, S::chan[], S::L[]).
template <class S>
__host__ __device__ constexpr bool shape_uses(int c, int l) {
  bool u = false;
  for (int k = 0; k < S::K; ++k) u = u || (S::chan[k] == c && S::L[k] == l);
  return u;
}

// One resonance's amplitude from its pair's terms: A_k = Ka H T with
// T = 1 / (a - i b) = (a + i b) d, a = m0^2 - s, b = Kw G, d = 1 / (a^2 + b^2)
// (rk: the resonance's row of the table), in two steps so that the
// reciprocals of several resonances can be formed together (rcp_group).
__device__ __forceinline__ void bw_denominator(const double* __restrict__ rk, double s, double G, double& a,
                                               double& b, double& D) {
  a = rk[dM0SQ] - s;
  b = rk[dKW] * G;
  D = __builtin_fma(a, a, b * b);
}

__device__ __forceinline__ void bw_amplitude(const double* __restrict__ rk, double H, double a, double b, double d,
                                             double& ar, double& ai) {
  const double u = (rk[dKA] * H) * d;
  ar = u * a;
  ai = u * b;
}

template <class S, int C>
__host__ __device__ constexpr bool pair_used() {
  return shape_uses<S>(C, 0) || shape_uses<S>(C, 1) || shape_uses<S>(C, 2);
}

// Pair terms of pair C (compile-time) at a point, when the shape uses it
// (is: 1/s_AB).
template <class S, int C>
__device__ __forceinline__ void dalitz_pair_terms(const DalitzConst& dc, double s12, double s13, double s23,
                                                  double is, PairTerms& pt) {
  if (!pair_used<S, C>()) return;
  // pair "12": (A,B,C) = (1,2,3); "13": (1,3,2); "23": (2,3,1)
  const double s_ab = C == 0 ? s12 : (C == 1 ? s13 : s23);
  const double s_ac = C == 0 ? s13 : s12;
  const double s_bc = C == 2 ? s13 : s23;
  pair_terms_is<shape_uses<S>(C, 1), shape_uses<S>(C, 2)>(dc.ch[C], s_ab, is, s_ac, s_bc, dc.r2, dc.rD2, pt);
}

// Amplitudes of all resonances (in model order, four at a time for the
// reciprocals), added to the coherent sum S = sum_k c_k A_k (SUM).  ACC: every
// reciprocal by itself, to half a unit in the last place instead of eleven and
// more (the density per event, whose values are handed out: with the grouped
// ones two events' densities differed by up to 45 units of 2^-53 where all else
// leaves 28 at most; a call on 1M events of the eight-resonance model takes 35.2
// us instead of 34.3).
template <class S, bool KEEP_A, bool KEEP_T, bool SUM = true, bool ACC = false>
__device__ __forceinline__ void dalitz_amps(const DalitzConst& dc, const double* __restrict__ r,
                                            cdouble* __restrict__ coef, double s12, double s13, double s23,
                                            double (&Are)[S::K], double (&Aim)[S::K], double (&Tre)[S::K],
                                            double (&Tim)[S::K], double (&Gk)[S::K], double& Sre, double& Sim) {
  constexpr int K = S::K;
  // 1/s of the pairs in use from one reciprocal (an unused pair's 1 drops out)
  double is[4] = {pair_used<S, 0>() ? s12 : 1.0, pair_used<S, 1>() ? s13 : 1.0, pair_used<S, 2>() ? s23 : 1.0, 1.0};
  if (ACC) {
#pragma unroll
    for (int j = 0; j < 3; ++j) is[j] = rcp_acc(is[j]);
  } else {
    rcp_group(is, 3);
  }
  PairTerms pt0, pt1, pt2;
  dalitz_pair_terms<S, 0>(dc, s12, s13, s23, is[0], pt0);
  dalitz_pair_terms<S, 1>(dc, s12, s13, s23, is[1], pt1);
  dalitz_pair_terms<S, 2>(dc, s12, s13, s23, is[2], pt2);
#pragma unroll
  for (int g = 0; g < K; g += 4) {
    const int n = K - g < 4 ? K - g : 4;
    double a[4], b[4], D[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j < n) {
        const int k = g + j;
        const PairTerms& pt = S::chan[k] == 0 ? pt0 : (S::chan[k] == 1 ? pt1 : pt2);
        bw_denominator(r + k * kDalFields, pt.s, pt.G[S::L[k]], a[j], b[j], D[j]);
      }
    }
    if (ACC) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < n) D[j] = rcp_acc(D[j]);
    } else {
      rcp_group(D, n);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j < n) {
        const int k = g + j;
        const int L = S::L[k];
        const PairTerms& pt = S::chan[k] == 0 ? pt0 : (S::chan[k] == 1 ? pt1 : pt2);
        const double* rk = r + k * kDalFields;
        double ar, ai;
        if (KEEP_T) {
          Tre[k] = a[j] * D[j]; Tim[k] = b[j] * D[j]; Gk[k] = pt.G[L];
          const double u = rk[dKA] * pt.H[L];
          ar = u * Tre[k];
          ai = u * Tim[k];
        } else {
          bw_amplitude(rk, pt.H[L], a[j], b[j], D[j], ar, ai);
        }
        if (KEEP_A) { Are[k] = ar; Aim[k] = ai; }
        if (SUM) {
          // S += c_k A_k as four chained FMAs
          const double cr = coef[2 * k], ci = coef[2 * k + 1];
          Sre = __builtin_fma(cr, ar, __builtin_fma(-ci, ai, Sre));
          Sim = __builtin_fma(cr, ai, __builtin_fma(ci, ar, Sim));
        }
      }
    }
  }
}

// One event or grid cell: its terms added to acc when `valid` (otherwise it
// contributes exact zeros, so the sum is unchanged).
template <class S, int MODE, int GRAD>
__device__ __forceinline__ void dalitz_point(const DalitzConst& dc, const double* __restrict__ r,
                                             cdouble* __restrict__ coef, double s12, double s13, bool valid,
                                             double (&acc)[dal_nv(MODE, GRAD, S::K)], LogProd& lp) {
  constexpr int K = S::K;
  constexpr bool KEEP_A = GRAD >= 1;
  constexpr bool KEEP_T = GRAD == 2;
  const double s23 = dc.msum - s12 - s13;
  double Are[K], Aim[K], Tre[K], Tim[K], Gk[K];
  double Sre = 0.0, Sim = 0.0;
  dalitz_amps<S, KEEP_A, KEEP_T>(dc, r, coef, s12, s13, s23, Are, Aim, Tre, Tim, Gk, Sre, Sim);
  auto add = [&](int idx, double v) { acc[idx] += valid ? v : 0.0; };
  // acc[idx] += x1 y1 + x2 y2 as two chained FMAs
  auto add2 = [&](int idx, double x1, double y1, double x2, double y2) {
    const double t = __builtin_fma(x2, y2, __builtin_fma(x1, y1, acc[idx]));
    acc[idx] = valid ? t : acc[idx];
  };
  const double Pt = __builtin_fma(Sre, Sre, Sim * Sim);
  double w;  // multiplies dP~/dtheta
  if (MODE == kEvents) {
    lp.mul(valid ? Pt : 1.0);  // -ln P~ enters acc[0] once per thread, at the end
    if (GRAD >= 1) w = -rcp_fast(Pt);
  } else {
    add(0, Pt);
    w = 1.0;
  }
  if (GRAD == 1) {
    const double w2 = 2.0 * w;
    const double ur = w2 * Sre, ui = w2 * Sim;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      // dP~/dRe c = 2 Re(conj(S) A), dP~/dIm c = 2 (Sim Are - Sre Aim)
      add2(1 + 2 * k, ur, Are[k], ui, Aim[k]);
      add2(2 + 2 * k, ui, Are[k], -ur, Aim[k]);
    }
  }
  if (GRAD == 2) {
    // with g = 2 w conj(S) A and E = c g: Re g and -Im g (the coefficients'
    // slots), Re(E T) and G Im(E T) (dalitz_lineshape_slots makes the rest)
    const double w2 = 2.0 * w;
    const double ur = w2 * Sre, ui = w2 * Sim;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double cr = coef[2 * k], ci = coef[2 * k + 1];
      const double gr = __builtin_fma(ui, Aim[k], ur * Are[k]), gi = __builtin_fma(ur, Aim[k], -(ui * Are[k]));
      const double er = __builtin_fma(-ci, gi, cr * gr), ei = __builtin_fma(ci, gr, cr * gi);
      add(1 + 2 * k, gr);
      add(2 + 2 * k, -gi);
      add2(1 + 2 * K + 2 * k, er, Tre[k], -ei, Tim[k]);
      const double q = __builtin_fma(er, Tim[k], ei * Tre[k]);
      const double t = __builtin_fma(Gk[k], q, acc[2 + 2 * K + 2 * k]);
      acc[2 + 2 * K + 2 * k] = valid ? t : acc[2 + 2 * K + 2 * k];
    }
  }
}

// Mass and width slots of a thread's sums.  dA/dm0 = A (dlnKa - T (2 m0 - i G
// dKw/dm0)) and dA/dGamma0 = i A T G Kw/Gamma0, so with E = 2 w conj(S) c A
//   sum dP~/dm0     = dlnKa sum Re E - 2 m0 sum Re(E T) - dKw/dm0 sum G Im(E T)
//   sum dP~/dGamma0 = -Kw/Gamma0 sum G Im(E T),
// and Re E follows from the coefficients' slots: fifteen operations per
// resonance and event instead of twenty-three.
template <class S, int NV>
__device__ __forceinline__ void dalitz_lineshape_slots(const double* __restrict__ r, cdouble* __restrict__ coef,
                                                       double (&acc)[NV]) {
  constexpr int K = S::K;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double* rk = r + k * kDalFields;
    const double e = __builtin_fma(coef[2 * k], acc[1 + 2 * k], coef[2 * k + 1] * acc[2 + 2 * k]);
    double& m = acc[1 + 2 * K + 2 * k];
    double& v = acc[2 + 2 * K + 2 * k];
    m = __builtin_fma(rk[dDLNKA], e, -__builtin_fma(rk[dTWOM0], m, rk[dDKW_DM0] * v));
    v = -rk[dKW_W0] * v;
  }
}

// One fixed chunk of events or grid cells -> one row of partial sums.
// GRAD: 0 none, 1 coefficients only, 2 coefficients + masses and widths.
// EPT events per thread and loop iteration (independent work for the
// scheduler to interleave); each thread still adds its points in index order.
// Two per iteration measured slower than one for the eight-resonance model on
// MI355X (more VGPRs); the events passes come in both forms and the
// autotuner times them, the grid passes use one.
template <class S, int MODE, int GRAD, int EPT = 1>
__device__ inline void dalitz_chunk(const DalitzConst& dc, const DalitzTable* __restrict__ tab,
                                    cdouble* __restrict__ coef0, const double* __restrict__ ev, int64_t ld,
                                    int64_t n, int64_t chunk_idx, int chunk, double* __restrict__ out_row,
                                    double* lds) {
  constexpr int NV = dal_nv(MODE, GRAD, S::K);
  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  const int64_t base = chunk_idx * chunk;
  const int64_t end = base + chunk < n ? base + chunk : n;
  const double* const r0 = &tab->r[0][0];
  LogProd lp;
  // The next iteration's points are loaded while one is worked on (their index
  // held to the chunk, so that the last round reads nothing else): with two
  // waves per SIMD the loads' latency was as long as the work on a point.
  double n12[EPT], n13[EPT];
  GridCell nc[EPT];
  auto load = [&](int64_t i) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int64_t j = i + e * kBlock, jj = j < end ? j : end - 1;
      if (MODE == kEvents) {
        n12[e] = ev[jj];
        n13[e] = ev[ld + jj];
      } else {
        // grid passes walk the list of the cells inside the region (ev)
        nc[e] = reinterpret_cast<const GridCell*>(ev)[jj];
      }
    }
  };
  if (base < end) load(base + threadIdx.x);
  for (int64_t i = base + threadIdx.x; i < end; i += EPT * kBlock) {
    // The per-resonance constants are read through the scalar cache on every
    // event: an empty asm makes a zero offset opaque to the loop so that the
    // compiler does not keep the whole table resident in SGPRs, which
    // overflows them into VGPR lanes (a v_readlane per use); the pointer keeps
    // its provenance, so the reads stay scalar loads.
    int zero = 0;
    asm volatile("" : "+s"(zero));
    const double* r = r0 + zero;
    cdouble* coef = coef0 + zero;
    double s12[EPT], s13[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      s12[e] = MODE == kEvents ? n12[e] : grid_centre(dc.a12, nc[e].ix, dc.d12);
      s13[e] = MODE == kEvents ? n13[e] : grid_centre(dc.a13, nc[e].iy, dc.d13);
    }
    load(i + EPT * kBlock);
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      dalitz_point<S, MODE, GRAD>(dc, r, coef, s12[e], s13[e], e == 0 || i + e * kBlock < end, acc, lp);
  }
  if (MODE == kEvents) acc[0] = -lp.log();
  if constexpr (GRAD == 2) dalitz_lineshape_slots<S>(r0, coef0, acc);
  block_sum_row<NV>(acc, lds, out_row);
}

// Normalization of a model with fixed lineshapes from the cached grid matrix
// M (K x K complex, M_kj = dA sum over cells of A_k conj(A_j)): I = c^H M c =
// sum_k Re(c_k X_k) with X_k = sum_j M_kj conj(c_j), dI/dRe c_k = 2 Re X_k,
// dI/dIm c_k = -2 Im X_k.  Writes out[0] = I and out[1 + 2k], out[2 + 2k];
// all threads of the workgroup call it.
template <class S>
__device__ inline void dalitz_cached_norm(const double* __restrict__ M, cdouble* __restrict__ coef,
                                          double* __restrict__ out) {
  constexpr int K = S::K;
  __shared__ double ip[K];
  const int t = threadIdx.x;
  if (t < K) {
    double xr = 0.0, xi = 0.0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const double mr = M[2 * (t * K + j)], mi = M[2 * (t * K + j) + 1];
      const double cr = coef[2 * j], ci = coef[2 * j + 1];
      xr = __builtin_fma(mr, cr, __builtin_fma(mi, ci, xr));
      xi = __builtin_fma(mi, cr, __builtin_fma(-mr, ci, xi));
    }
    ip[t] = __builtin_fma(coef[2 * t], xr, -(coef[2 * t + 1] * xi));
    out[1 + 2 * t] = 2.0 * xr;
    out[2 + 2 * t] = -2.0 * xi;
  }
  __syncthreads();
  if (t == 0) {
    double I = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) I += ip[k];
    out[0] = I;
  }
}

// One workgroup per chunk, one row of NV partial sums each.
// coef: (Re c_k, Im c_k) of the resonances (theta's first 2K entries, the
// launch's own arguments, or the
// table's copy of them).  Events pass with a cached grid
// matrix (M not null): the last workgroup, whose chunk is the shortest,
// also evaluates the normalization into norm_out (dalitz_cached_norm), so
// that the level-2 step only sums rows.  span: the launch's span record
// (span_begin / span_end), null when the launch is not measured.
template <class S, int MODE, int GRAD, int EPT = 1>
__device__ inline void dalitz_pass_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab,
                                        cdouble* __restrict__ coef, const double* __restrict__ ev, int64_t ld,
                                        int64_t n, int chunk, double* __restrict__ part,
                                        const double* __restrict__ M, double* __restrict__ norm_out,
                                        unsigned long long* __restrict__ span) {
  constexpr int NV = dal_nv(MODE, GRAD, S::K);
  __shared__ double lds[block_sum_lds(NV)];
  if (span) span_begin(span);
  dalitz_chunk<S, MODE, GRAD, EPT>(dc, tab, coef, ev, ld, n, blockIdx.x, chunk,
                                   part + (int64_t)blockIdx.x * NV, lds);
  if (MODE == kEvents && M && blockIdx.x == gridDim.x - 1) dalitz_cached_norm<S>(M, coef, norm_out);
  if (span) span_end(span);
}

// Grid cell c (column-major over the whole grid, nx ny < 2^30): its centre and
// whether it lies inside the region.
__device__ __forceinline__ bool dalitz_cell(const DalitzConst& dc, uint32_t c, double& s12, double& s13) {
  const uint32_t ix = c / (uint32_t)dc.ny;
  s12 = grid_centre(dc.a12, ix, dc.d12);
  s13 = grid_centre(dc.a13, c - ix * (uint32_t)dc.ny, dc.d13);
  return dalitz_inside(dc, s12, s13);
}

// One workgroup per chunk of grid cells, one row of sum A_i conj(A_j) each
// (Gram); a wave whose 64 cells all lie outside the region skips them.
template <class S>
__device__ inline void dalitz_gram_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab, int chunk,
                                        double* __restrict__ part) {
  constexpr int K = S::K;
  using G = Gram<K>;
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
    double Are[K], Aim[K], Tre[K], Tim[K], Gk[K], Sre = 0.0, Sim = 0.0;
    dalitz_amps<S, true, false, false>(dc, r0 + zero, (cdouble*)nullptr, s12, s13, dc.msum - s12 - s13, Are, Aim, Tre,
                                       Tim, Gk, Sre, Sim);
    if (!in) {
#pragma unroll
      for (int k = 0; k < K; ++k) Are[k] = Aim[k] = 0.0;
    }
    g.add(Are, Aim, lds);
  }
  g.reduce(lds, part + (int64_t)blockIdx.x * 2 * gram_count(K));
}

// ---------------------------------------------------------------- toy events
// P~(s12, s13) = |sum_k c_k A_k|^2 at one point.
template <class S>
__device__ __forceinline__ double dalitz_value(const DalitzConst& dc, const double* __restrict__ r,
                                               cdouble* __restrict__ coef, double s12, double s13) {
  constexpr int K = S::K;
  const double s23 = dc.msum - s12 - s13;
  double Are[K], Aim[K], Tre[K], Tim[K], Gk[K];
  double Sre = 0.0, Sim = 0.0;
  dalitz_amps<S, false, false>(dc, r, coef, s12, s13, s23, Are, Aim, Tre, Tim, Gk, Sre, Sim);
  return __builtin_fma(Sre, Sre, Sim * Sim);
}

// P~(x_i) / I per event (I: the level-2 step's output): the events pass's own
// amplitudes for the model's structure (ACC), one event per thread.  Bound by their
// FP64 instructions, as that pass.
template <class S>
__device__ inline void dalitz_eval_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab,
                                        const double* __restrict__ ev, int64_t ld, int64_t n,
                                        const double* __restrict__ norm, double* __restrict__ p) {
  constexpr int K = S::K;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const double s12 = ev[i], s13 = ev[ld + i];
  double Are[K], Aim[K], Tre[K], Tim[K], Gk[K];
  double Sre = 0.0, Sim = 0.0;
  dalitz_amps<S, false, false, true, true>(dc, &tab->r[0][0], (cdouble*)tab->coef, s12, s13, dc.msum - s12 - s13,
                                           Are, Aim, Tre, Tim, Gk, Sre, Sim);
  p[i] = __builtin_fma(Sre, Sre, Sim * Sim) / *norm;
}

// Largest P~ over the centres of the grid cells inside the region, as the
// bit pattern of a non-negative double (ordered like the value) in *vmax.
template <class S>
__device__ inline void dalitz_gridmax_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab,
                                           unsigned long long* __restrict__ vmax) {
  const uint32_t ncell = (uint32_t)dc.nx * (uint32_t)dc.ny;
  const double* r = &tab->r[0][0];
  double m = 0.0;
  for (uint32_t c = blockIdx.x * kBlock + threadIdx.x; c < ncell; c += gridDim.x * kBlock) {
    double s12, s13;
    if (!dalitz_cell(dc, c, s12, s13)) continue;
    m = fmax(m, dalitz_value<S>(dc, r, (cdouble*)tab->coef, s12, s13));
  }
  block_max(m, vmax);
}

// Events distributed as P~ by accept-reject from the bounding box
// [box12] x [box13] (the box of the kinematic limits, as the host computes
// it): event i, attempt a takes (u1, u2) from counter (i, 2a, 1) and u3 from
// counter (i, 2a + 1, 1) under key (k0, k1); the candidate
// (box12.lo + u1 (box12.hi - box12.lo), box13.lo + u2 (...)) is kept when it
// lies in the region and u3 W < P~.  An event whose accepted P~ exceeds W
// (the envelope was too low there) counts in bad[0]; an event not accepted
// within max_attempts is NaN and counts in bad[1].
template <class S>
__device__ inline void dalitz_gen_body(const DalitzConst& dc, const DalitzTable* __restrict__ tab, uint32_t k0,
                                       uint32_t k1, int64_t n, const double* __restrict__ Wp, double lo12,
                                       double hi12, double lo13, double hi13, int per_wave, int max_attempts,
                                       double* __restrict__ ev, int64_t ld,
                                       unsigned long long* __restrict__ bad) {
#pragma clang fp contract(off)
  __shared__ StagedLds lds;
  const double W = *Wp;
  if (!(W > 0.0 && W < __builtin_inf())) return;  // the host reports it
  const double* r = &tab->r[0][0];
  const double w12 = hi12 - lo12, w13 = hi13 - lo13;
  double p;
  accept_reject_staged(
      lds, n, per_wave, max_attempts,
      [&](int64_t i, int a, double& s12, double& s13) {
#pragma clang fp contract(off)
        double u1, u2;
        philox_uniforms((uint64_t)i, 2u * a, 1u, k0, k1, u1, u2);
        s12 = lo12 + u1 * w12;
        s13 = lo13 + u2 * w13;
        return dalitz_inside_quick(dc, s12, s13);
      },
      [&](int64_t i, int a, double s12, double s13) {
#pragma clang fp contract(off)
        double u3, unused;
        philox_uniforms((uint64_t)i, 2u * a + 1u, 1u, k0, k1, u3, unused);
        p = dalitz_value<S>(dc, r, (cdouble*)tab->coef, s12, s13);
        return u3 * W < p;
      },
      [&](int64_t i, double s12, double s13) {
        ev[i] = s12;
        ev[ld + i] = s13;
        if (p > W) atomicAdd(bad, 1ull);
      },
      [&](int64_t i) {
        ev[i] = ev[ld + i] = __builtin_nan("");
        atomicAdd(bad + 1, 1ull);
      });
}

}  // namespace fn

// Kernel NAME for shape S, mode, gradient level and events per thread and
// iteration (used by the generated source).
// coef null: the coefficients are the launch's arguments.
#define FN_DALITZ_KERNEL(NAME, S, MODE, GRAD, EPT)                                                           \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void NAME(                                               \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, const double* __restrict__ coef,           \
      fn::CoefArg ca, const double* __restrict__ ev, int64_t ld, int64_t n, int chunk,                         \
      double* __restrict__ part, const double* __restrict__ M, double* __restrict__ norm_out,                  \
      unsigned long long* __restrict__ span) {                                                                 \
    fn::cdouble* c = coef ? (fn::cdouble*)coef : (fn::cdouble*)&ca.v[0];                                       \
    fn::dalitz_pass_body<S, MODE, GRAD, EPT>(dc, tab, c, ev, ld, n, chunk, part, M, norm_out, span);       \
  }

// Density per event for shape S.
#define FN_DALITZ_EVAL(NAME, S)                                                                               \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void NAME(                                               \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, const double* __restrict__ ev, int64_t ld,  \
      int64_t n, const double* __restrict__ norm, double* __restrict__ p) {                                    \
    fn::dalitz_eval_body<S>(dc, tab, ev, ld, n, norm, p);                                                      \
  }

// Matrix pass for shape S.
#define FN_DALITZ_GRAM(NAME, S)                                                                               \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void NAME(                                               \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, int chunk, double* __restrict__ part) {     \
    fn::dalitz_gram_body<S>(dc, tab, chunk, part);                                                             \
  }

// Grid maximum and accept-reject generator for shape S.
#define FN_DALITZ_GEN(GRIDMAX, GEN, S)                                                                        \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void GRIDMAX(                                            \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, unsigned long long* __restrict__ vmax) {   \
    fn::dalitz_gridmax_body<S>(dc, tab, vmax);                                                                 \
  }                                                                                                            \
  extern "C" __global__ __launch_bounds__(fn::kBlock) void GEN(                                                \
      fn::DalitzConst dc, const fn::DalitzTable* __restrict__ tab, uint32_t k0, uint32_t k1, int64_t n,        \
      const double* __restrict__ W, double lo12, double hi12, double lo13, double hi13, int per_wave,          \
      int max_attempts, double* __restrict__ ev, int64_t ld, unsigned long long* __restrict__ bad) {           \
    fn::dalitz_gen_body<S>(dc, tab, k0, k1, n, W, lo12, hi12, lo13, hi13, per_wave, max_attempts, ev, ld,      \
                           bad);                                                                                \
  }
