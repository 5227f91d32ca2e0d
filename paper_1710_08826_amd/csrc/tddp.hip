// Time-dependent three-body Dalitz-plot model with D0 mixing (the paper's
// pi+ pi- pi0 time-dependent amplitude fit, Sec. 1 Table 2 and Fig. 2): host
// launchers and the kernels that do not depend on the model's structure (the
// level-2 step with the normalization quadratic form).  The per-event and
// normalization-matrix passes live in tddp_device.hpp and are compiled at
// model creation with the model's structure as compile-time constants.
#include <algorithm>
#include <sstream>

#include "internal.hpp"
#include "jit.hpp"
#include "kernels.hpp"
#include "tddp.hpp"

namespace fn {

int tddp_nv(int K, bool grad) { return grad ? 3 + 4 * K : 1; }

std::string tddp_jit_source(const DalitzConst& dc, const double* fixed_ls) {
  std::ostringstream o;
  o << "#include \"tddp_device.hpp\"\n";
  o << "struct fn_shape {\n  static constexpr int K = " << dc.K << ";\n  static constexpr int chan[" << dc.K
    << "] = {";
  for (int k = 0; k < dc.K; ++k) o << (k ? ", " : "") << dc.chan[k];
  o << "};\n  static constexpr int L[" << dc.K << "] = {";
  for (int k = 0; k < dc.K; ++k) o << (k ? ", " : "") << dc.L[k];
  // the first resonance with the same lineshape, among pairs 12 and 13 or in pair 23
  o << "};\n  static constexpr int REP[" << dc.K << "] = {";
  for (int k = 0; k < dc.K; ++k) {
    int rep = 0;
    while (rep < k && ((dc.chan[rep] == 2) != (dc.chan[k] == 2) || dc.L[rep] != dc.L[k] ||
                       fixed_ls[2 * rep] != fixed_ls[2 * k] || fixed_ls[2 * rep + 1] != fixed_ls[2 * k + 1]))
      ++rep;
    o << (k ? ", " : "") << rep;
  }
  o << "};\n};\n";
  o << "FN_TDDP_EVENTS(fn_tddp_ev0, fn_shape, false)\n"
       "FN_TDDP_EVENTS(fn_tddp_ev1, fn_shape, true)\n"
       "FN_TDDP_GRAM(fn_tddp_gram, fn_shape)\n"
       "FN_TDDP_GEN(fn_tddp_gmax, fn_tddp_gen, fn_shape)\n";
  return o.str();
}

std::shared_ptr<TddpJit> tddp_jit(const DalitzConst& dc, const double* fixed_ls) {
  auto j = std::make_shared<TddpJit>();
  j->prog = jit_load(tddp_jit_source(dc, fixed_ls), {"fn_tddp_ev0", "fn_tddp_ev1", "fn_tddp_gram", "fn_tddp_gmax",
                                                     "fn_tddp_gen"});
  const auto& f = j->prog->fns;
  j->ev[0] = f[0];
  j->ev[1] = f[1];
  j->gram = f[2];
  j->gmax = f[3];
  j->gen = f[4];
  return j;
}

// ------------------------------------------------------------- kernels
__global__ void tddp_copy_theta(ParamBlock pb, int P, double* __restrict__ dst) {
  const int p = threadIdx.x;
  if (p < P) dst[p] = pb.v[p];
}

struct TddpFinalLds {
  double scratch[kFinalBlock];
  double res[kBlock];
  double X[kDalMaxRes][2], Xb[kDalMaxRes][2], U[kDalMaxRes][2], V[kDalMaxRes][2];
  double form[4][kDalMaxRes];  // resonance k's term of Ia, Ib, Re Z, Im Z
};

// Level 2 and the normalization
//   I = 1/2 [cy (Ia + Ib) + cx (Ia - Ib) - 2 y cy Re Z - 2 x cx Im Z],
//   Ia = sum c_i conj(c_j) MAA_ij, Ib = sum cbar_i conj(cbar_j) MBB_ij,
//   Z = sum conj(c_i) cbar_j MAB_ij, cy = tau/(1-y^2), cx = tau/(1+x^2),
// with X_k = sum_j MAA_kj conj(c_j), Xb_k = sum_j MBB_kj conj(cbar_j),
// U_i = sum_j MAB_ij cbar_j, V_j = sum_i conj(c_i) MAB_ij:
//   dIa/dRe c_k = 2 Re X_k, dIa/dIm c_k = -2 Im X_k (Ib, cbar and Xb alike),
//   dZ/dRe c_i = U_i, dZ/dIm c_i = -i U_i, dZ/dRe cbar_j = V_j, dZ/dIm cbar_j = i V_j.
// out = [NLL, grad(P), I, dI(P)].
__global__ __launch_bounds__(kFinalBlock) void tddp_finalize(DalitzConst dc, const DalitzTable* __restrict__ tab,
                                                             TddpTime tt, const double* __restrict__ coef_dev,
                                                             TddpArg ca, const double* __restrict__ part,
                                                             int64_t nrows, int nv,
                                                             int with_grad, const double* __restrict__ Mc,
                                                             double n_events, double* __restrict__ out,
                                                             double* __restrict__ out_user) {
  __shared__ TddpFinalLds L;
  const double* coef = coef_dev ? coef_dev : ca.v;  // null: theta is the launch's argument
  const int K = dc.K;
  const int P = 4 * K + 2;
  const int t = threadIdx.x;
  // Row k of the matrix-vector products goes to 16 lanes, one column j each,
  // whose sums take four steps: with a thread per row, its serial sum and then
  // the serial sum over k took half of the step (1M events, 16 resonances: the
  // step 11.5 -> 8.4 us).  The elements and coefficients are loaded before the row
  // sums, so that their latency overlaps them.
  const int k = t >> 4, j = t & 15;
  const bool on = k < K && j < K;
  static_assert(kDalMaxRes == 16, "a row of 16 lanes per resonance");
  cplx maa{0.0, 0.0}, mbb{0.0, 0.0}, mab{0.0, 0.0}, mba{0.0, 0.0}, cj{0.0, 0.0}, bj{0.0, 0.0}, ck{0.0, 0.0}, bk{0.0, 0.0};
  if (on) {
    const double* m = Mc + 2 * (k * K + j);
    const int nm = 2 * K * K;
    const double* mt = Mc + 2 * nm + 2 * (j * K + k);
    maa = {m[0], m[1]};
    mbb = {m[nm], m[nm + 1]};
    mab = {m[2 * nm], m[2 * nm + 1]};
    mba = {mt[0], mt[1]};
    cj = {coef[2 * j], coef[2 * j + 1]};
    bj = {coef[2 * K + 2 * j], coef[2 * K + 2 * j + 1]};
    ck = {coef[2 * k], coef[2 * k + 1]};
    bk = {coef[2 * K + 2 * k], coef[2 * K + 2 * k + 1]};
  }
  // the same for the uniform values, as vector loads (a lane-varying zero
  // offset): scalar ones would be waited for before the rows are requested
  int zero = 0;
  asm volatile("" : "+v"(zero));
  const double x = coef[4 * K + zero], y = coef[4 * K + 1 + zero], valid = (&tab->valid)[zero];
  sum_rows_t<kFinalBlock>(part, nrows, nv, L.scratch, L.res);
  if (t < 16 * kDalMaxRes) {
    // X_k = sum_j MAA_kj conj(c_j), Xb_k alike, U_k = sum_j MAB_kj cbar_j, V_k = sum_i conj(c_i) MAB_ik
    const double xr = row16_sum(maa.re * cj.re + maa.im * cj.im), xi = row16_sum(maa.im * cj.re - maa.re * cj.im);
    const double br = row16_sum(mbb.re * bj.re + mbb.im * bj.im), bi = row16_sum(mbb.im * bj.re - mbb.re * bj.im);
    const double ur = row16_sum(mab.re * bj.re - mab.im * bj.im), ui = row16_sum(mab.re * bj.im + mab.im * bj.re);
    const double vr = row16_sum(cj.re * mba.re + cj.im * mba.im), vi = row16_sum(cj.re * mba.im - cj.im * mba.re);
    if (j == 0) {
      L.X[k][0] = xr; L.X[k][1] = xi;
      L.Xb[k][0] = br; L.Xb[k][1] = bi;
      L.U[k][0] = ur; L.U[k][1] = ui;
      L.V[k][0] = vr; L.V[k][1] = vi;
      L.form[0][k] = ck.re * xr - ck.im * xi;  // Re(c_k X_k)
      L.form[1][k] = bk.re * br - bk.im * bi;
      L.form[2][k] = ck.re * ur + ck.im * ui;  // conj(c_k) U_k
      L.form[3][k] = ck.re * ui - ck.im * ur;
    }
  }
  __syncthreads();
  if (t >= ((P + 63) & ~63)) return;  // (whole waves: no barrier follows)
  const double Ia = row16_sum(L.form[0][j]), Ib = row16_sum(L.form[1][j]);
  const double Zr = row16_sum(L.form[2][j]), Zi = row16_sum(L.form[3][j]);
  const double tau = 1.0 / tt.gamma;
  const double dy = 1.0 - y * y, dx = 1.0 + x * x;
  const double cy = tau / dy, cx = tau / dx;
  const double I = 0.5 * (cy * (Ia + Ib) + cx * (Ia - Ib) - 2.0 * y * cy * Zr - 2.0 * x * cx * Zi);
  const bool ok = valid != 0.0 && I > 0.0 && isfinite(I) && dy > 0.0;
  if (t == 0) {
    const double v = ok ? L.res[0] + n_events * log(I) : INFINITY;
    out[0] = v;
    out[1 + P] = I;
    if (out_user) out_user[0] = v;
  }
  if (t < P) {
    double dI;
    if (t < 2 * K) {
      const int k = t >> 1;
      dI = (t & 1) == 0 ? 0.5 * (2.0 * (cy + cx) * L.X[k][0] - 2.0 * y * cy * L.U[k][0] - 2.0 * x * cx * L.U[k][1])
                        : 0.5 * (-2.0 * (cy + cx) * L.X[k][1] - 2.0 * y * cy * L.U[k][1] + 2.0 * x * cx * L.U[k][0]);
    } else if (t < 4 * K) {
      const int k = (t - 2 * K) >> 1;
      dI = (t & 1) == 0 ? 0.5 * (2.0 * (cy - cx) * L.Xb[k][0] - 2.0 * y * cy * L.V[k][0] - 2.0 * x * cx * L.V[k][1])
                        : 0.5 * (-2.0 * (cy - cx) * L.Xb[k][1] + 2.0 * y * cy * L.V[k][1] - 2.0 * x * cx * L.V[k][0]);
    } else if (t == 4 * K) {
      const double dcx = -2.0 * x * tau / (dx * dx), dxcx = tau * (1.0 - x * x) / (dx * dx);
      dI = 0.5 * ((Ia - Ib) * dcx - 2.0 * Zi * dxcx);
    } else {
      const double dcy = 2.0 * y * tau / (dy * dy), dycy = tau * (1.0 + y * y) / (dy * dy);
      dI = 0.5 * ((Ia + Ib) * dcy - 2.0 * Zr * dycy);
    }
    out[2 + P + t] = dI;
    if (with_grad) {
      const double g = ok ? L.res[1 + t] + n_events * dI / I : NAN;
      out[1 + t] = g;
      if (out_user) out_user[1 + t] = g;
    }
  }
}

// ------------------------------------------------------------- launchers
void tddp_launch_copy_theta(const ParamBlock& pb, int P, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(tddp_copy_theta, dim3(1), dim3(kBlock), 0, s, pb, P, dst);
}

size_t tddp_gram_doubles(const DalitzConst& dc) {
  const int64_t ncell = (int64_t)dc.nx * dc.ny;
  const int chunk = gram_chunk(ncell);
  return (size_t)((ncell + chunk - 1) / chunk) * 2 * gram_count(2 * dc.K);
}

void tddp_launch_mmatrices(const TddpJit& j, const DalitzConst& dc, const DalitzTable* tab, double* part, double* Mc,
                           hipStream_t s) {
  const int64_t ncell = (int64_t)dc.nx * dc.ny;
  DalitzConst c = dc;
  const DalitzTable* t = tab;
  int ch = gram_chunk(ncell);
  const int64_t nch = (ncell + ch - 1) / ch;
  double* p = part;
  void* args[] = {&c, &t, &ch, &p};
  jit_launch(j.gram, (unsigned)nch, kBlock, s, args);
  launch_gram_finalize(part, nch, 2 * dc.K, kGramMixing, dc.K, dc.dA, 1, nullptr, Mc, 0, s);
}

void tddp_launch_gridmax(const TddpJit& j, const DalitzConst& dc, const DalitzTable* tab, const double* coef,
                         unsigned long long* vmax, hipStream_t s) {
  const int64_t ncell = (int64_t)dc.nx * dc.ny;
  const int64_t blocks = std::min<int64_t>((ncell + kBlock - 1) / kBlock, kMaxBlocks);
  DalitzConst c = dc;
  const DalitzTable* t = tab;
  const double* cf = coef;
  unsigned long long* v = vmax;
  void* args[] = {&c, &t, &cf, &v};
  jit_launch(j.gmax, (unsigned)blocks, kBlock, s, args);
}

void tddp_launch_gen(const TddpJit& j, const DalitzConst& dc, const DalitzTable* tab, const double* coef,
                     const TddpTime& tt, uint32_t k0, uint32_t k1, int64_t n, const double* W, const double box[4],
                     int max_attempts, double* ev, int64_t ld, unsigned long long* bad, hipStream_t s) {
  if (n == 0) return;
  DalitzConst c = dc;
  const DalitzTable* t = tab;
  const double* cf = coef;
  TddpTime tm = tt;
  uint32_t a0 = k0, a1 = k1;
  int64_t nn = n, l = ld;
  const double* w = W;
  double b0 = box[0], b1 = box[1], b2 = box[2], b3 = box[3];
  int pw = gen_per_wave(n), ma = max_attempts;
  double* e = ev;
  unsigned long long* b = bad;
  void* args[] = {&c, &t, &cf, &tm, &a0, &a1, &nn, &w, &b0, &b1, &b2, &b3, &pw, &ma, &e, &l, &b};
  jit_launch(j.gen, gen_blocks(n), kBlock, s, args);
}

void tddp_launch_events(const TddpJit& j, const DalitzConst& dc, const DalitzTable* tab, const TddpTime& tt,
                        const double* coef, const TddpArg& ca, const double* ev, int64_t ld, int64_t n, int chunk,
                        int64_t nchunks, bool grad, double* part, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  if (nchunks == 0) return;
  DalitzConst c = dc;
  const DalitzTable* t = tab;
  TddpTime tm = tt;
  const double* cf = coef;
  TddpArg a = ca;
  const double* e = ev;
  int64_t l = ld, nn = n;
  int ch = chunk;
  double* p = part;
  void* args[] = {&c, &t, &tm, &cf, &a, &e, &l, &nn, &ch, &p};
  jit_launch(j.ev[grad ? 1 : 0], (unsigned)nchunks, kBlock, s, args, start, stop);
}

void tddp_launch_finalize(const DalitzConst& dc, const DalitzTable* tab, const TddpTime& tt, const double* coef,
                          const TddpArg& ca, const double* part, int64_t nrows, bool grad, const double* Mc, double n_events,
                          double* out, double* out_user, hipStream_t s) {
  hipLaunchKernelGGL(tddp_finalize, dim3(1), dim3(kFinalBlock), 0, s, dc, tab, tt, coef, ca, part, nrows,
                     tddp_nv(dc.K, grad), grad ? 1 : 0, Mc, n_events, out, out_user);
}

}  // namespace fn
