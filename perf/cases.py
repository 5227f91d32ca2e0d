"""Timed cases of the fitting engine: what a fit, a toy study or a systematics study has the library do,
over the sizes the benchmark, the tests and the model descriptions of this repository use.

A case is a dict of plain values: the model ("model"), the entry point ("call") and the sizes.  Models:
  mix     one-observable mixture (signal peak over background), 3 to 6 parameters
  dal     three-body Dalitz plot, fixed lineshapes: normalization matrix cached in the model
  dalfree the same with free masses and widths: normalization grid integrated on every call
  tddp    time-dependent three-body Dalitz plot with mixing
  td4     time-dependent four-body decay with a phase-space normalization sample
Calls: "nll" (value, or value and gradient, theta on the host: what a minimizer calls), "async" (theta and
result on the device), "eval" (density per event), "fits" (a batch of toy fits to convergence),
"variations" (one sample, many sets of fixed constants) and "toys" (events drawn from the model).
"""
import math

import numpy as np
import torch

from paper_1710_08826_amd import Batch, Model, VariationBatch

# ------------------------------------------------------------------ models
# (pair, L, mass, width, Re c, Im c): the eight-resonance D0 -> K pi pi0-like model
DAL_MASSES = (1.865, 0.494, 0.140, 0.135)
DAL_RES = (("23", 1, 0.770, 0.150, 1.0, 0.0), ("12", 1, 0.892, 0.050, -0.4662, 0.1697),
           ("13", 1, 0.892, 0.050, 0.3778, -0.1375), ("12", 0, 1.430, 0.270, 0.0796, 0.1378),
           ("13", 0, 1.430, 0.270, -0.0651, -0.1127), ("12", 2, 1.430, 0.100, 0.8751, 0.5052),
           ("23", 1, 1.700, 0.250, -0.2214, 1.2557), ("13", 1, 1.900, 0.300, 0.4792, -0.8300))
# sixteen resonances of a pi0 pi+ pi- final state, time-dependent
TDDP_MASSES = (1.86484, 0.1349766, 0.13957, 0.13957)
TDDP_RES = (("12", 1, 0.7753, 0.1491, 1.0, 0.0), ("13", 1, 0.7753, 0.1491, 0.588, 0.010),
            ("23", 1, 0.7753, 0.1491, 0.714, -0.020), ("12", 1, 1.465, 0.400, -0.252, 0.189),
            ("13", 1, 1.465, 0.400, -0.179, 0.118), ("23", 1, 1.465, 0.400, 0.213, -0.156),
            ("12", 1, 1.720, 0.250, 0.310, -0.270), ("13", 1, 1.720, 0.250, 0.220, 0.190),
            ("23", 1, 1.720, 0.250, -0.140, 0.330), ("23", 0, 0.990, 0.070, 0.080, -0.035),
            ("23", 0, 1.370, 0.350, 0.160, 0.120), ("23", 0, 1.505, 0.109, -0.090, 0.070),
            ("23", 0, 1.720, 0.135, 0.050, -0.040), ("23", 2, 1.2755, 0.1867, 0.194, -0.110),
            ("23", 0, 0.500, 0.400, 0.210, 0.150), ("23", 2, 1.525, 0.073, 0.060, 0.045))
TDDP_TAU, TDDP_SIGMA = 0.4101, 0.1
# K+ K- pi+ pi-: pair entries (L, mass, width; mass 0 is flat), basis functions (r12, r34, angular factor)
TD4_MASSES = (1.865, 0.494, 0.494, 0.140, 0.140)
TD4_TAU, TD4_SIGMA = 0.41, 0.05
TD4_R12 = ((0, 0.0, 0.0), (1, 1.019461, 0.004249), (0, 1.370, 0.350), (0, 1.505, 0.109))
TD4_R34 = ((0, 0.0, 0.0), (1, 0.77526, 0.1491), (0, 0.990, 0.070), (1, 0.78266, 0.00868))
TD4_ABAR = ((1, 1, 3), (1, 1, 4), (1, 1, 5), (1, 0, 2), (1, 2, 2), (0, 1, 1), (2, 1, 1), (0, 0, 0), (0, 2, 0), (2, 2, 0))
TD4_A = ((1, 3, 3), (1, 3, 4), (1, 3, 5), (0, 3, 1), (2, 3, 1), (3, 1, 1), (3, 3, 1), (2, 0, 0), (3, 0, 0), (3, 2, 0))
TD4_CBAR = (1.0, 0.0, 0.55, -0.35, -0.40, 0.60, 1.30, 0.25, 0.35, -0.45, 0.70, 0.40, -0.25, 0.50, 0.60, -0.20, 0.45, 0.35,
            -0.30, -0.25)
TD4_C = (0.20, 0.0, 0.06, 0.08, -0.05, 0.09, 0.12, -0.07, 0.04, 0.10, 0.09, -0.11, -0.07, 0.05, 0.10, 0.03, -0.04, -0.08,
         0.06, 0.05)
GRID = (1024, 1024)
MIX_LO, MIX_HI = {"gauss+exp": -10.0, "argus+gauss": 0.0, "gauss+gauss+exp": -10.0}, 10.0


def listed():
    return [
        # one toy of a coverage study: the smallest sample the toy batches are drawn from is about this size
        {"name": "mix toy", "model": "mix", "call": "nll", "shape": "gauss+exp", "n": 3001, "grad": True},
        # a mass fit of ordinary size, one evaluation of its minimizer
        {"name": "mix 1e5", "model": "mix", "call": "nll", "shape": "gauss+exp", "n": 100000, "grad": True},
        # a mass fit above the last-level cache, evaluated back to back
        {"name": "mix 2^26", "model": "mix", "call": "async", "shape": "gauss+exp", "n": 1 << 26, "grad": True},
        # a toy study: samples of log-uniform size fitted to convergence together
        {"name": "toy fits", "model": "mix", "call": "fits", "shape": "gauss+exp", "fits": 512, "n_lo": 1000, "n_hi": 200000},
        # an amplitude fit of a small selected sample
        {"name": "dalitz 2e4", "model": "dal", "call": "nll", "res": 8, "n": 20011, "grad": True},
        # the headline amplitude fit, evaluated back to back with theta on the device
        {"name": "dalitz 1e6", "model": "dal", "call": "async", "res": 8, "n": 1000000, "grad": True},
        # masses and widths free: the normalization is integrated again on each evaluation
        {"name": "dalitz free 4e6", "model": "dalfree", "call": "nll", "res": 8, "n": 4000000, "grad": True},
        # the time-dependent mixing fit
        {"name": "mixing 1e6", "model": "tddp", "call": "nll", "res": 16, "n": 1000000, "grad": True},
        # the four-body mixing fit, the largest sample of the benchmark
        {"name": "four-body 1e7", "model": "td4", "call": "nll", "n": 10000000, "n_mc": 500000, "grad": True},
        # systematics: the first evaluation of a new set of fixed constants per fit
        {"name": "four-body variations", "model": "td4", "call": "variations", "fits": 16, "n": 300007, "n_mc": 300000, "grad": True},
        # density per event of a fitted model, for projections and weights
        {"name": "four-body density", "model": "td4", "call": "eval", "n": 1000003, "n_mc": 100000},
        # toy events drawn from the model
        {"name": "dalitz toys", "model": "dal", "call": "toys", "res": 8, "n": 500009},
    ]


def draw(rng):
    def size(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return n | 1 if rng.random() < 0.5 else n

    kind = rng.choice(["mix", "mix", "mix async", "fits", "dal", "dal async", "dalfree", "tddp", "td4", "variations", "eval", "toys"])
    grad = rng.random() < 0.8  # the others: scans and line searches that ask for the value alone
    shape = rng.choice(sorted(MIX_LO))
    if kind in ("mix", "mix async"):
        return {"model": "mix", "call": "nll" if kind == "mix" else "async", "shape": shape, "n": size(1000, 1 << 25), "grad": grad}
    if kind == "fits":
        return {"model": "mix", "call": "fits", "shape": "gauss+exp", "fits": size(8, 500), "n_lo": 1000, "n_hi": size(5000, 150000)}
    if kind in ("dal", "dal async"):
        return {"model": "dal", "call": "nll" if kind == "dal" else "async", "res": rng.randint(3, 8), "n": size(5000, 4000000), "grad": grad}
    if kind == "dalfree":
        return {"model": "dalfree", "call": "nll", "res": rng.randint(3, 8), "n": size(5000, 3900000), "grad": grad}
    if kind == "tddp":
        return {"model": "tddp", "call": "nll", "res": rng.randint(6, 16), "n": size(10000, 2000000), "grad": grad}
    if kind == "td4":
        return {"model": "td4", "call": "nll", "n": size(20000, 6000000), "n_mc": size(100000, 400000), "grad": grad}
    if kind == "variations":
        return {"model": "td4", "call": "variations", "fits": rng.randint(2, 16), "n": size(20000, 300000), "n_mc": size(50000, 290000), "grad": grad}
    if kind == "eval":
        return {"model": rng.choice(["td4", "dal"]), "call": "eval", "res": 8, "n": size(10000, 1000000), "n_mc": 50000}
    return {"model": "dal", "call": "toys", "res": rng.randint(5, 8), "n": size(10000, 500000)}


# ------------------------------------------------------------------ inputs
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _uniforms(seed, stream, rows, n):
    g = torch.Generator(device=_device())
    g.manual_seed(int(seed) * 64 + stream)
    return torch.rand((rows, n), generator=g, device=_device(), dtype=torch.float64)


def _normal(u, v):
    return torch.sqrt(-2.0 * torch.log1p(-u)) * torch.cos(2.0 * math.pi * v)


def _mix_events(case, seed, n, stream=1):
    """Peak over a falling background, inside the range (reflected into it where a draw falls outside)."""
    lo, hi = MIX_LO[case["shape"]], MIX_HI
    u = _uniforms(seed, stream, 4, n)
    if case["shape"] == "argus+gauss":
        peak, tail = 5.0 + 0.8 * _normal(u[1], u[2]), 9.0 * torch.sqrt(u[3]) * torch.sqrt(torch.sqrt(u[1]))
    else:
        width = torch.where(u[2] < 0.3, 2.2, 1.1) if case["shape"] == "gauss+gauss+exp" else 1.1
        peak, tail = 0.2 + width * _normal(u[1], u[2]), lo + torch.log1p(u[3] * math.expm1(-0.3 * (hi - lo))) / -0.3
    x = torch.where(u[0] < 0.7, peak, tail)
    x = torch.where(x < lo, 2.0 * lo - x, x)
    x = torch.where(x > hi, 2.0 * hi - x, x)
    return x.clamp(lo + 1e-3, hi - 1e-3).reshape(1, n)


def _cauchy(u, m0, w, lo, hi):
    a, b = torch.atan((lo - m0) / (0.5 * w)), torch.atan((hi - m0) / (0.5 * w))
    return torch.minimum(torch.maximum(m0 + 0.5 * w * torch.tan(a + u * (b - a)), lo), hi)


def _dalitz_events(masses, res, seed, n):
    """(s12, s13): a smooth component and one band per resonance, isotropic in the pair's rest frame."""
    M, m = masses[0], {1: masses[1], 2: masses[2], 3: masses[3]}
    msum = sum(v * v for v in masses)
    u = _uniforms(seed, 1, 3, n)
    which = (u[0] * (len(res) + 2)).long()  # the last two shares: the smooth component
    out = torch.empty((2, n), dtype=torch.float64, device=u.device)
    table = [(r[0], r[2], r[3]) for r in res] + [("12", None, None)]
    for k, (pair, m0, w) in enumerate(table):
        at = which == k if m0 is not None else which >= k
        a, b, c = {"12": (1, 2, 3), "13": (1, 3, 2), "23": (2, 3, 1)}[pair]
        lo, hi = torch.tensor([m[a] + m[b] + 1e-6, M - m[c] - 1e-6], dtype=torch.float64, device=u.device)
        v = u[1][at]
        s = (lo + v * (hi - lo) if m0 is None else _cauchy(v, m0, w, lo, hi)) ** 2
        r = torch.sqrt(s)
        ea, ec = (s + m[a] ** 2 - m[b] ** 2) / (2 * r), (M * M - s - m[c] ** 2) / (2 * r)
        pa, pc = torch.sqrt((ea * ea - m[a] ** 2).clamp(min=0.0)), torch.sqrt((ec * ec - m[c] ** 2).clamp(min=0.0))
        s_ac = m[a] ** 2 + m[c] ** 2 + 2 * (ea * ec - pa * pc * (2 * u[2][at] - 1))
        s_bc = msum - s - s_ac
        out[0, at], out[1, at] = {"12": (s, s_ac), "13": (s_ac, s), "23": (s_ac, s_bc)}[pair]
    return out


def _td4_points(seed, stream, n, bands):
    """(m12, m34, cos12, cos34, phi): masses uniform or in a resonance band, angles uniform."""
    M, m1, m2, m3, m4 = TD4_MASSES
    u = _uniforms(seed, stream, 7, n)
    lo, hi = torch.tensor(m1 + m2 + 1e-6, dtype=torch.float64, device=u.device), M - m3 - m4 - 1e-5
    hi = torch.tensor(hi, dtype=torch.float64, device=u.device)
    m12 = lo + u[0] * (hi - lo)
    if bands:
        m12 = torch.where(u[5] < bands, _cauchy(u[0], *TD4_R12[1][1:], lo, hi), m12)
    lo = torch.full_like(m12, m3 + m4 + 1e-6)
    hi = M - m12 - 1e-6
    m34 = lo + u[1] * (hi - lo)
    if bands:
        m34 = torch.where(u[6] < bands, _cauchy(u[1], *TD4_R34[1][1:], lo, hi), m34)
    return torch.stack([m12, m34, 2 * u[2] - 1, 2 * u[3] - 1, (2 * u[4] - 1) * math.pi])


def _times(seed, stream, n, tau, sigma):
    u = _uniforms(seed, stream, 3, n)
    return (-tau * torch.log1p(-u[0]) + sigma * _normal(u[1], u[2])).reshape(1, n)


def _events(case, seed):
    n = case["n"]
    if case["model"] == "mix":
        return _mix_events(case, seed, n)
    if case["model"] in ("dal", "dalfree"):
        return _dalitz_events(DAL_MASSES, DAL_RES[: case["res"]], seed, n)
    if case["model"] == "tddp":
        d = _dalitz_events(TDDP_MASSES, TDDP_RES[: case["res"]], seed, n)
        return torch.cat([d, _times(seed, 2, n, TDDP_TAU, TDDP_SIGMA)])
    return torch.cat([_td4_points(seed, 1, n, 0.3), _times(seed, 2, n, TD4_TAU, TD4_SIGMA)])


def _description(case):
    def res(table):
        return [{"pair": r[0], "L": r[1], "m0": r[2], "w0": r[3]} for r in table]

    if case["model"] == "mix":
        comps = {"gauss+exp": [("gauss", [0, 1]), ("exp", [2])], "argus+gauss": [("argus", [0, 1]), ("gauss", [2, 3])],
                 "gauss+gauss+exp": [("gauss", [0, 1]), ("gauss", [0, 2]), ("exp", [3])]}[case["shape"]]
        first = 1 + max(i for _, p in comps for i in p)
        return {"kind": "mix1d", "lo": MIX_LO[case["shape"]], "hi": MIX_HI, "n_params": first + len(comps) - 1,
                "components": [{"type": t, "params": p} for t, p in comps], "fracs": list(range(first, first + len(comps) - 1))}
    if case["model"] in ("dal", "dalfree"):
        return {"kind": "dalitz3", "M": DAL_MASSES[0], "m": list(DAL_MASSES[1:]), "r_res": 1.5, "r_D": 5.0, "grid": list(GRID),
                "free_lineshapes": case["model"] == "dalfree", "resonances": res(DAL_RES[: case["res"]])}
    if case["model"] == "tddp":
        return {"kind": "tddp3", "M": TDDP_MASSES[0], "m": list(TDDP_MASSES[1:]), "r_res": 1.5, "r_D": 5.0, "grid": list(GRID),
                "tau": TDDP_TAU, "sigma_t": TDDP_SIGMA, "resonances": res(TDDP_RES[: case["res"]])}
    return {"kind": "td4", "M": TD4_MASSES[0], "m": list(TD4_MASSES[1:]), "r_res": 1.5, "tau": TD4_TAU, "sigma_t": TD4_SIGMA,
            "r12": [{"L": a, "m0": b, "w0": c} for a, b, c in TD4_R12], "r34": [{"L": a, "m0": b, "w0": c} for a, b, c in TD4_R34],
            "amps": [list(a) + ["Abar"] for a in TD4_ABAR] + [list(a) + ["A"] for a in TD4_A]}


def _truth(case):
    if case["model"] == "mix":
        return {"gauss+exp": [0.2, 1.1, -0.3, 0.7], "argus+gauss": [10.5, -1.5, 5.0, 0.8, 0.3],
                "gauss+gauss+exp": [0.2, 1.1, 2.2, -0.3, 0.5, 0.2]}[case["shape"]]
    if case["model"] in ("dal", "dalfree"):
        r = DAL_RES[: case["res"]]
        return [v for t in r for v in t[4:]] + ([v for t in r for v in t[2:4]] if case["model"] == "dalfree" else [])
    if case["model"] == "tddp":
        c = [v for t in TDDP_RES[: case["res"]] for v in t[4:]]
        return c + c + [0.0039, 0.0065]
    return list(TD4_C) + list(TD4_CBAR) + [0.004, 0.006]


def _theta(case, seed, rows=0):
    """A point of the minimizer's path: the generation point moved by about a percent."""
    t = np.array(_truth(case), dtype=np.float64)
    z = np.random.RandomState(seed % (1 << 31)).standard_normal((max(rows, 1), t.size)).clip(-3, 3)
    th = t * (1.0 + 0.01 * z)
    return th if rows else th[0]


def _fit_sizes(case, seed):
    u = np.random.RandomState((seed + 17) % (1 << 31)).random_sample(case["fits"])
    return np.rint(np.exp(math.log(case["n_lo"]) + u * (math.log(case["n_hi"]) - math.log(case["n_lo"])))).astype(np.int64)


def _variations(case, seed, fixed):
    """Fixed constants of each fit: masses, widths and the resolution moved by up to half a percent."""
    z = np.random.RandomState((seed + 29) % (1 << 31)).uniform(-1, 1, (case["fits"], fixed.size))
    return fixed * (1.0 + 0.005 * z)


def _td4_fixed():
    return np.array([v for r in TD4_R12 + TD4_R34 for v in r[1:]] + [TD4_SIGMA])


# ------------------------------------------------------------------ the calls
def prepare(case, seed):
    s = {"case": case, "model": Model(_description(case))}
    call = case["call"]
    if call == "fits":
        sizes = _fit_sizes(case, seed)
        x = _mix_events(case, seed, int(sizes.sum()))
        s["events"] = [t.contiguous() for t in torch.split(x, sizes.tolist(), dim=1)]
        s["theta"] = torch.from_numpy(_theta(case, seed, case["fits"])).cuda()
        s["batch"] = Batch(s["model"], case["fits"], int(sizes.max()))
        return s
    if call == "toys":
        s["theta"], s["seed"] = _theta(case, seed), int(seed) % (1 << 31)
        return s
    s["events"] = _events(case, seed)
    if case["model"] == "td4":
        s["model"].set_norm_sample(_td4_points(seed, 3, case["n_mc"], 0.0))
    if call == "variations":
        s["theta"] = _theta(case, seed, case["fits"])
        s["fixed"] = _variations(case, seed, s["model"].fixed())
        s["batch"] = VariationBatch(s["model"], case["fits"])
        return s
    s["theta"] = _theta(case, seed)
    if call == "async":
        s["theta"] = torch.from_numpy(s["theta"]).cuda()
        s["out"] = torch.zeros(1 + s["model"].n_params, dtype=torch.float64, device="cuda")
    return s


def run(s):
    case, model = s["case"], s["model"]
    call = case["call"]
    if call == "nll":
        return model.nll(s["theta"], s["events"], grad=case["grad"])
    if call == "async":
        model.nll_async(s["theta"], s["events"], s["out"], with_grad=case["grad"])
        return s["out"] if case["grad"] else s["out"][:1]
    if call == "eval":
        return model.eval(s["theta"], s["events"])
    if call == "fits":
        s["batch"].set(s["events"], s["theta"])
        s["batch"].run()
        r = s["batch"].results()
        return {"status": r.status, "theta": r.theta, "nll": r.nll, "errors": r.errors}
    if call == "variations":
        for f, fixed in enumerate(s["fixed"]):
            s["batch"].set_fixed(f, fixed)
        return s["batch"].nll(s["theta"], s["events"], grad=case["grad"])
    events, envelope = model.generate(s["theta"], case["n"], s["seed"])
    return events, envelope


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes: each event read once, each result written once.  Operations: an addition or a product counts 1, a
    quotient or a square root 10, an exponential, a logarithm, a sine and cosine or an error function 30."""
    model, call, grad = case["model"], case["call"], case.get("grad", True)
    obs = {"mix": 1, "dal": 2, "dalfree": 2, "tddp": 3, "td4": 6}[model]
    k = case.get("res", 20)
    pars = len(_truth(case))
    if model == "mix":
        comps = len(case["shape"].split("+"))
        per = comps * 34 + 12 + (10 + 4 * pars if grad else 0)
    elif model in ("dal", "dalfree"):
        per = 3 * 60 + k * (24 + (8 if grad else 0) + (24 if grad and model == "dalfree" else 0)) + 20
    elif model == "tddp":
        per = 3 * 60 + 2 * k * (24 + (8 if grad else 0)) + 3 * 90 + 60
    else:
        per = 2 * 40 + 6 * 20 + 20 * (12 + (12 if grad else 0)) + 3 * 90 + 30 + 60
    if call == "fits":  # twenty evaluations to convergence with errors, of the mean size
        n = 20.0 * case["fits"] * (case["n_hi"] - case["n_lo"]) / math.log(case["n_hi"] / case["n_lo"])
        return {"bytes": 8 * n, "flops": per * n}
    if call == "toys":  # twenty attempts per event, half of them outside the region
        return {"bytes": 16 * case["n"], "flops": case["n"] * 10.0 * (per - 8 * k)}
    n, extra = case["n"], 0.0
    if call == "variations":  # every fit's normalization matrix: Hermitian, 20 x 20
        extra = case["fits"] * case["n_mc"] * (2 * 40 + 6 * 20 + 30 + 20 * 8 + 8 * 210)
        return {"bytes": 8 * (6 * n + 5 * case["n_mc"]), "flops": case["fits"] * n * per + extra}
    if model == "dalfree":
        extra = 0.475 * GRID[0] * GRID[1] * per
    return {"bytes": 8.0 * (obs * n + (n if call == "eval" else 1 + pars)), "flops": n * per + extra}


# ------------------------------------------------------------------ the same in plain torch, 64 bits
def _mix_log_density(case, th, x):
    lo, hi = torch.tensor(MIX_LO[case["shape"]], dtype=torch.float64, device=x.device), MIX_HI
    hi = torch.tensor(hi, dtype=torch.float64, device=x.device)

    def gauss(mu, sg):
        z = torch.erf((hi - mu) / (sg * math.sqrt(2))) - torch.erf((lo - mu) / (sg * math.sqrt(2)))
        return torch.exp(-0.5 * ((x - mu) / sg) ** 2) / (sg * math.sqrt(math.pi / 2) * z)

    def expo(tau):
        return torch.exp(tau * x) / ((torch.exp(tau * hi) - torch.exp(tau * lo)) / tau)

    def argus(m0, c):
        w, wl, wh = (1 - (v / m0) ** 2 for v in (x, lo, hi))
        g = [math.sqrt(math.pi) / 2 * torch.erf(torch.sqrt(-c * v)) - torch.sqrt(-c * v) * torch.exp(c * v) for v in (wl, wh)]
        return x * torch.sqrt(w) * torch.exp(c * w) / (0.5 * m0 ** 2 * (-c) ** -1.5 * (g[0] - g[1]))

    if case["shape"] == "gauss+exp":
        return torch.log(th[3] * gauss(th[0], th[1]) + (1 - th[3]) * expo(th[2]))
    if case["shape"] == "argus+gauss":
        return torch.log(th[4] * argus(th[0], th[1]) + (1 - th[4]) * gauss(th[2], th[3]))
    return torch.log(th[4] * gauss(th[0], th[1]) + th[5] * gauss(th[0], th[2]) + (1 - th[4] - th[5]) * expo(th[3]))


def _lam(a, b, c):
    return (a - (math.sqrt(b) + math.sqrt(c)) ** 2) * (a - (math.sqrt(b) - math.sqrt(c)) ** 2)


def _amplitudes(masses, res, s12, s13, ls=None):
    """The isobar amplitudes of the resonances (ls: their masses and widths, the table's by default)."""
    M, m = masses[0], masses
    s23 = sum(v * v for v in m) - s12 - s13
    out = []
    for k, (pair, L, m0, w0, *_) in enumerate(res):
        if ls is not None:
            m0, w0 = ls[2 * k], ls[2 * k + 1]
        a, b, c = {"12": (1, 2, 3), "13": (1, 3, 2), "23": (2, 3, 1)}[pair]
        s, s_ac, s_bc = {"12": (s12, s13, s23), "13": (s13, s12, s23), "23": (s23, s12, s13)}[pair]
        ma, mb, mc = m[a] ** 2, m[b] ** 2, m[c] ** 2
        lq, lp = _lam(s, ma, mb).clamp(min=0.0), _lam(s, M * M, mc).clamp(min=0.0)
        q2, p2, q02 = lq / (4 * s), lp / (4 * s), _lam(m0 * m0, ma, mb) / (4 * m0 * m0)

        def poly(z):
            return 1.0 if L == 0 else 1 + z if L == 1 else z * z + 3 * z + 9

        fr2 = poly(q02 * 2.25) / poly(q2 * 2.25)
        gam = w0 * (q2 / q02) ** L * torch.sqrt(q2 / q02) * m0 / torch.sqrt(s) * fr2
        z1 = s_ac - s_bc + (M * M - mc) * (mb - ma) / s
        z = 1.0 if L == 0 else z1 if L == 1 else z1 * z1 - lp * lq / (3 * s * s)
        h = torch.sqrt(torch.as_tensor(fr2, dtype=torch.float64, device=s.device) / poly(p2 * 25.0)) * z
        re, im = m0 * m0 - s, m0 * gam
        out.append(torch.complex(h * re, h * im) / (re * re + im * im))
    return out


def _grid(masses, device):
    M, m1, m2, m3 = masses
    a, b = (m1 + m2) ** 2, (m1 + m3) ** 2
    d, e = ((M - m3) ** 2 - a) / GRID[0], ((M - m2) ** 2 - b) / GRID[1]
    s12, s13 = np.meshgrid(a + (np.arange(GRID[0]) + 0.5) * d, b + (np.arange(GRID[1]) + 0.5) * e, indexing="ij")
    r = np.sqrt(s12)
    e2, e3 = (s12 - m1 * m1 + m2 * m2) / (2 * r), (M * M - s12 - m3 * m3) / (2 * r)
    p2, p3 = np.sqrt(np.maximum(e2 * e2 - m2 * m2, 0)), np.sqrt(np.maximum(e3 * e3 - m3 * m3, 0))
    s23 = M * M + m1 * m1 + m2 * m2 + m3 * m3 - s12 - s13
    at = (s23 >= (e2 + e3) ** 2 - (p2 + p3) ** 2) & (s23 <= (e2 + e3) ** 2 - (p2 - p3) ** 2)
    return torch.from_numpy(np.stack([s12[at], s13[at]])).to(device), d * e


def _coefs(th, first, k):
    return [torch.complex(th[first + 2 * j], th[first + 2 * j + 1]) for j in range(k)]


def _time_functions(x, y, t, tau, sigma):
    """Hc, Hs, Hcos, Hsin: the Gaussian-smeared decay functions, from Taylor series of h(a; t) in a about 1/tau
    (h' = (a s^2 - t) h - s/sqrt(2 pi) exp(-t^2 / 2 s^2); x and y are far below one)."""
    G, s2 = 1.0 / tau, sigma * sigma
    g, u = torch.exp(-t * t / (2 * s2)), G * s2 - t
    z = u / (sigma * math.sqrt(2))
    ex = 0.5 * g * torch.special.erfcx(z.abs())
    h = [torch.where(z >= 0, ex, torch.exp(0.5 * G * G * s2 - G * t) - ex)]
    h.append(u * h[0] - sigma / math.sqrt(2 * math.pi) * g)
    for n in range(1, 18):
        h.append(u * h[n] + n * s2 * h[n - 1])
    even_y, odd_y, even_x, odd_x = 0.0, 0.0, 0.0, 0.0
    for n, v in enumerate(h):
        f = G ** n / math.factorial(n)
        if n % 2:
            odd_y, odd_x = odd_y - f * y ** n * v, odd_x - (-1) ** (n // 2) * f * x ** n * v
        else:
            even_y, even_x = even_y + f * y ** n * v, even_x + (-1) ** (n // 2) * f * x ** n * v
    return even_y, odd_y, even_x, odd_x


def _rate(A, B, H):
    a2, b2, z = A.real ** 2 + A.imag ** 2, B.real ** 2 + B.imag ** 2, A.conj() * B
    return 0.5 * ((a2 + b2) * H[0] + (a2 - b2) * H[2] - 2 * z.real * H[1] - 2 * z.imag * H[3])


def _integrals(x, y, tau):
    cy, cx = tau / (1 - y * y), tau / (1 + x * x)
    return cy, y * cy, cx, x * cx


def _td4_pair(m, entries, ma, mb, fixed):
    s, out = m * m, []
    q2 = (_lam(s, ma * ma, mb * mb) / (4 * s)).clamp(min=0.0)
    for r, (L, *_) in enumerate(entries):
        m0, w0 = float(fixed[2 * r]), float(fixed[2 * r + 1])
        if m0 == 0.0:
            out.append(torch.ones_like(s, dtype=torch.complex128))
            continue
        q02 = _lam(m0 * m0, ma * ma, mb * mb) / (4 * m0 * m0)
        f2 = (1 + q02 * 2.25) / (1 + q2 * 2.25) if L else torch.ones_like(s)
        gam = w0 * (q2 / q02) ** L * torch.sqrt(q2 / q02) * m0 / m * f2
        re, im = m0 * m0 - s, m0 * gam
        out.append(torch.sqrt(f2) * torch.complex(re, im) / (re * re + im * im))
    return out


def _td4_basis(p, fixed):
    M, m1, m2, m3, m4 = TD4_MASSES
    a = _td4_pair(p[0], TD4_R12, m1, m2, fixed[: 2 * len(TD4_R12)])
    b = _td4_pair(p[1], TD4_R34, m3, m4, fixed[2 * len(TD4_R12): -1])
    ss = 0.5 * torch.sqrt((1 - p[2] ** 2).clamp(min=0.0)) * torch.sqrt((1 - p[3] ** 2).clamp(min=0.0))
    om = (1.0, p[3], p[2], p[2] * p[3], torch.polar(ss, p[4]), torch.polar(ss, -p[4]))
    return [a[r1] * b[r2] * om[t] for r1, r2, t in TD4_ABAR + TD4_A]


def _sums(case, th, ev, fixed):
    """-sum ln P~ over the events, differentiable in th."""
    model = case["model"]
    if model == "mix":
        return -_mix_log_density(case, th, ev[0]).sum()
    if model in ("dal", "dalfree"):
        return -torch.log(_dal_density(case, th, ev)).sum()
    if model == "tddp":
        A, B = _tddp_sums(case, th, ev)
        return -torch.log(_rate(A, B, _time_functions(th[-2], th[-1], ev[2], TDDP_TAU, TDDP_SIGMA))).sum()
    return -torch.log(_td4_rate(th, ev, fixed)).sum()


def _dal_density(case, th, ev):
    k = case["res"]
    amp = _amplitudes(DAL_MASSES, DAL_RES[:k], ev[0], ev[1], th[2 * k:] if case["model"] == "dalfree" else None)
    S = sum(c * a for c, a in zip(_coefs(th, 0, k), amp))
    return S.real ** 2 + S.imag ** 2


def _tddp_sums(case, th, ev):
    k = case["res"]
    res = TDDP_RES[:k]
    A = sum(c * a for c, a in zip(_coefs(th, 0, k), _amplitudes(TDDP_MASSES, res, ev[0], ev[1])))
    B = sum(c * a for c, a in zip(_coefs(th, 2 * k, k), _amplitudes(TDDP_MASSES, res, ev[1], ev[0])))
    return A, B


def _td4_sums(th, p, fixed):
    b = _td4_basis(p, fixed)
    return sum(c * v for c, v in zip(_coefs(th, 0, 10), b[10:])), sum(c * v for c, v in zip(_coefs(th, 20, 10), b[:10]))


def _td4_rate(th, ev, fixed):
    A, B = _td4_sums(th, ev, fixed)
    return _rate(A, B, _time_functions(th[-2], th[-1], ev[5], TD4_TAU, float(fixed[-1])))


def _norm(case, th, seed, fixed):
    """The normalization integral, by adding up parts; each part is differentiated before the next."""
    if case["model"] == "mix":
        return
    if case["model"] == "td4":
        mc = _td4_points(seed, 3, case["n_mc"], 0.0)
        for p in torch.split(mc, 100000, dim=1):
            A, B = _td4_sums(th, p, fixed)
            yield _rate(A, B, _integrals(th[-2], th[-1], TD4_TAU)).sum() / case["n_mc"]
        return
    cells, area = _grid(TDDP_MASSES if case["model"] == "tddp" else DAL_MASSES, th.device)
    for p in torch.split(cells, 100000, dim=1):
        if case["model"] == "tddp":
            A, B = _tddp_sums(case, th, p)
            yield area * _rate(A, B, _integrals(th[-2], th[-1], TDDP_TAU)).sum()
        else:
            yield area * _dal_density(case, th, p).sum()


def _added(parts, th, grad):
    value, slope = 0.0, np.zeros(th.numel())
    for v in parts:
        value += float(v)
        if grad:
            slope += torch.autograd.grad(v, th)[0].cpu().numpy()
    return value, slope


def _nll(case, theta, ev, seed, fixed, grad):
    th = torch.from_numpy(np.array(theta)).to(ev.device).requires_grad_(grad)
    part = 4000000 if case["model"] == "mix" else 200000
    v, g = _added((_sums(case, th, p, fixed) for p in torch.split(ev, part, dim=1)), th, grad)
    if case["model"] != "mix":
        I, dI = _added(_norm(case, th, seed, fixed), th, grad)
        v, g = v + ev.shape[1] * math.log(I), g + ev.shape[1] * dI / I
    return v, g


def exact(case, seed):
    call = case["call"]
    if call in ("fits", "toys"):  # a fit stops within its tolerance of the minimum; toys are accepted draws
        return None
    grad, fixed = case.get("grad", False), _td4_fixed()
    ev = _events(case, seed)
    if call == "variations":
        both = [_nll(case, t, ev, seed, f, grad) for t, f in zip(_theta(case, seed, case["fits"]), _variations(case, seed, fixed))]
        v = np.array([b[0] for b in both])
        return (v, np.stack([b[1] for b in both])) if grad else v
    theta = _theta(case, seed)
    if call == "eval":
        th = torch.from_numpy(theta).to(ev.device)
        I, _ = _added(_norm(case, th, seed, fixed), th, False)
        parts = [_td4_rate(th, p, fixed) if case["model"] == "td4" else _dal_density(case, th, p) for p in torch.split(ev, 200000, dim=1)]
        return torch.cat(parts) / I
    v, g = _nll(case, theta, ev, seed, fixed, grad)
    if call == "async":
        return np.concatenate([[v], g]) if grad else np.array([v])
    return (v, g) if grad else v
