"""The workloads that the performance of this framework is measured on.

A case is one call, or one short run of calls, that a forecasting or
likelihood program makes through the public entry points (``wlcov.Problem``
and ``serve.Server``): the data vector, its response, the joint covariance and
the signal-to-noise of one survey set-up (``step``), the signal-to-noise of a
covariance that is already there (``snr2``), the principal components (``pca``),
the integer lattice counts (``lattice``) and a burst of likelihood requests
against a running server (``serve``).

Inputs are synthetic tables of the shape and distribution of the Euclid-like
forecast (flat LCDM background, equipopulated redshift bins, a broken power
law P(k), an exponentially cut mass function and a Gaussian halo profile),
their cosmology and survey scalars drawn from the seed.  ``exact`` evaluates
the same quantities with plain torch in 64 bits.
"""
import math
import random
from itertools import product

import numpy as np
import torch

from paper_1812_07437_amd import serve, wlcov

DEV = "cuda:0"
F64 = torch.float64
H0 = 1.0 / 2997.92458  # h/Mpc, c = 1
RHO_CRIT = 2.775e11    # (M_sun/h) / (Mpc/h)^3
N_K = 768              # k nodes of the P and u tables
N_EPS = 16384          # nodes of the survey window's integral


# --------------------------------------------------------------- the cases
def _step(name, n_z, n_ell, ell_min, ell_max, n_chi, n_m, precision, tomo="paper", snr="direct", ssc_chi=False,
          n_sub=1, bias=False, kind="step"):
    return dict(name=name, kind=kind, n_z=n_z, n_ell=n_ell, ell_min=ell_min, ell_max=ell_max, n_chi=n_chi, n_m=n_m,
                precision=precision, tomo=tomo, snr=snr, ssc_chi=ssc_chi, n_sub=n_sub, bias=bias)


def listed():
    return [
        # the smallest survey (143 rows): what a unit test, a smoke run or the
        # inner loop of a tiny likelihood pays, launches and latency above all
        _step("step tiny fp64", 2, 5, 100.0, 1000.0, 64, 32, "fp64"),
        # three bins, distinct rows only (382), the S/N as a function of the
        # largest multipole in one call
        _step("step mid sorted lmax", 3, 7, 50.0, 2000.0, 96, 48, "bf16_auto", tomo="sorted", snr="lmax"),
        # the Euclid-like forecast, five bins (4550 rows), at the precision
        # that the benchmark uses
        _step("step euclid5 auto", 5, 10, 20.0, 3000.0, 256, 128, "bf16_auto"),
        # the same survey beyond the bin-centre and single-mode readings: the
        # line-of-sight super-sample term, 3 x 3 sub-bins, mass-dependent
        # bias, FP64 through the factorisation along chi
        _step("step euclid5 chi full", 5, 10, 20.0, 3000.0, 256, 128, "fp64_chi", snr="structured", ssc_chi=True,
              n_sub=3, bias=True),
        # the paper's own 14-bin binning with five bins (10000 rows), the
        # compensated bf16 product
        _step("step paper14 bf16x3", 5, 14, 10.0, 5000.0, 256, 128, "bf16x3"),
        # seven bins on the finest grid in plain FP64 (29463 rows of PAPER
        # tomography, S/N through the 12768 distinct ones)
        _step("step large7 fp64", 7, 15, 10.0, 5000.0, 512, 256, "fp64", snr="structured"),
        # ten bins on the finest grid, distinct rows (33165), the largest
        # matrix that is factored whole here
        _step("step large10 sorted", 10, 15, 10.0, 5000.0, 512, 256, "bf16_auto", tomo="sorted"),
        # S/N alone of a covariance at hand, results left on the device: an
        # MCMC step with a fixed covariance (818 rows)
        _step("snr2 paper14 z2", 2, 14, 10.0, 5000.0, 64, 32, "fp64", snr="noalloc", kind="snr2"),
        # the principal components of the paper's two-bin and three-bin
        # studies (818 and 2420 rows)
        _step("pca paper14 z2", 2, 14, 10.0, 5000.0, 64, 32, "fp64", kind="pca"),
        _step("pca paper14 z3", 3, 14, 10.0, 5000.0, 64, 32, "fp64", kind="pca"),
        # the integer mode and triangle counts of the Euclid-like binning
        dict(name="lattice euclid5", kind="lattice", n_ell=10, ell_min=20.0, ell_max=3000.0, f_sky=0.36),
        # four likelihood requests of different size that arrive together at
        # a server (2733 to 17059 rows), results fetched to the caller
        dict(name="serve burst of 4", kind="serve", requests="3:5000 5:1000 5:3000 7:1000", precision="bf16_auto",
             snr="structured", n_chi=256, n_m=128),
    ]


def _rows_of(case):
    """(rows of the vector, distinct rows, triangles) of a step-like case."""
    cen = _bins(case)[1]
    n_p = len(cen) * case["n_z"] * (case["n_z"] + 1) // 2
    n_b = n_r = 0
    tris = _triangles(cen)
    z = case["n_z"]
    sb = z * (z + 1) * (z + 2) // 6
    for i, j, k in tris:
        n_b += z ** 3 if i < j < k else sb if i == j == k else z * z * (z + 1) // 2
        n_r += sb
    paper = case["tomo"] == "paper"
    return n_p + (n_b if paper else n_r), n_p + n_r, len(tris)


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def log_real(lo, hi):
        return round(math.exp(rng.uniform(math.log(lo), math.log(hi))), 3)

    kind = rng.choice(["step"] * 6 + ["snr2", "pca", "lattice", "serve"])
    if kind == "lattice":
        return dict(kind=kind, n_ell=rng.randint(4, 12), ell_min=log_real(10, 100), ell_max=log_real(500, 3000),
                    f_sky=round(rng.uniform(0.05, 0.37), 4))
    if kind == "serve":
        picks = [(rng.choice([3, 5, 7]), rng.choice([1000, 3000, 5000])) for _ in range(rng.randint(2, 4))]
        picks = [(z, 1000 if z == 7 else m) for z, m in picks]
        return dict(kind=kind, requests=" ".join("%d:%d" % p for p in picks),
                    precision=rng.choice(["bf16_auto", "bf16x3", "fp64"]), snr=rng.choice(["structured", "direct"]),
                    n_chi=log_int(48, 256), n_m=log_int(24, 128))
    while True:
        c = _step("", rng.randint(1, 3 if kind == "pca" else 8), rng.randint(3, 15), log_real(10, 100),
                  log_real(800, 5000), log_int(32, 512), log_int(16, 256),
                  rng.choice(["fp64", "fp64_chi", "bf16_auto", "bf16x3", "bf16", "fp32"]),
                  tomo=rng.choice(["paper", "paper", "sorted"]), snr=rng.choice(["direct", "structured", "lmax"]),
                  ssc_chi=rng.random() < 0.25, n_sub=rng.choice([1, 1, 1, 2, 3]), bias=rng.random() < 0.3, kind=kind)
        del c["name"]
        n, n_r, _ = _rows_of(c)
        if c["tomo"] == "sorted" and c["snr"] == "structured":
            c["snr"] = "direct"
        if kind in ("snr2", "pca"):
            c.update(precision="fp64", ssc_chi=False, n_sub=1, bias=False, n_chi=min(64, c["n_chi"]),
                     n_m=min(32, c["n_m"]))
            c["snr"] = "noalloc" if kind == "snr2" and n <= 2200 else "direct"
        most = dict(step=30000, snr2=12000, pca=2450)[kind]
        unit = dict(fp64=1.0, fp32=0.5, bf16x3=0.1).get(c["precision"], 0.05)
        work = unit * n_r ** 2 * c["n_chi"] * c["n_m"] + n ** 3 / 3
        if 10 <= n <= most and work < 1.9e13:
            return c


# ------------------------------------------------------------------ inputs
def _bins(case):
    """Edges and centres of the log-spaced ell-bins (centre: the midpoint)."""
    a, b, n = math.log(case["ell_min"]), math.log(case["ell_max"]), case["n_ell"]
    e = [math.exp(a + i * (b - a) / n) for i in range(n + 1)]
    cen = [(e[i] + e[i + 1]) / 2.0 for i in range(n)]
    cut = case.get("ell_cut") or 0.0
    return e, [c for c in cen if c < cut] if cut > 0 else cen


def _triangles(cen):
    return [(i, j, k) for k in range(len(cen)) for i in range(k + 1) for j in range(i, k + 1) if cen[i] + cen[j] > cen[k]]


def _cumtrapz(y, x):
    return torch.cat([y.new_zeros(1), torch.cumsum(0.5 * (y[1:] + y[:-1]) * (x[1:] - x[:-1]), 0)])


def _interp(x, xp, fp):
    j = torch.searchsorted(xp, x, right=True).clamp(1, len(xp) - 1)
    t = ((x - xp[j - 1]) / (xp[j] - xp[j - 1])).clamp(0.0, 1.0)
    return fp[j - 1] + t * (fp[j] - fp[j - 1])


def _linspace(a, b, n):
    return torch.linspace(float(a), float(b), n, dtype=F64, device=DEV)


def _distance(om, n=20001):
    z = _linspace(0.0, 2.5, n)
    return z, _cumtrapz(1.0 / (H0 * torch.sqrt(om * (1 + z) ** 3 + 1 - om)), z)


def _shape(z):
    return (z / 0.64) ** 2 * torch.exp(-((z / 0.64) ** 1.5))


def _kernels(chi, om, n_z, nodes=2001):
    """Lensing kernels of n_z equipopulated source bins on the chi nodes."""
    zg = _linspace(0.001, 2.5, 20001)
    cdf = _cumtrapz(_shape(zg), zg)
    q = torch.arange(1, n_z, dtype=F64, device=DEV) / n_z
    edges = torch.cat([zg[:1], _interp(q, cdf / cdf[-1], zg), zg[-1:]])
    zt, ct = _distance(om)
    zc = _interp(chi, ct, zt)
    W = []
    for i in range(n_z):
        zs = _linspace(edges[i], edges[i + 1], nodes)
        w = torch.full_like(zs, float(zs[1] - zs[0]))
        w[0] *= 0.5
        w[-1] *= 0.5
        ni = _shape(zs) * w
        ni = ni / ni.sum()
        cs = _interp(zs, zt, ct)
        f = (1.0 - chi[:, None] / cs[None, :]).clamp_min(0.0) @ ni
        W.append(1.5 * om * H0 ** 2 * (1 + zc) * chi * f)
    return torch.stack(W)


def _scalars(seed):
    r = random.Random(seed)
    return dict(om=r.uniform(0.28, 0.32), s8=r.uniform(0.78, 0.86), f_sky=0.36 * r.uniform(0.97, 1.03),
                sigma_eps=0.3 * r.uniform(0.97, 1.03), n_gal=30.0 * r.uniform(0.97, 1.03))


def _tables(case, sc, grid_om=None):
    """(configuration, tables on the GPU) of a step-like case."""
    om, n_chi, n_m = sc["om"], case["n_chi"], case["n_m"]
    cfg = dict(n_z=case["n_z"], n_ell=case["n_ell"], n_chi=n_chi, n_k=N_K, n_m=n_m, ell_min=case["ell_min"],
               ell_max=case["ell_max"], ell_cut=case.get("ell_cut") or 0.0, f_sky=sc["f_sky"],
               sigma_eps=sc["sigma_eps"], n_gal_arcmin2=sc["n_gal"], sigma_b2=1e-4, k_max=50.0, rho_mean=om * RHO_CRIT)
    chi_max = float(_distance(grid_om or om)[1][-1])
    dchi = chi_max / n_chi
    chi = (torch.arange(n_chi, dtype=F64, device=DEV) + 0.5) * dchi
    theta = math.acos(1.0 - 2.0 * cfg["f_sky"])
    k = torch.exp(_linspace(math.log(min(0.5 * cfg["ell_min"] / chi_max, 0.02 / (chi_max * theta))), math.log(50.0), N_K))
    k[-1] = 50.0
    # linear growth, D(0) = 1, and sigma_8 in a top hat of 8 Mpc/h
    a = _linspace(1e-6, 1.0, 50001)
    e = torch.sqrt(om / a ** 3 + 1 - om)
    D = e * _cumtrapz(1.0 / (a * e) ** 3, a)
    zt, ct = _distance(om)
    D = _interp(1.0 / (1.0 + _interp(chi, ct, zt)), a, D / D[-1])
    kk = torch.exp(_linspace(math.log(1e-5), math.log(1e3), 100001))
    x = kk * 8.0
    win = torch.where(x < 1e-3, 1 - x * x / 10, 3 * (torch.sin(x) - x * torch.cos(x)) / x ** 3)
    s2 = float(_cumtrapz(kk ** 3 * kk / (1 + (kk / 0.02) ** 2) ** 1.4 * win ** 2 / (2 * math.pi ** 2), torch.log(kk))[-1])
    P = sc["s8"] ** 2 / s2 * (k / (1 + (k / 0.02) ** 2) ** 1.4)[None, :] * (D ** 2)[:, None]
    lnm = _linspace(math.log(1e11), math.log(1e16), n_m)
    m = torch.exp(lnm)
    w_m = m * float(lnm[1] - lnm[0])
    w_m[0] *= 0.5
    w_m[-1] *= 0.5
    rho = cfg["rho_mean"]
    nm = m ** -1.9 * torch.exp(-m / 1e14)
    nm = nm / (w_m * (m / rho) * nm).sum()
    r = (3 * m / (4 * math.pi * 200 * rho)) ** (1.0 / 3.0)
    u = torch.exp(-0.5 * (k[None, :] * r[:, None]) ** 2).clamp_min(1e-300)
    t = dict(chi=chi, w_chi=torch.full_like(chi, dchi), k=k, m=m, w_m=w_m, W=_kernels(chi, om, case["n_z"]), P=P.contiguous(),
             u=u.contiguous(), n_m=nm)
    if case.get("bias"):
        b1 = 0.7 + (m / 1e13) ** 0.45
        b1 = b1 / (w_m * (m / rho) * nm * b1).sum()
        t.update(b1=b1, b2=0.412 - 2.143 * b1 + 0.929 * b1 ** 2 + 0.008 * b1 ** 3)
    return cfg, t


def _serve_case(case, z=10, ell_max=0.0):
    return _step("", z, 15, 10.0, 5000.0, case["n_chi"], case["n_m"], case["precision"]) | {"ell_cut": float(ell_max)}


def _requests(case, seed):
    """The fiducial tables of a server and the requests against them."""
    sc = _scalars(seed) | {"om": 0.3, "s8": 0.8}
    cfg, fid = _tables(_serve_case(case), sc, grid_om=0.28)
    r = random.Random(seed + 1)
    reqs = []
    for word in case["requests"].split():
        z, ell_max = (int(x) for x in word.split(":"))
        om, s8 = r.uniform(0.28, 0.32), r.uniform(0.78, 0.86)
        reqs.append(dict(W=_kernels(fid["chi"], om, z).cpu().numpy(), n_z=z, ell_max=float(ell_max),
                         p_scale=(s8 / 0.8) ** 2, n_scale=om / 0.3, rho_mean=om * RHO_CRIT))
    return cfg, fid, reqs


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        cfg, fid, reqs = _requests(case, seed)
        arrays = {k: v for k, v in fid.items() if k != "W"}
        need = 2 << 30
        for q in reqs:  # each request's covariance, product, factor and S/N workspace, with room
            n, n_r, _ = _rows_of(_serve_case(case, q["n_z"], q["ell_max"]))
            k_len = case["n_chi"] * case["n_m"]
            need += 20 * n * n + 40 * n_r * n_r + 10 * n_r * k_len + (1 << 30)
        srv = serve.Server(cfg, arrays, int(need), max_inflight=4, precision=case["precision"], device=DEV)
        return dict(kind=kind, server=srv, requests=reqs, snr=case["snr"])
    if kind == "lattice":
        f = case["f_sky"] * random.Random(seed).uniform(0.99, 1.01)
        c = _step("", 2, case["n_ell"], case["ell_min"], case["ell_max"], 8, 4, "fp64")
        cfg, t = _tables(c, _scalars(seed) | {"f_sky": f})
        return dict(kind=kind, prob=wlcov.Problem(cfg, t, precision="fp64", device=DEV))
    sc = _scalars(seed)
    cfg, t = _tables(case, sc)
    prob = wlcov.Problem(cfg, t, precision=case["precision"], tomo=case["tomo"], device=DEV, ssc_chi=case["ssc_chi"],
                         n_sub=case["n_sub"])
    s = dict(kind=kind, prob=prob, snr=case["snr"])
    if kind in ("snr2", "pca"):  # a covariance and a data vector at hand
        x = _model(case, cfg, t)
        prob.d.copy_(x["d"])
        prob.C.copy_(x["C"])
        prob.row_exp2.copy_(x["t"])
    if case["snr"] == "noalloc":
        s["out"] = torch.zeros(1, dtype=F64, device=DEV)
        s["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    return s


# -------------------------------------------------------------------- runs
def _snr(s):
    p, how = s["prob"], s["snr"]
    if how == "direct":
        return p.snr2()
    if how == "structured":
        return p.snr2_structured()
    if how == "lmax":
        return p.snr2_lmax()
    p.snr2_noalloc(s["out"], s["status"])
    return dict(snr2=s["out"], status=s["status"])


def run(state):
    kind = state["kind"]
    if kind == "serve":
        srv = state["server"]
        tickets = [srv.submit(q["W"], q["n_z"], q["ell_max"], p_scale=q["p_scale"], n_scale=q["n_scale"],
                              rho_mean=q["rho_mean"], snr=state["snr"]) for q in state["requests"]]
        out = []
        for t in tickets:
            res, d, r, C, e = srv.fetch(t)
            srv.release(t)
            out.append(dict(d=d, r=r, C=C, t=e, snr2=res.snr2, status=res.status))
        return out
    p = state["prob"]
    if kind == "lattice":
        modes, tris = p.lattice_counts()
        return dict(modes=modes, tris=tris)
    if kind == "snr2":
        return dict(snr2=_snr(state))
    if kind == "pca":
        lam, snr, cum, _, _ = p.pca(vectors=False)
        return dict(lam=lam, snr=snr, cum=cum)
    p.run()
    return dict(d=p.d, r=p.r, C=p.C, t=p.row_exp2, snr2=_snr(state))


# -------------------------------------------------------------------- work
def _step_work(case):
    n, n_r, n_tri = _rows_of(case)
    el = 8 if case["precision"] in ("fp64", "fp64_chi") else 4
    n_cfg = len(_bins(case)[1]) + n_tri
    tables = 8.0 * (N_K * (case["n_chi"] + case["n_m"]) + case["n_chi"] * (case["n_z"] + 2))
    # the covariance written once and read once by the S/N; the one-halo term
    # summed over the masses per pair of configurations, then along chi; the
    # factorisation of the matrix that the S/N needs
    one_halo = float(n_r) * n_r * case["n_chi"] + float(n_cfg) * n_cfg * case["n_chi"] * case["n_m"]
    nf = n_r if case["snr"] == "structured" else n
    if case["kind"] == "snr2":
        return dict(bytes=el * n * (n + 1) / 2.0 + 12.0 * n, flops=n ** 3 / 3.0)
    if case["kind"] == "pca":
        return dict(bytes=el * n * (n + 1) / 2.0 + 36.0 * n, flops=n ** 3 / 3.0 + 4.0 / 3.0 * n ** 3)
    return dict(bytes=el * (float(n) * n + (n * (n + 1) / 2.0 if nf == n else n_r * (n_r + 1) / 2.0)) + 28.0 * n + tables,
                flops=one_halo + nf ** 3 / 3.0)


def work(case):
    if case["kind"] == "lattice":
        lf = 2 * math.pi / math.sqrt(4 * math.pi * case["f_sky"])
        e, cen = _bins(case)
        modes = [math.pi * ((e[b + 1] / lf) ** 2 - (e[b] / lf) ** 2) for b in range(len(cen))]
        # each mode of the shortest side once per triangle, with one interval
        # of partners per row of the second side's ring
        ops = sum(modes[i] / 8 * 4 * e[j + 1] / lf for i, j, k in _triangles(cen))
        return dict(bytes=8.0 * (len(cen) + 3 * len(_triangles(cen))), flops=ops)
    if case["kind"] == "serve":
        b = f = 0.0
        for word in case["requests"].split():
            z, m = (int(x) for x in word.split(":"))
            w = _step_work(_serve_case(case, z, m) | {"snr": case["snr"]})
            n = _rows_of(_serve_case(case, z, m))[0]
            b += w["bytes"] + 2.0 * n * n * (8 if case["precision"] == "fp64" else 4)  # fetched: read and written
            f += w["flops"]
        return dict(bytes=b, flops=f)
    return _step_work(case)


# ------------------------------------------------------------ 64-bit values
def _entries(case, e, cen):
    """Per configuration (kind, legs, [(sub-bin legs, weight)]), and the
    sub-bin centres: the bin centres, or the average over n_sub sub-bins."""
    S, out = max(1, case["n_sub"]), []
    sub = list(cen) if S == 1 else [e[b] + (s + 0.5) * (e[b + 1] - e[b]) / S for b in range(len(cen)) for s in range(S)]
    for b in range(len(cen)):
        w = [sub[b * S + s] for s in range(S)] if S > 1 else [1.0]
        out.append((2, (b, b), [((b * S + s,) * 2, x / sum(w)) for s, x in enumerate(w)]))
    x, gw = np.polynomial.legendre.leggauss(8)
    for tri in _triangles(cen):
        if S == 1:
            out.append((3, tri, [(tri, 1.0)]))
            continue
        cells = []
        h = [(e[b + 1] - e[b]) / S / 2 for b in tri]
        for s in product(range(S), repeat=3):
            g = tuple(b * S + q for b, q in zip(tri, s))
            l = [sub[q] for q in g]
            if not 2 * max(l) < sum(l):
                continue
            l1, l2 = l[0] + h[0] * x[:, None], l[1] + h[1] * x[None, :]
            cos = [np.clip(((l[2] + q * h[2]) ** 2 - l1 ** 2 - l2 ** 2) / (2 * l1 * l2), -1, 1) for q in (-1, 1)]
            pairs = float((gw[:, None] * gw[None, :] * h[0] * h[1] * l1 * l2 * 2 * (np.arccos(cos[0]) - np.arccos(cos[1]))).sum())
            if pairs > 0:
                cells.append((g, pairs))
        tot = sum(w for _, w in cells)
        out.append((3, tri, [(g, w / tot) for g, w in cells]))
    return out, sub


def _model(case, cfg, t, scale=None):
    """Data vector, response and scaled covariance in 64 bits: the halo-model
    spectra at k = ell / chi, their Limber projections, and Gaussian + one-halo
    + super-sample covariance, all with plain torch."""
    p_scale, n_scale, rho = scale or (1.0, 1.0, cfg["rho_mean"])
    e, cen = _bins(case)
    cfgs, sub = _entries(case, e, cen)
    nz, k_max = cfg["n_z"], cfg["k_max"]
    omega = 4 * math.pi * cfg["f_sky"]
    chi, w, k, W = t["chi"], t["w_chi"], t["k"], t["W"]
    P, nm = t["P"] * p_scale, t["n_m"] * n_scale
    mr = t["m"] / rho
    b1 = t.get("b1") if t.get("b1") is not None else torch.ones_like(mr)
    b2 = t.get("b2") if t.get("b2") is not None else torch.zeros_like(mr)
    # table values at ell / chi: linear in ln k, the slope from the nodes
    ell = torch.tensor(sub, dtype=F64, device=DEV)
    kk = ell[:, None] / chi[None, :]
    ok = kk <= k_max
    j = (torch.searchsorted(k, kk.clamp(max=k_max), right=True) - 1).clamp(0, N_K - 2)
    lk = torch.log(k)
    f = (torch.log(kk) - lk[j]) / (lk[j + 1] - lk[j])
    lu, lp = torch.log(t["u"]).T.contiguous(), torch.log(P)
    U = torch.exp((1 - f)[..., None] * lu[j] + f[..., None] * lu[j + 1]) * ok[..., None]
    n_at = torch.arange(len(chi), device=DEV)[None, :]
    Pk = torch.exp((1 - f) * lp[n_at, j] + f * lp[n_at, j + 1]) * ok
    lo, hi = torch.arange(N_K, device=DEV).sub(1).clamp_min(0), torch.arange(N_K, device=DEV).add(1).clamp_max(N_K - 1)
    slope = (lp[:, hi] - lp[:, lo]) / (lk[hi] - lk[lo])
    ne = (1 - f) * slope[n_at, j] + f * slope[n_at, j + 1]
    wm = t["w_m"] * nm
    R_lin = 47.0 / 21.0 * Pk - ne * Pk / 3.0

    def halo(mu, bias, legs):
        x = wm * mr ** mu * bias
        for q in legs:
            x = x * U[q]
        return x.sum(-1)

    one = torch.ones_like(mr)
    I11 = [halo(1, b1, [q]) for q in range(len(sub))]
    I2 = {}

    def pair(beta, a, b):
        key = (beta, min(a, b), max(a, b))
        if key not in I2:
            I2[key] = halo(2, b1 if beta == 1 else b2, [a, b])
        return I2[key]

    X, R, G = [], [], []
    sm = torch.sqrt(wm)
    for kind, _, cells in cfgs:
        xs, rs, gs = 0.0, 0.0, 0.0
        for g, wt in cells:
            on = (kk[list(set(g))].amax(0) <= k_max).to(F64)
            if kind == 2:
                q = g[0]
                x = halo(2, one, [q, q]) + I11[q] ** 2 * Pk[q]
                r = I11[q] ** 2 * R_lin[q] + pair(1, q, q)
            else:
                x, r = halo(3, one, g), halo(3, b1, g)
                bpt = bg2 = dil = 0.0
                for a in range(3):
                    q, s, v = g[a], g[(a + 1) % 3], g[(a + 2) % 3]
                    x = x + I11[q] * pair(1, s, v) * Pk[q]
                    r = r + I11[q] * pair(2, s, v) * Pk[q] + I11[q] * pair(1, s, v) * R_lin[q]
                    ki, kj, kl = sub[q], sub[s], sub[v]
                    mu = (kl * kl - ki * ki - kj * kj) / (2 * ki * kj)
                    F = 5.0 / 7.0 + 0.5 * mu * (ki / kj + kj / ki) + 2.0 / 7.0 * mu * mu
                    pp = Pk[q] * Pk[s]
                    bpt, bg2, dil = bpt + 2 * F * pp, bg2 + 2 * (mu * mu - 1) * pp, dil + 2 * F * pp * (ne[q] + ne[s])
                I3 = I11[g[0]] * I11[g[1]] * I11[g[2]]
                x = x + I3 * bpt
                r = r + I3 * (433.0 / 126.0 * bpt + 5.0 / 126.0 * bg2 - dil / 3.0)
            y = sm * mr ** kind
            for q in g:
                y = y * U[q]
            xs, rs, gs = xs + wt * x * on, rs + wt * r * on, gs + wt * y * on[:, None]
        X.append(xs)
        R.append(rs)
        G.append(gs)
    X, R, G = torch.stack(X), torch.stack(R), torch.stack(G)
    n_ell, n_cfg = len(cen), len(cfgs)
    # the one-halo term over the masses for each pair of configurations
    H = torch.bmm(G.permute(1, 0, 2).contiguous(), G.permute(1, 2, 0).contiguous()).permute(1, 2, 0) / omega
    if case["ssc_chi"]:
        eps = torch.exp(_linspace(float(lk[0]), float(lk[-1]), N_EPS))
        eps[0], eps[-1] = k[0], k[-1]
        hl = float(lk[-1] - lk[0]) / (N_EPS - 1)
        we = torch.full_like(eps, hl)
        we[0] *= 0.5
        we[-1] *= 0.5
        je = (torch.searchsorted(k, eps, right=True) - 1).clamp(0, N_K - 2)
        fe = (torch.log(eps) - lk[je]) / (lk[je + 1] - lk[je])
        Pe = torch.exp((1 - fe) * lp[:, je] + fe * lp[:, je + 1])
        x = eps[None, :] * chi[:, None] * math.acos(1.0 - 2.0 * cfg["f_sky"])
        sw = 2.0 / math.pi * (we * eps ** 2 * (torch.special.bessel_j1(x) / x) ** 2 * Pe).sum(1)
        H = H + (chi ** 2 * sw)[None, None, :] * R[:, None, :] * R[None, :, :]
    # distinct rows: bins in increasing order, ell-bins then triangles
    zp = torch.tensor([(a, b) for a in range(nz) for b in range(a, nz)], device=DEV)
    zb = torch.tensor([(a, b, c) for a in range(nz) for b in range(a, nz) for c in range(b, nz)], device=DEV)
    Wp, Wb = W[zp].prod(1), W[zb].prod(1)
    dP, dB = (X[:n_ell] * w * chi ** -2.0) @ Wp.T, (X[n_ell:] * w * chi ** -4.0) @ Wb.T
    rP, rB = (R[:n_ell] * w * chi ** -2.0) @ Wp.T, (R[n_ell:] * w * chi ** -4.0) @ Wb.T
    dR, rR = torch.cat([dP.reshape(-1), dB.reshape(-1)]), torch.cat([rP.reshape(-1), rB.reshape(-1)])
    sp, sb, n_tri = len(zp), len(zb), n_cfg - n_ell
    Tp, Tb = torch.sqrt(w) * chi ** -3.0 * Wp, torch.sqrt(w) * chi ** -5.0 * Wb
    M = torch.empty((len(dR), len(dR)), dtype=F64, device=DEV)
    groups = [(0, n_ell, sp, 0, Tp)] + ([(n_ell, n_tri, sb, n_ell * sp, Tb)] if n_tri else [])
    for c0, nc, s, o, T in groups:
        for c in range(nc):
            rows = slice(o + c * s, o + (c + 1) * s)
            for d0, nd, s2, o2, T2 in groups:
                A = H[c0 + c, d0:d0 + nd, None, :] * T2[None]  # [nd][s2][chi]
                M[rows, o2:o2 + nd * s2] = T @ A.reshape(nd * s2, -1).T
    # the rows of the data vector and their distinct rows
    at = {tuple(z): i for i, z in enumerate(zb.tolist())}
    zrow, owner, dist = [], [], []
    for c in range(n_ell):
        for i, z in enumerate(zp.tolist()):
            zrow.append((z[0], z[1], -1)), owner.append(c), dist.append(c * sp + i)
    for c in range(n_ell, n_cfg):
        i, jj, q = cfgs[c][1]
        for z in product(range(nz), repeat=3):
            if case["tomo"] == "sorted":
                keep = z[0] <= z[1] <= z[2]
            else:
                keep = (i != jj or z[0] <= z[1]) and (jj != q or z[1] <= z[2])
            if keep:
                zrow.append(z), owner.append(c), dist.append(n_ell * sp + (c - n_ell) * sb + at[tuple(sorted(z))])
    zrow = torch.tensor(zrow, device=DEV)
    dist_t = torch.tensor(dist, device=DEV)
    d, r = dR[dist_t], rR[dist_t]
    sorted_rows = len(dist) == len(dR) and dist == list(range(len(dR)))
    C = M if sorted_rows else M[dist_t][:, dist_t]
    if not case["ssc_chi"]:
        for a in range(0, len(d), 4096):
            C[a:a + 4096] += cfg["sigma_b2"] * r[a:a + 4096, None] * r[None, :]
    # Gaussian term, block by block
    noise = cfg["sigma_eps"] ** 2 / (cfg["n_gal_arcmin2"] * (10800.0 / math.pi) ** 2 / nz)
    Ps = torch.zeros((n_ell, nz, nz), dtype=F64, device=DEV)
    Ps[:, zp[:, 0], zp[:, 1]] = dP
    Ps[:, zp[:, 1], zp[:, 0]] = dP
    Ps += noise * torch.eye(nz, dtype=F64, device=DEV)
    ends = np.cumsum(np.bincount(owner, minlength=n_cfg))
    for c, (kind, legs, _) in enumerate(cfgs):
        a, b = (0 if c == 0 else int(ends[c - 1])), int(ends[c])
        z = zrow[a:b]
        if kind == 2:
            Q = Ps[c]
            g = Q[z[:, 0]][:, z[:, 0]] * Q[z[:, 1]][:, z[:, 1]] + Q[z[:, 0]][:, z[:, 1]] * Q[z[:, 1]][:, z[:, 0]]
            C[a:b, a:b] += g / (2 * cen[c] * (e[c + 1] - e[c]) * cfg["f_sky"])
            continue
        l = [cen[q] for q in legs]
        lam2 = 2 * (l[0] * l[1]) ** 2 + 2 * (l[0] * l[2]) ** 2 + 2 * (l[1] * l[2]) ** 2 - l[0] ** 4 - l[1] ** 4 - l[2] ** 4
        vol = l[0] * l[1] * l[2]
        for q in legs:
            vol *= e[q + 1] - e[q]
        ntri = omega ** 2 * vol / (2 * math.pi ** 3 * math.sqrt(lam2))
        for s in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
            if all(legs[s[q]] == legs[q] for q in range(3)):
                g = omega / ntri
                for q in range(3):
                    g = g * Ps[legs[q]][z[:, q]][:, z[:, s[q]]]
                C[a:b, a:b] += g
    ex = np.frexp(C.diagonal().cpu().numpy())[1]
    tt = -((ex - 1) // 2)
    sc = torch.from_numpy(np.ldexp(1.0, tt)).to(DEV)
    for a in range(0, len(d), 4096):
        C[a:a + 4096] *= sc[a:a + 4096, None] * sc[None, :]
    last = torch.tensor([max(cfgs[c][1]) for c in owner], device=DEV)
    return dict(d=d, r=r, C=C, t=torch.from_numpy(tt.astype(np.int32)).to(DEV), ds=d * sc, last=last)


MOST_SNR = 12000  # rows up to which plain torch factors the matrix in seconds


def _exact_snr(x, how):
    if len(x["d"]) > MOST_SNR:
        return None
    C, ds = x["C"], x["ds"]
    if how == "lmax":
        order = torch.argsort(x["last"], stable=True)
        C, ds = C[order][:, order], ds[order]
    y = torch.linalg.solve_triangular(torch.linalg.cholesky(C), ds[:, None], upper=False)[:, 0]
    if how != "lmax":
        return float((y * y).sum())
    cum = torch.cumsum(y * y, 0)
    ends = torch.bincount(x["last"]).cumsum(0)
    return cum[ends - 1].cpu().numpy()


def _exact_pca(x):
    """Eigenvalues over many decades and the S/N of each mode: one-sided
    Jacobi on the graded Cholesky factor, all pairs of a round together."""
    n = len(x["d"])
    if n > 1000:
        return None
    L = torch.linalg.cholesky(x["C"])
    y = torch.linalg.solve_triangular(L, x["ds"][:, None], upper=False)[:, 0]
    # C_true = A A^T with A = 2^-t L; orthogonal rows after the rotations
    A = L / torch.from_numpy(np.ldexp(1.0, x["t"].cpu().numpy())).to(DEV)[:, None]
    m = n + n % 2
    if m > n:
        A = torch.cat([A, A.new_zeros(1, n)])
    ids = torch.arange(m, device=DEV)
    for _ in range(30):
        worst = torch.zeros((), dtype=F64, device=DEV)
        for _ in range(m - 1):
            p, q = ids[:m // 2], ids[m // 2:].flip(0)
            a, b = A[p], A[q]
            aa, bb, ab = (a * a).sum(1), (b * b).sum(1), (a * b).sum(1)
            live = ab.abs() > 1e-17 * torch.sqrt(aa * bb)
            worst = torch.maximum(worst, (ab.abs() / torch.sqrt(aa * bb).clamp_min(1e-300)).max())
            tau = (bb - aa) / (2 * torch.where(live, ab, torch.ones_like(ab)))
            tn = torch.where(tau >= 0, 1.0, -1.0) / (tau.abs() + torch.sqrt(1 + tau * tau))
            tn = torch.where(live, tn, torch.zeros_like(tn))
            cs = 1 / torch.sqrt(1 + tn * tn)
            sn = cs * tn
            A[p], A[q] = cs[:, None] * a - sn[:, None] * b, sn[:, None] * a + cs[:, None] * b
            ids = torch.cat([ids[:1], ids[-1:], ids[1:-1]])
        if float(worst) < 1e-15 * n:
            break
    # now A = J^T 2^-t L and A A^T = diag(lambda); S_a . d = (A y)_a, since d = 2^-t L y
    lam = (A * A).sum(1)
    keep = torch.argsort(lam)[m - n:]
    lam, proj = lam[keep], (A @ y)[keep]
    return lam, proj


def exact(case, seed):
    kind = case["kind"]
    if kind == "lattice":
        return None
    if kind == "serve":
        cfg, fid, reqs = _requests(case, seed)
        out = []
        for q in reqs:
            c = _serve_case(case, q["n_z"], q["ell_max"])
            t = fid | {"W": torch.from_numpy(q["W"]).to(DEV)}
            x = _model(c, cfg | {"n_z": q["n_z"]}, t, (q["p_scale"], q["n_scale"], q["rho_mean"]))
            out.append(dict(d=x["d"], r=x["r"], C=x["C"], t=x["t"], snr2=_exact_snr(x, "direct"), status=0))
        return out
    x = _model(case, *_tables(case, _scalars(seed)))
    if kind == "snr2":
        v = _exact_snr(x, "direct")
        if case["snr"] == "noalloc":
            return dict(snr2=dict(snr2=torch.tensor([v], dtype=F64, device=DEV), status=None))
        return dict(snr2=v)
    if kind == "pca":
        got = _exact_pca(x)
        if got is None:
            return None
        lam, proj = got
        s = proj ** 2 / lam
        return dict(lam=lam, snr=s, cum=torch.cumsum(torch.sort(s, descending=True)[0], 0))
    return dict(d=x["d"], r=x["r"], C=x["C"], t=x["t"], snr2=_exact_snr(x, case["snr"]))
