"""Parity of the principal component analysis (Sec. 6) between the HIP path
(one-sided block Jacobi on FP64 MFMA, through the C ABI) and the oracle
(LAPACK's Jacobi SVD), on the same covariance definitions."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def wl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_07437_amd import wlcov
    return wlcov


_REF = {}


def _ref(preset, tomo):
    if (preset, tomo) not in _REF:
        t = synth.make_tables(preset)
        o = oracle.Oracle(t, tomo=tomo)
        r = o.run()
        _REF[(preset, tomo)] = (t, r, oracle.Oracle.pca(r["C"], r["d"]))
    return _REF[(preset, tomo)]


@pytest.mark.parametrize("precision", ["fp64", "fp64_chi"])
@pytest.mark.parametrize("preset,tomo", [("tiny", "paper"), ("tiny", "sorted"), ("mid", "paper")])
def test_pca_parity(wl, preset, tomo, precision):
    """Eigenvalues over all decades to 1e-9 relative, the cumulative curve to
    1e-9 of the total, and the eigenvectors of well-separated modes."""
    _say("case pca %s %s %s" % (precision, preset, tomo))
    t, r, (lam0, snr0, cum0, S0) = _ref(preset, tomo)
    prob = wl.Problem(t.cfg, t.arrays(), precision=precision, tomo=tomo)
    prob.run()
    snr2 = prob.snr2()
    lam, snr, cum, sweeps, S = prob.pca()
    torch.cuda.synchronize()
    _say("  sweeps %d, lambda %.3e .. %.3e" % (sweeps, lam[0], lam[-1]))
    err = np.max(np.abs(lam / lam0 - 1.0))
    _say("  lambda max rel %.3e" % err)
    assert err < 1e-9
    assert np.max(np.abs(cum - cum0)) < 1e-9 * cum0[-1]
    assert abs(cum[-1] - snr2) < 1e-10 * snr2
    # modes whose eigenvalue is separated from its neighbours by > 1e-3
    gap = np.minimum(np.r_[np.inf, lam0[1:] / lam0[:-1] - 1], np.r_[lam0[1:] / lam0[:-1] - 1, np.inf])
    sep = gap > 1e-3
    assert np.count_nonzero(sep) > 0.5 * len(lam0)
    assert np.max(np.abs(snr[sep] - snr0[sep])) < 1e-8 * cum0[-1]
    Sg = S.cpu().numpy()
    assert np.max(np.abs(Sg[sep] - S0[sep])) < 1e-7
    prob.close()


def test_pca_mixed(wl):
    """bf16x3 covariance: the cumulative curve within 1e-4 of the FP64 one."""
    _say("case pca bf16x3 mid")
    t, r, (lam0, snr0, cum0, S0) = _ref("mid", "paper")
    prob = wl.Problem(t.cfg, t.arrays(), precision="bf16x3")
    prob.run()
    lam, snr, cum, sweeps, _ = prob.pca(vectors=False)
    assert np.max(np.abs(cum - cum0)) < 1e-4 * cum0[-1]
    prob.close()


def test_pca_euclid5_properties(wl):
    """Euclid-like size (N = 4550): the sum rule against the Cholesky S/N,
    ascending positive eigenvalues, orthonormal eigenvectors, and the
    reconstruction of sampled covariance entries."""
    _say("case pca fp64 euclid5")
    t = synth.make_tables("euclid5")
    prob = wl.Problem(t.cfg, t.arrays(), precision="fp64")
    prob.run()
    snr2 = prob.snr2()
    lam, snr, cum, sweeps, S = prob.pca()
    torch.cuda.synchronize()
    _say("  sweeps %d, lambda %.3e .. %.3e, (S/N)^2 %.6e vs %.6e" % (sweeps, lam[0], lam[-1], cum[-1], snr2))
    assert abs(cum[-1] - snr2) < 1e-9 * snr2
    assert np.all(lam > 0) and np.all(np.diff(lam) >= 0)
    G = S @ S.T
    assert torch.max(torch.abs(G - torch.eye(len(lam), dtype=G.dtype, device=G.device))).item() < 1e-10
    pairs = synth.sample_pairs(len(lam), 200, seed=3)
    a = torch.as_tensor(pairs[:, 0], device=S.device)
    b = torch.as_tensor(pairs[:, 1], device=S.device)
    L = torch.as_tensor(lam, device=S.device)
    rec = torch.sum(S[:, a] * S[:, b] * L[:, None], dim=0)
    te = prob.row_exp2.long()
    Ct = prob.C[a, b].double() * torch.exp2(-(te[a] + te[b]).double())
    sc = torch.sqrt(prob.C[a, a].double() * torch.exp2(-2.0 * te[a].double()) *
                    prob.C[b, b].double() * torch.exp2(-2.0 * te[b].double()))
    assert torch.max(torch.abs(rec - Ct) / sc).item() < 1e-9
    prob.close()


@pytest.mark.parametrize("n_z", [1, 2])
def test_pca_paper_binning(wl, n_z):
    """The paper's 14 ell-bins over 10-5000 with one and two redshift bins
    (N = 144 and 818): eigenvalues against the oracle, and the number of
    modes holding 99 % of (S/N)^2 the same on both sides unless the oracle's
    own cumulative curve sits within 1e-8 of that threshold."""
    _say("case pca paper binning n_z=%d" % n_z)
    t = synth.make_tables("paper14", n_z=n_z)
    r = oracle.Oracle(t).run()
    lam0, snr0, cum0 = oracle.Oracle.pca(r["C"], r["d"], vectors=False)
    prob = wl.Problem(t.cfg, t.arrays(), precision="fp64")
    prob.run()
    lam, snr, cum, sweeps, _ = prob.pca(vectors=False)
    torch.cuda.synchronize()
    err = np.max(np.abs(lam / lam0 - 1.0))
    _say("  N %d, sweeps %d, lambda max rel %.3e" % (len(lam), sweeps, err))
    assert len(lam) == {1: 144, 2: 818}[n_z]
    assert err < 1e-9
    assert np.max(np.abs(cum - cum0)) < 1e-9 * cum0[-1]
    thr = 0.99 * cum0[-1]
    k0 = int(np.searchsorted(cum0, thr) + 1)
    k = int(np.searchsorted(cum, 0.99 * cum[-1]) + 1)
    near = np.min(np.abs(cum0[max(0, k0 - 2):k0 + 1] - thr)) < 1e-8 * cum0[-1]
    assert k == k0 or near
    prob.close()


# (n_data, n_z, n_ell, ell_min, ell_max): less than one block of 32, one pair of
# blocks exactly and not, one row more than a pair, odd and even numbers of
# 64-column chunks, and one column slice against several
@pytest.mark.parametrize("shape", [(2, 1, 1, 10.0, 500.0), (17, 1, 4, 50.0, 500.0), (64, 2, 4, 10.0, 500.0),
                                   (65, 2, 3, 200.0, 500.0), (128, 1, 8, 400.0, 500.0), (143, 2, 5, 50.0, 500.0),
                                   (383, 2, 9, 10.0, 500.0)], ids=lambda s: str(s[0]))
def test_pca_block_edges(wl, shape):
    """A graded covariance Delta M Delta, M = 1.5 I + V V^T with four columns in
    V and Delta over 20 decades, in no order: Jacobi on the Cholesky factor
    finds every eigenvalue to a modest multiple of n eps kappa(M) (Demmel and
    Veselic 1992, theorem 3.1 and section 4), here 40 n eps kappa(M); the
    cumulative curve ends at d^T C^-1 d, a 4 x 4 solve."""
    n, n_z, n_ell, lo, hi = shape
    _say("case pca block edges n = %d" % n)
    cfg = dict(synth.PRESETS["tiny"], **synth.SURVEY_DEFAULTS, rho_mean=8.3e10)
    cfg.update(n_z=n_z, n_ell=n_ell, ell_min=lo, ell_max=hi, n_chi=8, n_m=4)
    prob = wl.Problem(cfg, synth.make_tables("tiny").arrays(), precision="fp64")
    assert prob.sizes.n_data == n
    rng = np.random.default_rng(n)
    V = rng.standard_normal((n, 4)) / np.sqrt(n)
    M = V @ V.T + 1.5 * np.eye(n)
    kappa = 1.0 + np.linalg.norm(V, 2) ** 2 / 1.5
    e = rng.integers(-33, 34, n).astype(np.int32)  # C_true = 2^-e M 2^-e
    z = rng.standard_normal(n)
    d = np.ldexp(z, -e)
    prob.C.copy_(torch.from_numpy(M))
    prob.row_exp2.copy_(torch.from_numpy(e))
    prob.d.copy_(torch.from_numpy(d))
    lam, snr, cum, sweeps, S = prob.pca()
    lam0, snr0, cum0, S0 = oracle.Oracle.pca(np.ldexp(M, -(e[:, None] + e[None, :])), d)
    tol = 40 * n * np.finfo(float).eps * kappa
    assert np.max(np.abs(lam / lam0 - 1.0)) < 2 * tol  # both sides
    want = float(z @ z / 1.5 - (z @ V) @ np.linalg.solve(np.eye(4) + V.T @ V / 1.5, V.T @ z) / 2.25)
    assert abs(cum[-1] / want - 1.0) < tol
    Sg = S.cpu().numpy()
    assert np.max(np.abs(Sg @ Sg.T - np.eye(n))) < tol
    assert np.all(Sg[np.arange(n), np.argmax(np.abs(Sg), axis=1)] > 0)
    # a diagonal that is not a number has no place in the order of the rows:
    # refused, like any matrix that is not positive definite
    for bad in (float("nan"), 0.0, -1.0):
        prob.C.copy_(torch.from_numpy(M))
        prob.C[n // 2, n // 2] = bad
        with pytest.raises(wl.WlcError) as ex:
            prob.pca(vectors=False)
        assert ex.value.code == wl.WLC_ENOTPD
    prob.close()
