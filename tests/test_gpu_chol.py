"""The bordered Cholesky of wlc_snr2 at the edges of its tiles: 16-row tiles,
128-column panels, a ragged last panel of odd and even width, one panel only,
and a size past the one up to which every panel updates the whole trailing
matrix.

The matrix is M = 1.5 I + V V^T with four columns in V, so that d^T M^-1 d is
a 4 x 4 solve (Sherman-Morrison-Woodbury).  Cholesky solves with a backward
error of at most (3 n + 1) eps |M| (Higham, Accuracy and Stability of Numerical
Algorithms, theorem 10.4), hence the tolerance (3 n + 8) eps kappa(M).
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# (n_data, n_z, n_ell, ell_min, ell_max, tomography)
SHAPES = [(2, 1, 1, 10.0, 500.0, "paper"), (16, 3, 1, 10.0, 500.0, "paper"), (17, 1, 4, 50.0, 500.0, "paper"),
          (33, 1, 5, 100.0, 500.0, "paper"), (64, 2, 4, 10.0, 500.0, "paper"), (111, 1, 12, 10.0, 1000.0, "paper"),
          (127, 1, 13, 10.0, 2000.0, "paper"), (128, 1, 8, 400.0, 500.0, "paper"), (143, 2, 5, 50.0, 500.0, "paper"),
          (144, 1, 14, 10.0, 5000.0, "paper"), (193, 2, 7, 400.0, 5000.0, "sorted"),
          (240, 2, 8, 50.0, 1000.0, "sorted"), (255, 5, 3, 10.0, 500.0, "sorted"), (383, 2, 9, 10.0, 500.0, "paper"),
          (10217, 3, 17, 400.0, 5000.0, "paper")]


@pytest.fixture(scope="module")
def wl():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1812_07437_amd import wlcov
    return wlcov


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: str(s[0]))
def test_snr2_tile_edges(wl, shape):
    import torch
    n, n_z, n_ell, lo, hi, tomo = shape
    print("case cholesky tile edges n = %d" % n, flush=True)
    cfg = dict(synth.PRESETS["tiny"], **synth.SURVEY_DEFAULTS, rho_mean=8.3e10)
    cfg.update(n_z=n_z, n_ell=n_ell, ell_min=lo, ell_max=hi, n_chi=8, n_m=4)
    prob = wl.Problem(cfg, synth.make_tables("tiny").arrays(), precision="fp64", tomo=tomo)
    assert prob.sizes.n_data == n
    rng = np.random.default_rng(n)
    V = rng.standard_normal((n, 4)) / np.sqrt(n)
    d = rng.standard_normal(n)
    e = rng.integers(-30, 30, n)
    kappa = 1.0 + np.linalg.norm(V, 2) ** 2 / 1.5
    tol = (3 * n + 8) * np.finfo(float).eps * kappa

    def want(keep):
        v, x = V[keep], d[keep]
        return float(x @ x / 1.5 - (x @ v) @ np.linalg.solve(np.eye(4) + v.T @ v / 1.5, v.T @ x) / 2.25)

    s = torch.from_numpy(np.ldexp(1.0, e)).cuda()
    Vg = torch.from_numpy(V).cuda()
    M = Vg @ Vg.T
    M.diagonal().add_(1.5)
    M.mul_(s[:, None]).mul_(s[None, :])
    prob.row_exp2.copy_(torch.from_numpy(e.astype(np.int32)))
    prob.d.copy_(torch.from_numpy(d))
    prob.C.copy_(M)
    every = np.arange(n)
    assert abs(prob.snr2() / want(every) - 1) < tol
    # a datum of infinite variance counts for nothing
    at = n // 2
    prob.C.copy_(M)
    prob.C[at, at] = float("inf")
    assert abs(prob.snr2() / want(every[every != at]) - 1) < tol
    # a pivot that is not positive, or not a number, at the first and the last
    # row and at the last row of the first tile and of the first panel
    for at in sorted({0, min(15, n - 1), min(127, n - 1), n - 1}):
        for bad in (-1.0, 0.0, float("nan")):
            prob.C.copy_(M)
            prob.C[at, at] = bad
            with pytest.raises(wl.WlcError) as ex:
                prob.snr2()
            assert ex.value.code == wl.WLC_ENOTPD
    prob.close()
