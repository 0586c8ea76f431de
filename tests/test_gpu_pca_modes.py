"""The principal components mode by mode, on the graded covariance of
test_pca_block_edges, C = 2^-e M 2^-e with M = 1.5 I + V V^T."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

# (n_data, n_z, n_ell, ell_min, ell_max): within one pair of blocks of 32 rows,
# exactly one and one row more, and several
SHAPES = [(2, 1, 1, 10.0, 500.0), (17, 1, 4, 50.0, 500.0), (64, 2, 4, 10.0, 500.0), (65, 2, 3, 200.0, 500.0),
          (128, 1, 8, 400.0, 500.0), (143, 2, 5, 50.0, 500.0), (383, 2, 9, 10.0, 500.0)]


@pytest.fixture(scope="module")
def wl():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1812_07437_amd import wlcov
    return wlcov


def _problem(wl, shape):
    n, n_z, n_ell, lo, hi = shape
    cfg = dict(synth.PRESETS["tiny"], **synth.SURVEY_DEFAULTS, rho_mean=8.3e10)
    cfg.update(n_z=n_z, n_ell=n_ell, ell_min=lo, ell_max=hi, n_chi=8, n_m=4)
    prob = wl.Problem(cfg, synth.make_tables("tiny").arrays(), precision="fp64")
    assert prob.sizes.n_data == n
    rng = np.random.default_rng(n)
    V = rng.standard_normal((n, 4)) / np.sqrt(n)
    M = V @ V.T + 1.5 * np.eye(n)
    kappa = 1.0 + np.linalg.norm(V, 2) ** 2 / 1.5
    return prob, M, rng.standard_normal(n), kappa


def _pca(prob, M, e, z):
    import torch
    prob.C.copy_(torch.from_numpy(M))
    prob.row_exp2.copy_(torch.from_numpy(e.astype(np.int32)))
    prob.d.copy_(torch.from_numpy(np.ldexp(z, -e)))
    lam, snr, cum, sweeps, S = prob.pca()
    return lam, snr, cum, sweeps, S.cpu().numpy()


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: str(s[0]))
def test_pca_modes(wl, shape):
    """Rows spread evenly over 64 powers of two of scale, in no order: every mode
    against its own eigenvector, (S_a d)^2 / lambda_a, and against the
    oracle, eigenvector and S/N.  Eigenvalues to 40 n eps kappa(M) as in
    test_pca_block_edges; an eigenvector to that over the eigenvalue's relative
    distance from the others (Demmel and Veselic 1992, theorem 2.2 and section 4),
    and its S/N, a square, to twice that of d^T C^-1 d; both sides err."""
    n = shape[0]
    print("case pca modes n = %d" % n, flush=True)
    prob, M, z, kappa = _problem(wl, shape)
    rng = np.random.default_rng(n + 2)
    e = rng.permutation(np.arange(n) * 64 // n - 32)
    # within a power of two the rows differ by factors of up to 1.4
    f = 1.0 + 0.4 * rng.permutation(n) / n
    M = M * f[:, None] * f[None, :]
    lam, snr, cum, _, S = _pca(prob, M, e, z)
    prob.close()
    d = np.ldexp(z, -e)
    lam0, snr0, cum0, S0 = oracle.Oracle.pca(np.ldexp(M, -(e[:, None] + e[None, :])), d)
    tol = 40 * n * np.finfo(float).eps * kappa
    total = cum0[-1]
    own = (S @ d) ** 2 / lam
    assert np.max(np.abs(snr - own)) < 4 * tol * total
    assert np.max(np.abs(cum - np.cumsum(np.sort(snr)[::-1]))) < n * np.finfo(float).eps * total
    near = np.minimum(np.r_[np.inf, lam0[1:] / lam0[:-1] - 1], np.r_[lam0[1:] / lam0[:-1] - 1, np.inf])
    sep = near > 1e-3
    assert np.count_nonzero(sep) > n // 2
    bound = 2 * tol / np.minimum(near[sep], 1.0)
    # the largest entry's sign is the vector's: two of nearly one size may differ
    S, S0 = S[sep], S0[sep]
    S *= np.sign(np.sum(S * S0, axis=1))[:, None]
    assert np.all(np.max(np.abs(S - S0), axis=1) < bound)
    assert np.all(np.abs(snr[sep] - snr0[sep]) < 2 * bound * total)
