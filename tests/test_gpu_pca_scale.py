"""The principal components over the range of double precision: on the graded
covariance of test_pca_modes a common power of two in all rows changes no
rounding, so that the results at any scale are those at unit scale, to the last
bit."""
import numpy as np
import pytest

from test_gpu_pca_modes import SHAPES, _pca, _problem, wl  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


# shifts of the row exponents: variances of 2^-506 ... 2^-374, whose products
# are normal numbers; then of 2^-666 ... 2^-534 and 2^534 ... 2^666, whose
# products are not
@pytest.mark.parametrize("shift", [220, 300, -300])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: str(s[0]))
def test_pca_any_scale(wl, shape, shift):
    print("case pca scale n = %d, 2^%d" % (shape[0], -2 * shift), flush=True)
    prob, M, z, _ = _problem(wl, shape)
    e = np.random.default_rng(shape[0] + 1).integers(-33, 34, shape[0])
    lam0, snr0, cum0, sweeps0, S0 = _pca(prob, M, e, z)
    lam, snr, cum, sweeps, S = _pca(prob, M, e + shift, z)
    prob.close()
    assert sweeps == sweeps0
    assert np.array_equal(np.ldexp(lam, 2 * shift), lam0)
    assert np.array_equal(snr, snr0) and np.array_equal(cum, cum0)
    assert np.array_equal(S, S0)
