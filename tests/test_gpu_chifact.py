"""Edges of the product factorised along chi against the oracle: configurations
around the 32 of a block of H, chi nodes around its 8 and the 16 of a stage,
columns around 16, row blocks of one row, of several 16-tiles and past 64."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def wl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_07437_amd import wlcov
    return wlcov


@pytest.mark.parametrize("n_z,n_ell,n_chi,n_m,ngins", [
    (1, 3, 7, 15, False), (1, 10, 8, 16, False), (2, 7, 9, 17, False), (3, 8, 16, 31, True), (5, 3, 17, 33, False),
    (7, 2, 33, 4, True), (8, 2, 31, 16, False)])
def test_chifact_edges(wl, n_z, n_ell, n_chi, n_m, ngins):
    """FP64 sums of positive products on both sides: 1e-10, as elsewhere."""
    print("case chifact n_z=%d n_ell=%d n_chi=%d n_m=%d" % (n_z, n_ell, n_chi, n_m), flush=True)
    sys.stdout.flush()
    t = synth.make_tables("tiny", n_z=n_z, n_ell=n_ell, n_chi=n_chi, n_m=n_m, ell_min=10.0, ell_max=3000.0)
    want = oracle.Oracle(t, tomo="sorted").covariance(None, ngins, "rank1")
    prob = wl.Problem(t.cfg, t.arrays(), precision="fp64_chi", tomo="sorted", ngins=ngins)
    prob.run()
    C = prob.covariance_true()
    assert np.max(np.abs(C - want) / np.abs(want)) < 1e-10
    prob.close()
