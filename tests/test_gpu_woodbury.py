"""Edges of the S/N through the distinct rows, against the oracle: blocks of one
row, of a tile and more, the largest that is factored in LDS (120 rows at eight
redshift bins) and one that is not (165 at nine), with scalene, isosceles and
equilateral triangles among them."""
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


@pytest.mark.parametrize("n_z,n_ell,precision", [(1, 6, "fp64"), (2, 5, "fp64_chi"), (4, 5, "fp64"), (6, 3, "fp64"),
                                                 (7, 3, "fp64_chi"), (8, 2, "fp64"), (9, 2, "fp64_chi")])
def test_structured_block_sizes(wl, n_z, n_ell, precision):
    """FP64 on both sides, an identity without cancellation: 1e-10, as for the
    other sizes."""
    print("case structured n_z=%d n_ell=%d %s" % (n_z, n_ell, precision), flush=True)
    t = synth.make_tables("tiny", n_z=n_z, n_ell=n_ell, n_chi=48, n_m=16)
    ref = oracle.Oracle(t).run()
    prob = wl.Problem(t.cfg, t.arrays(), precision=precision)
    prob.run()
    assert abs(prob.snr2_structured() / ref["snr2"] - 1.0) < 1e-10
    assert abs(prob.snr2() / ref["snr2"] - 1.0) < 1e-10
    prob.close()
