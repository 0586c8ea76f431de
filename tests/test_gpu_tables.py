"""Edges of the table kernels (staging by wavefronts, list averages over the
masses, rows, the survey window) against the oracle, through the C ABI."""
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


def _rel(a, b):
    return np.max(np.abs(a - b) / np.abs(b))


# masses around one and two lanes' worth and past them, chi nodes around a
# wavefront, k tables around one and two rounds of 64 probes, lists of one, eight
# and 27 entries, with and without bias tables and the window's column
@pytest.mark.parametrize("n_m,n_chi,n_k,n_sub,bias,ssc", [
    (2, 3, 2, 1, False, "rank1"), (63, 4, 3, 2, True, "chi"), (64, 64, 65, 1, True, "rank1"),
    (65, 65, 66, 3, False, "chi"), (128, 17, 768, 3, True, "rank1"), (129, 63, 4097, 2, False, "rank1"),
    (200, 5, 4098, 1, True, "chi"), (250, 5, 64, 3, False, "rank1")])
def test_table_edges(wl, n_m, n_chi, n_k, n_sub, bias, ssc):
    """Sums of positive products and a few differences of the response, in
    FP64 on both sides: the 1e-10 of the other parity tests."""
    _say("case tables n_m=%d n_chi=%d n_k=%d n_sub=%d %s" % (n_m, n_chi, n_k, n_sub, ssc))
    t = synth.make_tables("tiny", n_m=n_m, n_chi=n_chi, n_k=n_k)
    if bias:
        t = synth.with_bias(t)
    o = oracle.Oracle(t, n_sub=n_sub)
    d, r = o.data_vector()
    want = o.covariance(None, False, ssc)
    for precision in ("fp64", "bf16_auto"):
        prob = wl.Problem(t.cfg, t.arrays(), precision=precision, n_sub=n_sub, ssc_chi=ssc == "chi")
        prob.run()
        torch.cuda.synchronize()
        assert _rel(prob.d.cpu().numpy(), d) < 1e-10
        assert _rel(prob.r.cpu().numpy(), r) < 1e-10
        C = prob.covariance_true()
        if precision == "fp64":
            assert _rel(C, want) < 1e-10
        else:  # its bound holds relative to the diagonal
            dg = np.sqrt(np.diag(want))
            assert np.max(np.abs(C - want) / np.outer(dg, dg)) < 1e-5
        prob.close()


@pytest.mark.parametrize("n_k", [2, 3, 4000, 4001])
def test_sigma_w2_table_lengths(wl, n_k):
    """Tables whose logarithms fit into LDS and not; every term of the sum is
    positive, 1e-12 as for the other tables."""
    _say("case sigma_w2 n_k=%d" % n_k)
    t = synth.make_tables("tiny", n_chi=5, n_k=n_k)
    want = oracle.Oracle(t).sigma_w2()
    prob = wl.Problem(t.cfg, t.arrays(), precision="fp64", ssc_chi=True)
    assert _rel(prob.sigma_w2().cpu().numpy(), want) < 1e-12
    prob.close()
