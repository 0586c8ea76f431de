"""Tables of very many chi nodes, so that one wavefront or workgroup for each node
passes the 2^32 threads that a launch can hold (and, at fewer, 65535 workgroups
along y).  All nodes but the last 64 lie before the first source (their lensing
kernels are zero), so that every result is that of the 64 nodes alone; sums of FP64
products in another order, 1e-12."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def wl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_07437_amd import wlcov
    return wlcov


def _tables(n_chi):
    t = synth.make_tables("tiny", n_z=1, n_ell=1, ell_min=100.0, ell_max=300.0, n_chi=64, n_m=2, n_k=3)
    a = {k: v for k, v in t.arrays().items() if v is not None}
    before = n_chi - 64
    a["chi"] = np.r_[np.linspace(0.9, 1.0, before, endpoint=False) * a["chi"][0], a["chi"]]
    a["w_chi"] = np.r_[np.ones(before), a["w_chi"]]
    a["W"] = np.c_[np.zeros((1, before)), a["W"]]
    a["P"] = np.r_[np.broadcast_to(a["P"][:1], (before, 3)), a["P"]]
    return dict(t.cfg, n_chi=n_chi), a


def _run(wl, n_chi, n_sub, ssc_chi):
    cfg, a = _tables(n_chi)
    prob = wl.Problem(cfg, a, precision="fp64_chi", n_sub=n_sub, ssc_chi=ssc_chi)
    prob.run()
    torch.cuda.synchronize()
    out = [prob.d.cpu().numpy(), prob.r.cpu().numpy(), prob.covariance_true(), prob.snr2()]
    if ssc_chi:
        out.append(prob.sigma_w2()[-64:].cpu().numpy())
    prob.close()
    torch.cuda.empty_cache()
    return out


@pytest.mark.parametrize("n_chi,n_sub,ssc_chi", [(64 * 9000, 0, False), (64 * 132000, 8, True)])
def test_many_nodes(wl, n_chi, n_sub, ssc_chi):
    print("case many nodes n_chi = %d" % n_chi, flush=True)
    for got, want in zip(_run(wl, n_chi, n_sub, ssc_chi), _run(wl, 64, n_sub, ssc_chi)):
        assert np.max(np.abs(got / want - 1.0)) < 1e-12
