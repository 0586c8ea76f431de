"""Small products (a wavefront to a 32 x 32 block) and their slices, on the
exact integer factors of test_gpu_gram_exact: remainders of the blocks' k-blocks
in flight, slices of one k-block and empty ones, panel extents, the largest
number of slices, and either side of the line to the tile kernels (48 items)."""
import numpy as np
import pytest

import oracle
import synth
import test_gpu_gram_exact as exact
from test_gpu_gram_exact import case, ext_case, wl  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [
    (256, 512),    # one tile, one slice of 16 k-blocks
    (200, 8192),   # four slices of 64 (1 mod 3, even), padding rows
    (256, 9216),   # four of 72 (0 mod 3)
    (256, 10400),  # four of 82 (1 mod 3), the last 80
    (512, 4672),   # 3 tiles: two slices of 73 (odd)
    (2304, 1056),  # 45 tiles: one slice of 34
    (2560, 2048),  # 55 tiles: one slice
    (2561, 4096),  # 66 tiles: two slices of 64
]


@pytest.mark.parametrize("case", CASES, indirect=True, ids=["n%d_k%d" % c for c in CASES])
def test_slices_exact(wl, case):
    nt = case["n_pad"] // 256
    F = np.array([1.0 if I % 2 == 0 else 0.1 for I in range(nt)])
    G = exact._run(wl, case, "bf16_auto", panel_f=F, lim=0.5)
    exact._check_tiles(G, lambda I, J: case["split"] if F[I] * F[J] > 0.5 else case["hh"], case["n_pad"])
    # a product's workspace: the slices past the first
    assert wl.wlc_gram_ws_bytes("bf16_auto", case["n"], case["k"]) % (4 * case["n_pad"] ** 2) == 0


@pytest.mark.parametrize("ext_case", [(600, 2000), (1100, 2000), (768, 8320)], indirect=True,
                         ids=lambda c: "n%d_k%d" % c)
@pytest.mark.parametrize("precision", ["bf16", "bf16x3", "bf16_auto"])
def test_extents_exact(wl, ext_case, precision):
    nt = ext_case["n_pad"] // 256
    F = np.array([1.0 if I % 2 == 0 else 0.1 for I in range(nt)])
    split = {"bf16": lambda I, J: False, "bf16x3": lambda I, J: True, "bf16_auto": lambda I, J: F[I] * F[J] > 0.5}
    G = exact._run(wl, ext_case, precision, panel_f=F if precision == "bf16_auto" else None, lim=0.5)
    exact._check_tiles(G, lambda I, J: ext_case["split" if split[precision](I, J) else "hh"], ext_case["n_pad"])


# FP64 products of few rows: one block of 16 and one row past it, a row less and
# more than a block for each CU would hold, one to nine steps of k for a
# wavefront, then eight and three slices
@pytest.mark.parametrize("n_z,n_ell,ell_max,n_chi,n_m", [
    (1, 1, 500.0, 3, 2), (1, 4, 500.0, 5, 13), (2, 3, 500.0, 9, 64), (2, 11, 4000.0, 65, 9), (2, 12, 4000.0, 8, 8),
    (1, 2, 500.0, 128, 65), (2, 5, 1500.0, 64, 50)])
def test_f64_few_rows(wl, n_z, n_ell, ell_max, n_chi, n_m):
    """Sums of positive products, against the oracle to the 1e-10 of the other
    parity tests."""
    t = synth.make_tables("tiny", n_z=n_z, n_ell=n_ell, ell_max=ell_max, n_chi=n_chi, n_m=n_m)
    want = oracle.Oracle(t).covariance()
    prob = wl.Problem(t.cfg, t.arrays(), precision="fp64")
    exact._say("case f64 few rows n=%d k=%d" % (prob.sizes.n_data, n_chi * n_m))
    prob.run()
    exact.torch.cuda.synchronize()
    assert np.max(np.abs(prob.covariance_true() / want - 1.0)) < 1e-10
    prob.close()
