"""Slices of the split-K choice for products that do not fill the chip, on the
exact integer factors of test_gpu_gram_exact: the shortest slices (8 k-blocks),
every residue mod 3 and both parities, slices left empty by the rounding up,
the largest number of slices, and either side of 64 tiles."""
import numpy as np
import pytest

import test_gpu_gram_exact as exact
from test_gpu_gram_exact import case, wl  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [
    (256, 512),    # one tile, two slices of 8 k-blocks
    (200, 8192),   # 32 slices of 8 (2 mod 3, even), padding rows
    (256, 9216),   # 32 of 9 (0 mod 3, odd)
    (256, 10240),  # 32 of 10 (1 mod 3)
    (512, 4672),   # 3 tiles: 18 slices of 9 of 146 k-blocks, one short and one empty
    (2560, 2048),  # 55 tiles: four slices of 16
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
