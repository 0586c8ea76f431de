"""Small products and their slices, on the exact integer factors of
test_gpu_gram_exact: every residue mod 3 and both parities of k-blocks, slices
cut short, the largest number of slices, and either side of 64 tiles."""
import numpy as np
import pytest

import test_gpu_gram_exact as exact
from test_gpu_gram_exact import case, wl  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [
    (256, 512),    # one tile, one slice of 16 k-blocks
    (200, 8192),   # four slices of 64 (1 mod 3, even), padding rows
    (256, 9216),   # four of 72 (0 mod 3)
    (256, 10400),  # four of 82 (1 mod 3), the last 80
    (512, 4672),   # 3 tiles: two slices of 73 (odd)
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
