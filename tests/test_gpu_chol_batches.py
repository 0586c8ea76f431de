"""The bordered Cholesky where the room for solved panels changes (one, three,
five, seven and eight at 1024, 1536, 2048 and 2560 rows, so that column blocks
wait for one, three or four panels) and where a group of eight panels just
begins to be taken and is followed by single ones (6000 columns): the matrix,
the reference and the tolerance of the tile edges."""
import pytest

import test_gpu_chol as chol
from test_gpu_chol import wl  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(1019, 2, 15, 10.0, 2000.0, "paper"), (1025, 2, 15, 200.0, 5000.0, "sorted"),
          (1518, 3, 13, 10.0, 500.0, "sorted"), (1536, 2, 10, 200.0, 500.0, "paper"),
          (2050, 5, 6, 400.0, 500.0, "sorted"), (2563, 3, 10, 50.0, 500.0, "paper"),
          (6012, 8, 7, 50.0, 500.0, "sorted"), (7140, 8, 7, 10.0, 2000.0, "paper")]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: str(s[0]))
def test_snr2_panel_batches(wl, shape):
    chol.test_snr2_tile_edges(wl, shape)
