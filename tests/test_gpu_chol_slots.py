"""The bordered Cholesky on both sides of the sizes at which one more panel, or two,
can wait in the scratch (from 1009 rows three instead of one, from 1521 five, from
2033 seven, from 2545 eight): the matrix, the reference and the tolerance of the
tile edges."""
import pytest

import test_gpu_chol as chol
from test_gpu_chol import wl  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(1000, 2, 16, 10.0, 500.0, "sorted"), (1012, 3, 7, 200.0, 1500.0, "paper"),
          (1520, 4, 8, 200.0, 1500.0, "sorted"), (1521, 2, 15, 20.0, 700.0, "paper"),
          (2032, 2, 14, 50.0, 500.0, "paper"), (2034, 2, 18, 10.0, 700.0, "paper"),
          (2544, 8, 4, 200.0, 500.0, "sorted"), (2547, 3, 9, 100.0, 500.0, "paper")]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: str(s[0]))
def test_snr2_panel_slots(wl, shape):
    chol.test_snr2_tile_edges(wl, shape)
