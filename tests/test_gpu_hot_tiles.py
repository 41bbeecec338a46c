"""Hot-area counts at the edges of the 32 x 32 labelling tiles against the
oracle: counts are integers and must be equal."""
import numpy as np
import pytest
import torch

from oracle import diagnostics as D

pytestmark = pytest.mark.gpu


def _masks(n, rng):
    y, x = np.mgrid[0:n, 0:n]
    yield "empty", np.zeros((n, n), bool)
    yield "full", np.ones((n, n), bool)
    yield "checkerboard", (x + y) % 2 == 0
    yield "rows", y % 2 == 0
    yield "columns", x % 2 == 0
    # one path that turns at alternating ends of every second row
    snake = (y % 2 == 0) | ((y % 4 == 1) & (x == n - 1)) | ((y % 4 == 3) & (x == 0))
    yield "snake", snake
    yield "snake, transposed", snake.T.copy()
    for density in (0.45, 0.59, 0.75):
        yield f"random {density}", rng.random((n, n)) < density


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 97, 160])
def test_counts_at_tile_edges(n):
    from paper_2306_15678_amd.march import hot_areas_static

    for name, mask in _masks(n, np.random.default_rng(n)):
        w = torch.from_numpy(mask.astype(np.float64)).cuda()
        for periodic in (False, True):
            got = hot_areas_static(w, 0.5, periodic)
            want = D.hot_area_count(mask.astype(np.float64), 0.5, periodic=periodic)
            assert got == want, (n, name, periodic, got, want)
