"""The density filter on boxes that are short along an axis (a tile as short as the box,
halo and taps inside it) and on boxes with more tiles than a grid has room for,
against the CPU reference, with the tolerances of the other routes."""
import numpy as np
import pytest

import test_gpu_filter_routes as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("shape,radius", [
    ((1, 40000), 2.5), ((2, 9001), 3.0), ((3, 5000), 7.5), ((20000, 1), 2.5), ((9001, 2), 1.5), ((5, 7000), 16.0),
    ((1, 3), 16.0), ((2, 2), 4.0), ((2, 300, 40), 2.5), ((3, 40, 300), 4.0), ((300, 2, 40), 2.5), ((40, 300, 2), 3.5),
    ((60, 1, 50), 2.5), ((60, 50, 1), 2.5), ((9, 2, 3), 4.0), ((2, 200, 700), 2.5), ((700, 3, 100), 3.0)])
def test_thin_boxes(prec, shape, radius):
    R.test_filter_routes(prec, shape, radius)


def test_a_row_with_more_tiles_than_a_grid():
    """2^27 + 5 cells in a row (2^32 threads in square tiles): far from the ends the
    filter of a periodic density is periodic."""
    import torch
    from paper_2203_01462_amd import design
    n = (1 << 27) + 5
    f = design.Filter((1, n), 2.5, torch.float32)
    pat = torch.tensor(np.random.default_rng(4).random(64), dtype=torch.float32)
    x = pat.cuda().repeat(n // 64 + 1)[:n].reshape(1, n)
    y = f.apply(x, 1.0)
    small = design.Filter((1, 64 * 9), 2.5, torch.float32)
    want = small.apply(pat.cuda().repeat(9).reshape(1, -1), 1.0)[0, 256:320]
    body = y[0, 256:n - 261].reshape(-1, 64)
    assert torch.equal(body.amax(0), want) and torch.equal(body.amin(0), want)
    f.close()
    small.close()
