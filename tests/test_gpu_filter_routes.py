"""The density filter's routes (all stages in one launch, a launch a stage on
small and large tiles, the plain kernels) against the CPU reference at the edges
of their tiles, out of place and in place, and the one-launch reductions beyond
one pass of their workgroups.

Tolerances.  FP64: 1e-12, the bar of the existing filter test (a few dozen
roundings per stage, values in [0, 1]).  FP32 stage outputs are rounded to 2^-24;
a stage with alpha = 1 passes an input error on with a factor of at most
((1 + alpha) / alpha)^2 = 4, so four stages give at most
2^-25 (1 + 4 + 16 + 64) = 2.5e-6, and the transpose's factors (e + alpha)^2 and
(u + alpha)^-2 four times twice that relative error: 1e-4 in the norm."""
import numpy as np
import pytest

from oracle import filter as OF

pytestmark = pytest.mark.gpu


# (shape, radius): one launch (stored tiles of 26, 20, 14 cells), tiles of 16 x 16
# and 32 x 32, of 8 x 8 x 4 and 16 x 8 x 8, plain
CASES = [((1, 1), 0.5), ((26, 27), 1.0), ((41, 40), 1.7), ((14, 43), 3.0), ((33, 16), 3.5), ((47, 70), 16.0),
         ((400, 411), 2.5), ((417, 329), 7.5), ((5, 9, 17), 2.5), ((4, 8, 8), 4.0), ((33, 65, 70), 1.5),
         ((7, 9, 10), 4.5)]


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("shape,radius", CASES)
def test_filter_routes(prec, shape, radius):
    import torch
    from paper_2203_01462_amd import design
    dt, alpha = (torch.float64 if prec == 64 else torch.float32), 1.0
    x = torch.tensor(np.random.default_rng(1).random(shape), dtype=dt)
    g = torch.tensor(np.random.default_rng(2).random(shape) - 0.5, dtype=dt)
    f = design.Filter(shape, radius, dt)
    xd, gd = x.cuda(), g.cuda()
    y, gt = f.apply(xd, alpha), f.transpose(gd)
    f.apply(xd, alpha, out=xd)
    f.transpose(gd, out=gd)
    yr, xs = OF.open_close(x.double().numpy(), radius, alpha)
    gr = OF.open_close_transpose(xs, g.double().numpy(), radius, alpha)
    ty, tg = (1e-12, 1e-12) if prec == 64 else (2.5e-6, 1e-4)
    assert np.abs(y.double().cpu().numpy() - yr).max() <= ty
    assert np.linalg.norm(gt.double().cpu().numpy() - gr) <= tg * np.linalg.norm(gr)
    assert torch.equal(xd, y) and torch.equal(gd, gt)
    f.close()


@pytest.mark.parametrize("n", [1, 1023, 1025, 262145, 1000003])
def test_reductions(n):
    """design.stats and the MMA sums against NumPy (FP64 sums of n terms in any
    order: relative 1e-12)."""
    import torch
    from paper_2203_01462_amd import design
    r = np.random.default_rng(n)
    x, g = r.random(n), r.standard_normal(n)
    xd, gd = torch.tensor(x).cuda(), torch.tensor(g).cuda()
    for _ in range(2):
        zeta, kkt = design.stats(xd, gd)
        assert abs(zeta - np.mean(4 * x * (1 - x))) <= 1e-12 * zeta
        assert abs(kkt - np.linalg.norm(x - np.clip(x - g, 0, 1))) <= 1e-12 * kkt
        m = design.MMA(n)
        assert abs(m.begin(xd, -1.0, gd) - 0.1 * np.abs(g).mean()) <= 1e-12
        xn = torch.empty_like(xd)
        approx, dist = m.solve(0.1, xn)
        gp, gm, L, U = np.maximum(g, 0), np.maximum(-g, 0), x - 0.5, x + 0.5
        p, q = 0.25 * (1.001 * gp + 0.001 * gm + 0.1), 0.25 * (0.001 * gp + 1.001 * gm + 0.1)
        z = xn.cpu().numpy()
        want = np.sum((z - x) * (p / ((U - z) * (U - x)) - q / ((z - L) * (x - L))))
        assert abs(approx + 1.0 - want) <= 1e-11 * max(1.0, abs(want))
        assert abs(dist - np.sum((U - L) * (z - x) ** 2 / ((U - z) * (z - L)))) <= 1e-11 * dist
        m.close()
