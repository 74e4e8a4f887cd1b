"""3D steps in one launch (small grids) against the list and plain launches of the
same step, from a random state with the plane wave on: sizes around the 32 x 8
tiles, two and four planes a chunk with a remainder, a design that meets the
absorber's tiles and one that does not, no absorber, checkpoints.

Both schedules run the same node updates, so only the rounding of a compiled
expression could differ: FP64 1e-11 and FP32 1e-4 / 1e-3 (F and state / gradient),
the bars against the oracle."""
import numpy as np
import pytest

import fdtd_workloads as W
from test_gpu_multi2d import solve
from test_gpu_parity_2d import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import paper_2203_01462_amd as P
    return P


# (n, pml, margin, design lo, design n, gap lo, gap n, steps, checkpoint interval)
CASES = [
    ((24, 24, 28), 5, 2, (8, 8, 11), (8, 8, 6), (11, 11, 13), (2, 2, 2), 31, 0),
    ((33, 17, 23), 0, 3, (10, 6, 8), (9, 5, 4), (12, 8, 10), (1, 1, 1), 20, 0),
    ((70, 41, 37), 4, 3, (30, 15, 14), (12, 9, 7), (40, 18, 16), (3, 2, 2), 21, 8),
    ((112, 114, 110), 6, 3, (40, 50, 50), (20, 16, 6), (50, 56, 52), (2, 2, 2), 11, 0),
]


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n,pml,m,dlo,dn,glo,gn,steps,ckpt", CASES)
def test_one_launch_step_matches_lists(gpu, prec, n, pml, m, dlo, dn, glo, gn, steps, ckpt):
    w = W.tiny3d(precision=prec, n=n, pml_cells=pml, tfsf_margin=m, n_steps=steps, t0_over_tau=0.2, design_lo=dlo,
                 design_n=dn, gap_lo=glo, gap_n=gn, pml_kappa_max=2.0)
    rho = W.seeded_rho(w, 5)
    state = np.random.default_rng(3).standard_normal((9, n[2], n[1], n[0]))
    state[3:6] *= 2.6e-3
    state[6:] *= 1e5
    say(f"[whole3d] {n} fp{prec} steps={steps} ckpt={ckpt}")
    F0, s0, g0 = solve(gpu, w, rho, state, True, ckpt)
    F1, s1, g1 = solve(gpu, w, rho, state, False, ckpt)
    assert F0 > 0 and np.abs(g0).max() > 0
    tf, tg = (1e-11, 1e-11) if prec == 64 else (1e-4, 1e-3)
    assert abs(F1 - F0) <= tf * abs(F0)
    assert np.linalg.norm(s1 - s0) <= tf * np.linalg.norm(s0)
    assert np.linalg.norm(g1 - g0) <= tg * np.linalg.norm(g0)


# A design in the absorber's tiles: from about 1200 (FP64) and 3100 (FP32) chunks of
# 32 x 8 x 4 nodes the adjoint takes the lists and the forward one launch, from 4000
# the FP64 forward the lists too.
THIN = [
    ((40, 160, 164), 5, 3, (14, 60, 60), (12, 20, 22), (19, 70, 70), (2, 2, 2), 12, 0),
    ((24, 402, 322), 3, 2, (8, 200, 150), (8, 30, 30), (11, 212, 164), (2, 2, 2), 13, 5),
]


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n,pml,m,dlo,dn,glo,gn,steps,ckpt", THIN)
def test_thin_grid_mixes_the_two(gpu, prec, n, pml, m, dlo, dn, glo, gn, steps, ckpt):
    test_one_launch_step_matches_lists(gpu, prec, n, pml, m, dlo, dn, glo, gn, steps, ckpt)
