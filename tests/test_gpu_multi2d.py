"""Several time steps per launch (2D TMz and TEz) against the per-step kernels at
the sizes where the regions can go wrong: grids smaller than a region, one node
around the multiples of the stored widths of each region shape, no absorber,
step counts that leave a shorter last launch, boxes at the edge of what is
allowed, a gap too large for the staged adjoint source.  Both paths start from
a random state with the plane wave on.  TMz in FP64: F, the final state and
the gradient to the last bit (both kernels write out the roundings of a node's
update); TEz in FP64 to 1e-11, the bar against the oracle.  FP32: 1e-4 on F and the state, 1e-3 on the gradient, the bars of
this precision against the oracle."""
import os

import numpy as np
import pytest

import fdtd_workloads as W
from test_gpu_parity_2d import gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu


def solve(gpu, w, rho, state, per_step, ckpt):
    old = os.environ.pop("FDTD_TEMPORAL_BLOCKING", None)
    if per_step:
        os.environ["FDTD_TEMPORAL_BLOCKING"] = "0"
    try:
        g = gpu.FDTD(w, ckpt_every=ckpt)
    finally:
        os.environ.pop("FDTD_TEMPORAL_BLOCKING", None)
        if old is not None:
            os.environ["FDTD_TEMPORAL_BLOCKING"] = old
    g.set_state(state)
    g.set_density(rho.astype(g.dtype))
    F = g.forward()
    s = g.get_state()
    g.adjoint()
    grad = g.gradient()
    g.close()
    return F, s, grad


# (nx, ny, pml, design box, gap box, steps, checkpoint interval)
CASES = [
    (30, 32, 3, 6, 2, 23, 0),       # smaller than one region
    (44, 24, 0, 5, 1, 21, 0),       # one stored width, walls without an absorber
    (45, 25, 2, 4, 3, 20, 7),       # one node more
    (89, 133, 6, 30, 20, 31, 10),   # a gap of 400 nodes (adjoint source not staged)
    (383, 385, 12, 90, 3, 17, 0),   # 48 x 16 stored nodes
    (481, 520, 16, 200, 5, 26, 0),  # 40 x 40 (FP32), 48 x 16 on several rounds (FP64)
    (700, 661, 20, 300, 7, 23, 9),  # 44 x 44
    (1801, 1700, 32, 700, 5, 11, 0),  # the large-grid regions
]


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("nx,ny,pml,box,gap,steps,ckpt", CASES)
def test_multi_step_matches_per_step(gpu, prec, nx, ny, pml, box, gap, steps, ckpt):
    m = 3
    lo = ((nx - box) // 2, pml + m + 2, 0)  # against the injection line
    glo = (nx // 2, lo[1] + box // 2, 0) if gap < box else (lo[0], lo[1], 0)
    glo = tuple(min(a, n - 2 - pml - m - gap - 1) for a, n in zip(glo[:2], (nx, ny))) + (0,)
    w = W.tiny2d(precision=prec, n=(nx, ny, 1), pml_cells=pml, tfsf_margin=m, n_steps=steps, t0_over_tau=0.2,
                 design_lo=lo, design_n=(box, box, 1), gap_lo=glo, gap_n=(gap, gap, 1), pml_kappa_max=2.0)
    rho = W.seeded_rho(w, 5)
    state = np.random.default_rng(3).standard_normal((4, 1, ny, nx))
    state[1:3] *= 2.6e-3
    state[3] *= 1e5
    say(f"[multi2d] {nx}x{ny} fp{prec} steps={steps} ckpt={ckpt}")
    F0, s0, g0 = solve(gpu, w, rho, state, True, ckpt)
    F1, s1, g1 = solve(gpu, w, rho, state, False, ckpt)
    assert F0 > 0 and np.abs(g0).max() > 0
    if prec == 64:
        assert F1 == F0
        assert np.array_equal(s1, s0)
        assert np.array_equal(g1, g0)
    else:
        assert abs(F1 - F0) <= 1e-4 * F0
        assert np.linalg.norm(s1 - s0) <= 1e-4 * np.linalg.norm(s0)
        assert np.linalg.norm(g1 - g0) <= 1e-3 * np.linalg.norm(g0)


# (nx, ny, pml, design cells, gap cells, steps)
TE_CASES = [
    (30, 32, 3, 6, 2, 23),        # smaller than one region
    (44, 24, 0, 5, 1, 21),        # one stored width, walls without an absorber
    (45, 25, 2, 4, 3, 20),        # one node more
    (89, 133, 6, 30, 20, 31),     # a gap of 840 edges (adjoint source not staged)
    (385, 400, 12, 90, 3, 17),    # 48 x 16 stored nodes on several rounds
    (901, 1000, 20, 300, 7, 13),  # the large-grid regions
]


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("nx,ny,pml,box,gap,steps", TE_CASES)
def test_te_multi_step_matches_per_step(gpu, prec, nx, ny, pml, box, gap, steps):
    m = 3
    lo = ((nx - box) // 2, pml + m + 1, 0)  # its lower edges next to the injection line
    glo = (nx // 2, lo[1] + box // 2, 0) if gap < box else lo
    glo = tuple(min(a, n - 2 - pml - m - gap - 1) for a, n in zip(glo[:2], (nx, ny))) + (0,)
    w = W.tiny_te(precision=prec, n=(nx, ny, 1), pml_cells=pml, tfsf_margin=m, n_steps=steps, t0_over_tau=0.2,
                  design_lo=lo, design_n=(box, box, 1), gap_lo=glo, gap_n=(gap, gap, 1), pml_kappa_max=2.0)
    rho = W.seeded_rho(w, 5)
    state = np.random.default_rng(3).standard_normal((5, 1, ny, nx))
    state[2] *= 2.6e-3
    state[3:] *= 1e5
    say(f"[multi2d] TEz {nx}x{ny} fp{prec} steps={steps}")
    F0, s0, g0 = solve(gpu, w, rho, state, True, 0)
    F1, s1, g1 = solve(gpu, w, rho, state, False, 0)
    assert F0 > 0 and np.abs(g0).max() > 0
    tf, tg = (1e-11, 1e-11) if prec == 64 else (1e-4, 1e-3)
    assert abs(F1 - F0) <= tf * abs(F0)
    assert np.linalg.norm(s1 - s0) <= tf * np.linalg.norm(s0)
    assert np.linalg.norm(g1 - g0) <= tg * np.linalg.norm(g0)
