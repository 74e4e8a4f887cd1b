"""Several time steps per launch (2D TMz and TEz) without a plane wave, against the
per-step kernels from a random state: total-field boxes that do not exist (incident
tables of 0, 1 and 2 entries) under regions that hold design and absorber nodes, and
TEz boxes that reach the walls.
TMz in FP64 to the last bit, TEz in FP64 to 1e-11 (the bar against the oracle);
FP32 1e-4 on F and the state, 1e-3 on the gradient."""
import numpy as np
import pytest

import fdtd_workloads as W
from test_gpu_multi2d import solve
from test_gpu_parity_2d import gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu


def both_paths(gpu, w, exact):
    nf = 5 if w.get("pol_axis") == "x" else 4
    rho = W.seeded_rho(w, 5)
    nx, ny = w["n"][:2]
    state = np.random.default_rng(3).standard_normal((nf, 1, ny, nx))
    h = slice(1, 3) if nf == 4 else slice(2, 3)
    state[h] *= 2.6e-3
    state[3:] *= 1e5
    F0, s0, g0 = solve(gpu, w, rho, state, True, 0)
    F1, s1, g1 = solve(gpu, w, rho, state, False, 0)
    assert F0 > 0 and np.abs(g0).max() > 0
    if exact:
        assert F1 == F0 and np.array_equal(s1, s0) and np.array_equal(g1, g0)
        return
    tf, tg = (1e-11, 1e-11) if w["precision"] == 64 else (1e-4, 1e-3)
    assert abs(F1 - F0) <= tf * abs(F0)
    assert np.linalg.norm(s1 - s0) <= tf * np.linalg.norm(s0)
    assert np.linalg.norm(g1 - g0) <= tg * np.linalg.norm(g0)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("te", [False, True])
@pytest.mark.parametrize("ny,margin,entries", [(28, 13, 0), (27, 12, 1), (28, 12, 2), (28, 5, 16)])
def test_no_plane_wave_needs_no_incident_tables(gpu, prec, te, ny, margin, entries):
    nx, pml = 120, 3
    assert ny - 1 - 2 * (pml + margin) + 5 == entries
    mk = W.tiny_te if te else W.tiny2d
    w = mk(precision=prec, n=(nx, ny, 1), pml_cells=pml, tfsf_margin=margin, source="none", weights="unit",
           n_steps=37, design_lo=(pml + 1, pml + 1, 0), design_n=(nx - 2 * pml - 4, ny - 2 * pml - 4, 1),
           gap_lo=(55, 12, 0), gap_n=(2, 2, 1), pml_kappa_max=2.0)
    say(f"[multi2d] no plane wave, {'TEz' if te else 'TMz'} fp{prec} {nx}x{ny} margin {margin}")
    both_paths(gpu, w, prec == 64 and not te)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("nx,ny,gap", [(40, 37, (0, 12)), (40, 37, (37, 34)), (130, 70, (60, 0)), (130, 70, (60, 30))])
def test_te_design_and_gap_up_to_the_walls(gpu, prec, nx, ny, gap):
    """TEz without an absorber and without a plane wave: the design box may reach the
    PEC walls, and the gap too.  Their edges on the walls keep E = 0 (and the
    current they were given) and have no gradient."""
    w = W.tiny_te(precision=prec, n=(nx, ny, 1), pml_cells=0, tfsf_margin=0, source="none", weights="unit", n_steps=43,
                  design_lo=(0, 0, 0), design_n=(nx - 1, ny - 1, 1), gap_lo=gap + (0,), gap_n=(2, 2, 1))
    say(f"[multi2d] TEz design up to the walls fp{prec} {nx}x{ny} gap {gap}")
    both_paths(gpu, w, False)
