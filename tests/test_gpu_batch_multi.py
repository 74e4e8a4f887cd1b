"""FP64 batches with the depths left to the library: all instances advance several
steps per launch.  Each of the three region shapes that a batch can take, uneven
instances that are not square, a step count that no launch length divides; eager and
replayed, against single contexts bit for bit (FP64 rounds alike in all step kernels)."""
import numpy as np
import pytest

import fdtd_workloads as W
from test_gpu_batch import run_batch, singles
from test_gpu_parity_2d import gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu


def instance(nx, ny, k, steps):
    w = W.tiny2d(precision=64, n=(nx, ny, 1), n_steps=steps, pml_cells=(6, 0, 10)[k % 3], tfsf_margin=3, t0_over_tau=0.6, n_freq=2 + k % 3,
                 gamma_mult=1.0 + 2 * k, name=f"m{k}")
    d, g = 9 + k % 5, 1 + k % 3
    lo = (nx // 2 - 4 - k % 2, ny // 2 - 6)
    w.update(design_lo=(*lo, 0), design_n=(d, d + 1, 1), gap_lo=(lo[0] + 3, lo[1] + 4, 0), gap_n=(g, 2, 1))
    return w


# regions of 44 x 12 exact nodes with 2 rows a thread while 256 hold the batch, then of
# 48 x 16, beyond with 4 rows on 8 wavefronts
@pytest.mark.parametrize("sizes,rows", [
    ([(64, 57), (45, 130), (131, 44), (89, 97)], 2),
    ([(200, 150), (97, 301), (257, 129), (64, 300), (50, 330)], 2),
    ([(300, 210), (97, 401), (401, 129), (64, 700), (50, 45)], 4),
])
def test_several_steps_per_launch_matches_single_contexts(gpu, sizes, rows):  # noqa: F811
    ws = [instance(nx, ny, k, 1499) for k, (nx, ny) in enumerate(sizes)]
    rhos = [W.seeded_rho(w, k) for k, w in enumerate(ws)]
    ref = singles(gpu, ws, rhos)
    (eager,), r0, d0 = run_batch(gpu, ws, rhos, 0, False)
    graph, r1, d1 = run_batch(gpu, ws, rhos, 0, True, repeats=3)
    say(f"[batch-multi] {sizes}: rows {r0}, depths {d0}")
    assert r0 == r1 == [rows] * len(ws) and d0 == d1 == [2] * len(ws)
    for F, grads in [eager] + graph:
        for k in range(len(ws)):
            assert F[k] == ref[k][0] and F[k] > 0, k
            assert np.array_equal(grads[k], ref[k][1]) and np.abs(grads[k]).max() > 0, k
