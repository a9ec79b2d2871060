"""Start fields from the network's coarse grid: cells that take the kernel with
staged tiles, narrow ones that gather, in value and in time."""

import ctypes
import time

import pytest

import test_gpu_nn_wide as wide
from test_gpu_nn import P, env  # noqa: F401

pytestmark = pytest.mark.gpu


# whole and partial tiles of 64 x 4 x 4; flat and thin cells, with and without
# enough voxels in their tiles
@pytest.mark.parametrize("coarse,fine", [((32, 32, 32), (64, 64, 64)), ((16, 40, 64), (33, 70, 130)),
                                         ((64, 64, 64), (66, 129, 127)), ((64, 64, 8), (150, 150, 20)),
                                         ((64, 64, 8), (150, 150, 30)), ((8, 64, 64), (2, 300, 200)),
                                         ((64, 8, 64), (300, 1, 200)), ((64, 8, 8), (5000, 1, 1))], ids=str)
def test_temperature(env, coarse, fine):  # noqa: F811
    wide.test_temperature_from_coarse_grid(env, coarse, fine)


@pytest.mark.parametrize("narrow,coarse", [((100000, 1, 1), (64, 8, 8)), ((1, 100000, 1), (8, 64, 8)), ((300, 300, 1), (64, 64, 8))],
                         ids=str)
def test_narrow_cells_take_no_longer(env, narrow, coarse):  # noqa: F811
    """At most one and a half times a call on 100000 voxels of 50 x 40 x 50."""
    L, torch = env
    best = []
    for fine, co in ((narrow, coarse), ((50, 40, 50), (64, 48, 64))):
        pred = torch.zeros((co[0] * co[1] * co[2], 16), device="cuda")
        T = torch.empty(fine, device="cuda")
        scratch = torch.empty(2048, dtype=torch.int32, device="cuda")
        bad = ctypes.c_longlong()
        t = 1e9
        for _ in range(60):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            assert L.mrtlbm_nn_to_temperature(P(pred), 16, *co, *fine, 10.0, 0.05, P(T), P(scratch), ctypes.byref(bad), None) == 0
            t = min(t, time.perf_counter() - t0)
        best.append(t)
    assert best[0] < 1.5 * best[1], best
