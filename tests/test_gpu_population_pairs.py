"""Two steps per pass of population storage: bit for bit the same as single
steps, which a caller-set block shape selects, and on the oracle."""

import numpy as np
import pytest

from oracle import ADIABATIC, PERIODIC, Oracle
from test_gpu_two_steps import A, ORACLE_SIDES, P, WALLS, _media, api  # noqa: F401

pytestmark = pytest.mark.gpu

# nx around the vector and wave widths (4 FP32 / 2 FP64 nodes per thread, 64
# lanes), ny and nz off the tiles' and chunks' ends, the smallest ny and nz
SHAPES = [(4, 500, 400), (5, 300, 301), (13, 211, 200), (75, 61, 87), (128, 65, 129), (129, 120, 63), (64, 640, 33),
          (127, 3, 900), (250, 2, 1900), (120, 2000, 2), (256, 200, 15), (96, 96, 96)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pairs_equal_single_steps(api, shape, prec):  # noqa: F811
    """11 steps for every mix of walls, from a state whose populations are not
    those of any moments."""
    import torch

    m, T0 = _media(shape, sum(shape))
    T0 = torch.from_numpy(T0).cuda()
    for axis, sides in WALLS:
        state = []
        for single in (True, False):
            g = api.Medium(m.phase, m.k, precision=prec, storage="populations")
            if single:
                g.set_launch(*g.info()["launch"])
            g.set_bc(axis, 0.8, -0.4, sides).init(T0, flux=True)
            s = g.state_get()
            gen = torch.Generator(device="cuda").manual_seed(axis)
            s *= 1 + 0.2 * torch.rand(s.shape, generator=gen, device="cuda", dtype=s.dtype)
            g.state_set(s)
            g.step(11)
            state.append(g.state_get())
        assert torch.equal(state[0], state[1]), (axis, sides)


def test_pairs_match_oracle(api):  # noqa: F811
    """FP64 cell large enough for the rule to take pairs: 20 steps within 1e-12
    of the oracle."""
    m, T0 = _media((90, 100, 120), 3)
    for axis, sides in ((0, (P, A, P)), (2, (P, P, P))):
        g = api.Medium(m.phase, m.k, precision="f64", storage="populations")
        g.set_bc(axis, 0.8, -0.4, sides).init(T0).step(20)
        o = Oracle(m.phase, m.k)
        o.set_bc(axis, 0.8, -0.4, [ORACLE_SIDES[s] for s in sides])
        o.init(T0)
        o.step(20)
        to = o.temperature()
        assert np.abs(g.temperature().cpu().numpy() - to).max() < 1e-12 * np.abs(to).max()
