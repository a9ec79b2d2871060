"""Several time steps per launch (pairs over large cells, more over small
ones): bit for bit the same as single steps, which a caller-set block shape
selects, and on the oracle."""

import numpy as np
import pytest

import workloads as w
from oracle import ADIABATIC, PERIODIC, Oracle

pytestmark = pytest.mark.gpu

P, A = "periodic", "adiabatic"
ORACLE_SIDES = {P: PERIODIC, A: ADIABATIC}
# cells that take pairs: nx around the vector and wave widths (4 FP32 / 2 or 4
# FP64 nodes per thread, 64 lanes), ny and nz off the tiles' and chunks' ends,
# the smallest ny and nz; and one small cell that takes single steps
SHAPES = [(4, 700, 400), (5, 300, 301), (13, 211, 200), (75, 61, 87), (128, 129, 65), (129, 120, 63), (64, 640, 33),
          (250, 2, 1900), (256, 900, 7), (256, 2000, 2), (13, 9, 7)]
WALLS = [(0, (P, P, P)), (1, (A, P, P)), (2, (P, A, P)), (0, (P, A, A)), (2, (A, A, A))]


@pytest.fixture(scope="module")
def api():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("no HIP device")
    from paper_1503_08718_amd import solver

    return solver


def _media(shape, seed):
    m = w.random_medium(seed, *shape, 3)
    return m, np.random.default_rng(seed).uniform(-0.5, 1.5, m.phase.shape)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pairs_equal_single_steps(api, shape, prec):
    """11 steps (five pairs and one single step) for every mix of walls."""
    import torch

    m, T0 = _media(shape, sum(shape))
    T0 = torch.from_numpy(T0).cuda()
    for axis, sides in WALLS:
        state = []
        for single in (True, False):
            g = api.Medium(m.phase, m.k, precision=prec, storage="moments")
            if single:
                g.set_launch(*g.info()["launch"])
            g.set_bc(axis, 0.8, -0.4, sides).init(T0, flux=True)
            g.step(11)
            state.append(g.state_get())
        assert torch.equal(state[0], state[1]), (axis, sides)


@pytest.mark.parametrize("shape", [(128, 128, 40), (75, 61, 87), (250, 100, 60)], ids=lambda s: "x".join(map(str, s)))
def test_pairs_match_oracle(api, shape):
    """FP64 cells large enough for the rule to take pairs: 50 steps within
    1e-12 of the oracle; a solve whose block of steps is replayed as a graph
    equals the same number of plain steps bit for bit."""
    import torch

    m, T0 = _media(shape, 3)
    g = api.Medium(m.phase, m.k, precision="f64", storage="moments")
    g.set_bc(1, 0.8, -0.4, (A, P, P)).init(T0)
    g.step(50)
    o = Oracle(m.phase, m.k)
    o.set_bc(1, 0.8, -0.4, [ORACLE_SIDES[s] for s in (A, P, P)])
    o.init(T0)
    o.step(50)
    to = o.temperature()
    assert np.abs(g.temperature().cpu().numpy() - to).max() < 1e-12 * np.abs(to).max()
    for every in (2, 4, 6, 10):
        h = api.Medium(m.phase, m.k, precision="f64", storage="moments")
        h.set_bc(1, 0.8, -0.4, (A, P, P)).init(T0)
        h.solve(1e-30, "keff", 3 * every, check_every=every)
        g.init(T0)
        g.step(3 * every)
        assert torch.equal(g.state_get(), h.state_get()), every


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("axis,shapes", [
    (0, [(64, 96, 64), (48, 64, 96), (128, 64, 64), (4, 40, 30)]),
    (1, [(75, 61, 87), (64, 50, 64), (96, 96, 40)]),
    (2, [(200, 64, 31), (30, 64, 128), (13, 130, 200)]),
])
def test_batched_pairs_equal_single_steps(api, axis, shapes, prec):
    """Batches of aligned and ragged cells; the first cell starts two blocks
    ahead and leaves the table after one.  Every state equals the same cell
    stepped alone in single steps, bit for bit."""
    import torch

    cells, alone = [], []
    for i, shape in enumerate(shapes):
        m, T0 = _media(shape, i)
        for out in (cells, alone):
            g = api.Medium(m.phase, m.k, precision=prec, storage="moments")
            if out is alone:
                g.set_launch(*g.info()["launch"])
            g.set_bc(axis, 0.8, -0.4, (P, A, P) if i % 2 else (P, P, A)).init(T0, flux=True)
            out.append(g)
    cells[0].step(20)
    res, _ = api.batch_solve(cells, tol=1e-30, kind="keff", max_steps=30, check_every=10)
    for g, h, r in zip(cells, alone, res):
        h.step(30)
        assert r["steps"] == 30
        assert torch.equal(g.state_get(), h.state_get())


@pytest.mark.parametrize("prec,storage", [("f32", "moments"), ("f64", "moments"), ("f64", "populations")])
@pytest.mark.parametrize("shape", [(1, 9, 7), (5, 2, 3), (7, 16, 20), (16, 16, 16), (24, 40, 30), (32, 32, 32), (64, 9, 8)],
                         ids=lambda s: "x".join(map(str, s)))
def test_small_cells_equal_single_steps(api, shape, prec, storage):
    """Every mix of walls; step counts that end on full and on shorter
    launches; a solve's replayed graph against plain steps."""
    import torch

    m, T0 = _media(shape, sum(shape))
    for axis, sides in WALLS:
        g = api.Medium(m.phase, m.k, precision=prec, storage=storage)
        h = api.Medium(m.phase, m.k, precision=prec, storage=storage)
        h.set_launch(*h.info()["launch"])
        for steps in (2, 7, 13):
            for c in (g, h):
                c.set_bc(axis, 0.8, -0.4, sides).init(T0, flux=True)
                c.step(steps)
            assert torch.equal(g.state_get(), h.state_get()), (axis, sides, steps)
        g.init(T0, flux=True)
        g.solve(1e-30, "keff", 30, check_every=10)
        h.init(T0, flux=True).step(30)
        assert torch.equal(g.state_get(), h.state_get()), (axis, sides)
