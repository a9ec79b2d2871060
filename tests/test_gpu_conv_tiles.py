"""The convolution kernels that stage tiles in LDS against the general ones,
which take the same call when the outputs (or the scratch) are not aligned
for them, and against the FP64 reference."""

import numpy as np
import pytest

from oracle import conv as C
from test_gpu_nn import P, bf, circ_bits, env, pack_w, rel_l2  # noqa: F401

pytestmark = pytest.mark.gpu

# extents at, below and off the tiles' 8 x 8 x 4 (and 8 x 4 x 4, 8 x 4 x 2), the
# smallest ones, and launches large enough for every tile size
SHAPES = [
    # (n, D, H, W, circ)
    (1, 1, 1, 1, (True, True, True)),
    (2, 2, 3, 5, (False, True, True)),
    (1, 4, 8, 8, (True, False, False)),
    (3, 5, 9, 17, (False, True, True)),
    (1, 6, 10, 12, (False, False, False)),
    (2, 20, 33, 40, (False, True, True)),
    (4, 32, 40, 64, (True, True, True)),
]
CHANNELS = [(8, 16), (16, 16), (16, 32), (32, 16), (32, 48), (64, 32), (128, 64), (64, 128)]


def _id(s):
    return "x".join(map(str, s[:4]))


def _unaligned(torch, shape, dtype):
    """A tensor one element off every vector boundary."""
    return torch.zeros(int(np.prod(shape)) + 8, dtype=dtype, device="cuda")[1:1 + int(np.prod(shape))].view(shape)


def _inputs(torch, L, s, cin, cout, seed):
    n, D, H, W, _ = s
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((n, D, H, W, cin), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.zeros((cout, L.mrtlbm_nn_kpad(cin)), device="cuda")
    w[:, :27 * cin] = torch.randn((cout, 27 * cin), generator=g, device="cuda") * 0.2
    b = torch.randn(cout, generator=g, device="cuda")
    dy = torch.randn((n, D, H, W, cout), generator=g, device="cuda").to(torch.bfloat16)
    return x, w.to(torch.bfloat16), b, dy


@pytest.mark.parametrize("cin,cout", CHANNELS)
@pytest.mark.parametrize("s", SHAPES, ids=_id)
def test_forward_equals_general_kernel(env, s, cin, cout):  # noqa: F811
    """Bit for bit: the same products in the same order; BF16 and FP32
    outputs, with and without bias and ReLU."""
    L, torch = env
    n, D, H, W, circ = s
    x, w, b, _ = _inputs(torch, L, s, cin, cout, cin + cout)
    for dtype, relu, bias in ((torch.bfloat16, 1, b), (torch.float32, 0, b), (torch.bfloat16, 0, None)):
        f32 = dtype == torch.float32
        got = torch.empty((n * D * H * W, cout), dtype=dtype, device="cuda")
        ref = _unaligned(torch, got.shape, dtype)
        for o in (got, ref):
            assert L.mrtlbm_nn_conv3d_fwd(P(x), n, D, H, W, cin, P(w), P(bias) if bias is not None else None, cout,
                                          circ_bits(circ), relu, None if f32 else P(o), P(o) if f32 else None, None) == 0
        assert torch.equal(got, ref), (dtype, relu)


def _wgrad(L, torch, s, cin, cout, x, dy, aligned):
    n, D, H, W, circ = s
    nbytes = L.mrtlbm_nn_wgrad_scratch_bytes(n, D, H, W, cin, cout)
    scratch = torch.empty(nbytes // 4 + 8, dtype=torch.float32, device="cuda")
    dw = torch.full((cout, L.mrtlbm_nn_kpad(cin)), 7.0, device="cuda")
    db = torch.full((cout,), 7.0, device="cuda")
    sp = scratch if aligned else scratch[1:]
    assert L.mrtlbm_nn_conv3d_wgrad(P(x), P(dy), n, D, H, W, cin, cout, circ_bits(circ), P(sp), P(dw), P(db), None) == 0
    return dw, db


@pytest.mark.parametrize("cin,cout", CHANNELS)
@pytest.mark.parametrize("s", SHAPES[:6], ids=_id)
def test_weight_gradient_on_reference(env, s, cin, cout):  # noqa: F811
    """FP32 sums of BF16 products within 1e-4 (relative L2) of FP64, padding
    columns zero; an infinite activation reaches the same weights as in the
    general kernel (partial tiles must not bring it to others)."""
    L, torch = env
    n, D, H, W, circ = s
    x, _, _, dy = _inputs(torch, L, s, cin, cout, cin * cout)
    dw, db = _wgrad(L, torch, s, cin, cout, x, dy, True)
    _, rw, rb = C.conv3d_backward(x.double().cpu().numpy(), np.zeros((cout, 3, 3, 3, cin)), dy.double().cpu().numpy(),
                                  circ)
    assert rel_l2(dw[:, :27 * cin].cpu().numpy(), rw.reshape(cout, 27 * cin)) < 1e-4
    assert rel_l2(db.cpu().numpy(), rb) < 1e-4
    assert not dw[:, 27 * cin:].any()
    x[0, D - 1, H - 1, W - 1, 0] = float("inf")
    a = _wgrad(L, torch, s, cin, cout, x, dy, True)[0]
    b = _wgrad(L, torch, s, cin, cout, x, dy, False)[0]
    assert torch.equal(torch.isfinite(a), torch.isfinite(b))


def test_weight_gradient_over_splits(env):  # noqa: F811
    """Splits that take several tiles each (more than 512 tiles), with and
    without a bias gradient."""
    L, torch = env
    s = (4, 32, 40, 64, (False, True, True))
    x, _, _, dy = _inputs(torch, L, s, 16, 16, 5)
    a, da = _wgrad(L, torch, s, 16, 16, x, dy, True)
    b, db = _wgrad(L, torch, s, 16, 16, x, dy, False)
    assert rel_l2(a.double().cpu().numpy(), b.double().cpu().numpy()) < 1e-5
    assert rel_l2(da.double().cpu().numpy(), db.double().cpu().numpy()) < 1e-5
    n, D, H, W, circ = s
    scratch = torch.empty(L.mrtlbm_nn_wgrad_scratch_bytes(n, D, H, W, 16, 16) // 4, dtype=torch.float32, device="cuda")
    c = torch.empty_like(a)
    assert L.mrtlbm_nn_conv3d_wgrad(P(x), P(dy), n, D, H, W, 16, 16, circ_bits(circ), P(scratch), P(c), None, None) == 0
    assert torch.equal(a, c)
