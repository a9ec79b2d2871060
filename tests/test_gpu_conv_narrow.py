"""Convolutions of volumes narrower than the tiles of the tiled kernels, which
gather their operands where a tile would be mostly padding: against the FP64
reference, and in time against a volume of as many voxels that fills tiles."""

import numpy as np
import pytest

from oracle import conv as C
from test_gpu_conv_tiles import _inputs, _wgrad
from test_gpu_nn import P, circ_bits, env, rel_l2  # noqa: F401

pytestmark = pytest.mark.gpu

# (n, D, H, W, circ): single voxels, lines and planes along each axis, small
# volumes; on both sides of the limits of padding and blocks
NARROW = [(300, 1, 1, 1, (True, True, True)), (600, 1, 1, 1, (False, False, False)), (40, 1, 1, 30, (False, True, True)),
          (1, 90, 60, 1, (False, True, True)), (2, 1, 70, 50, (True, False, True)), (150, 2, 3, 2, (False, True, True)),
          (60, 3, 5, 7, (True, True, True))]


@pytest.mark.parametrize("cin,cout", [(8, 48), (16, 32), (32, 128), (64, 64), (128, 64)])
@pytest.mark.parametrize("s", NARROW, ids=lambda s: "x".join(map(str, s[:4])))
def test_narrow_forward_on_reference(env, s, cin, cout):  # noqa: F811
    """FP32 sums of BF16 products within 1e-4 (relative L2) of FP64."""
    L, torch = env
    n, D, H, W, circ = s
    x, w, b, _ = _inputs(torch, L, s, cin, cout, cin + cout)
    y = torch.empty((n * D * H * W, cout), device="cuda")
    assert L.mrtlbm_nn_conv3d_fwd(P(x), n, D, H, W, cin, P(w), P(b), cout, circ_bits(circ), 0, None, P(y), None) == 0
    ref = C.conv3d(x.double().cpu().numpy(), w[:, :27 * cin].double().cpu().numpy().reshape(cout, 3, 3, 3, cin),
                   b.double().cpu().numpy(), circ)
    assert rel_l2(y.cpu().numpy(), ref.reshape(-1, cout)) < 1e-4


@pytest.mark.parametrize("cin,cout", [(8, 48), (16, 32), (32, 128), (64, 64), (128, 64)])
@pytest.mark.parametrize("s", NARROW, ids=lambda s: "x".join(map(str, s[:4])))
def test_narrow_weight_gradient_on_reference(env, s, cin, cout):  # noqa: F811
    """FP32 sums of BF16 products within 1e-4 (relative L2) of FP64."""
    L, torch = env
    x, _, _, dy = _inputs(torch, L, s, cin, cout, cin * cout)
    dw, db = _wgrad(L, torch, s, cin, cout, x, dy, True)
    _, rw, rb = C.conv3d_backward(x.double().cpu().numpy(), np.zeros((cout, 3, 3, 3, cin)), dy.double().cpu().numpy(),
                                  s[4])
    assert rel_l2(dw[:, :27 * cin].cpu().numpy(), rw.reshape(cout, 27 * cin)) < 1e-4
    assert rel_l2(db.cpu().numpy(), rb) < 1e-4
    assert not dw[:, 27 * cin:].any()


def _best(torch, f):
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        f()
        a.record()
        for _ in range(20):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 20)
    return best


SAME_VOXELS = [((2048, 1, 1, 1), (1, 8, 16, 16)), ((1, 256, 256, 1), (1, 64, 32, 32)), ((4, 64, 64, 1), (1, 16, 32, 32))]


@pytest.mark.parametrize("cin,cout", [(16, 32), (64, 64), (128, 128)])
@pytest.mark.parametrize("narrow,full", SAME_VOXELS, ids=lambda s: "x".join(map(str, s)))
def test_narrow_forward_takes_no_longer(env, narrow, full, cin, cout):  # noqa: F811
    """At most twice the time of a volume of as many voxels, or three quarters
    of that of a volume that fills the same tiles (8 voxels along the last
    axis): where gathering is the cheaper of the two, and no cheaper than that."""
    L, torch = env
    t = []
    for s in (narrow, full, narrow[:3] + (8,)):
        x, w, b, _ = _inputs(torch, L, s + ((False, True, True),), cin, cout, 1)
        y = torch.empty((int(np.prod(s)), cout), dtype=torch.bfloat16, device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        t.append(_best(torch, lambda: L.mrtlbm_nn_conv3d_fwd(P(x), *s, cin, P(w), P(b), cout, 6, 1, P(y), None, stream)))
    assert t[0] < max(2.0 * t[1], 0.75 * t[2]), t


@pytest.mark.parametrize("cin,cout", [(16, 32), (64, 64), (128, 128)])
def test_narrow_weight_gradient_takes_no_longer(env, cin, cout):  # noqa: F811
    """2048 single voxels: at most four times the time of one volume of as
    many (three quarters of which is the fixed time of a launch or two)."""
    L, torch = env
    t = []
    for s in ((2048, 1, 1, 1), (1, 8, 16, 16)):
        x, _, _, dy = _inputs(torch, L, s + ((False, True, True),), cin, cout, 1)
        scratch = torch.empty(L.mrtlbm_nn_wgrad_scratch_bytes(*s, cin, cout) // 4 + 4, device="cuda")
        dw, db = torch.empty((cout, L.mrtlbm_nn_kpad(cin)), device="cuda"), torch.empty(cout, device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        t.append(_best(torch, lambda: L.mrtlbm_nn_conv3d_wgrad(P(x), P(dy), *s, cin, cout, 6, P(scratch), P(dw), P(db),
                                                               stream)))
    assert t[0] < 4.0 * t[1], t


def test_input_gradient_of_more_weights_than_32_bits_count(env):  # noqa: F811
    """12624 -> 12624 channels (4.3e9 weights, 8.6 GB) on one voxel with all
    axes periodic, so that every tap and weight counts.  Whole numbers: the
    FP32 sums are exact and the BF16 result is their rounding."""
    L, torch = env
    c = 12624
    kpad = L.mrtlbm_nn_kpad(c)
    assert c * kpad > 1 << 32
    g = torch.Generator(device="cuda").manual_seed(1)
    w = torch.zeros((c, kpad), dtype=torch.bfloat16, device="cuda")
    dy = torch.randint(-1, 2, (c,), generator=g, device="cuda").to(torch.bfloat16)
    ref = torch.zeros(c, device="cuda")
    for t in range(27):
        part = torch.randint(-1, 2, (c, c), generator=g, device="cuda", dtype=torch.int8).to(torch.bfloat16)
        w[:, t * c:(t + 1) * c] = part
        ref += dy.float() @ part.float()
    wt = torch.full((c * kpad,), float("nan"), dtype=torch.bfloat16, device="cuda")
    dx = torch.empty(c, dtype=torch.bfloat16, device="cuda")
    assert L.mrtlbm_nn_conv3d_dgrad(P(dy), 1, 1, 1, 1, c, P(w), c, 7, P(wt), P(dx), None) == 0
    torch.cuda.synchronize()
    assert torch.equal(dx, ref.to(torch.bfloat16))
