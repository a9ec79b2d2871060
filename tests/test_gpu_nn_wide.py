"""The pooling and upsampling kernels that take 8 channels per thread against
the one-channel kernels, which take the same call when the output is not
aligned for them."""

import ctypes

import pytest

from test_gpu_nn import P, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 2, 2, 2, 8), (3, 4, 6, 10, 24), (2, 2, 34, 18, 128), (4, 32, 32, 64, 16)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("forward", [1, 0])
def test_pool_and_upsampling_equal_general_kernels(env, shape, forward):  # noqa: F811
    """Bit for bit: the same sums in the same order."""
    L, torch = env
    n, D, H, W, c = shape
    g = torch.Generator(device="cuda").manual_seed(c + forward)
    fine = torch.randn(n * D * H * W * c, generator=g, device="cuda").to(torch.bfloat16)
    coarse = fine[:fine.numel() // 8].clone()
    for op, (d, h, w), x, size in ((L.mrtlbm_nn_pool2, (D, H, W), *((fine, coarse) if forward else (coarse, fine))),
                                   (L.mrtlbm_nn_up2, (D // 2, H // 2, W // 2),
                                    *((coarse, fine) if forward else (fine, coarse)))):
        got = torch.empty_like(size)
        ref = torch.empty(size.numel() + 8, dtype=torch.bfloat16, device="cuda")
        assert op(forward, P(x), n, d, h, w, c, P(got), None) == 0
        assert op(forward, P(x), n, d, h, w, c, ctypes.c_void_p(ref.data_ptr() + 2), None) == 0
        assert torch.equal(got, ref[1:1 + size.numel()])
