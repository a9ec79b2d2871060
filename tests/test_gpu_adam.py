"""Adam on one tensor of each size class against the kernel that takes many."""

import ctypes

import pytest

from test_gpu_nn import P, env  # noqa: F401

pytestmark = pytest.mark.gpu

ONE = 4 << 20  # values from which on a tensor of its own takes the other kernel


@pytest.mark.parametrize("n", [1, 255, 1000001, ONE - 1, ONE, ONE + 1025])
@pytest.mark.parametrize("low", [True, False])
def test_one_tensor_equals_many(env, n, low):  # noqa: F811
    """Bit for bit, two steps, with and without the BF16 copy."""
    L, torch = env
    g = torch.Generator(device="cuda").manual_seed(n)
    first = [torch.rand(n, generator=g, device="cuda") for _ in range(4)]
    other = [torch.rand(5, generator=g, device="cuda") for _ in range(4)]
    out = []
    for many in (False, True):
        t = [x.clone() for x in first]
        u = [x.clone() for x in other]
        wb = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
        for step in (1, 2):
            if many:
                pp = [(ctypes.c_void_p * 2)(a.data_ptr(), b.data_ptr()) for a, b in zip(t, u)]
                pb = (ctypes.c_void_p * 2)(wb.data_ptr() if low else None, None)
                assert L.mrtlbm_nn_adam_all(2, pp[0], pp[1], pp[2], pp[3], (ctypes.c_longlong * 2)(n, 5), 1e-3, 0.9, 0.999,
                                            1e-8, step, pb, None) == 0
            else:
                assert L.mrtlbm_nn_adam(*(P(x) for x in t), n, 1e-3, 0.9, 0.999, 1e-8, step, P(wb) if low else None,
                                        None) == 0
        out.append(t + [wb])
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert not torch.equal(out[0][0], first[0]) and bool(out[0][4].any()) == low
