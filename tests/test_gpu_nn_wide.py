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


def test_upsampling_beyond_32_bit_groups(env):  # noqa: F811
    """2^31 groups of 8 channels (a 34 GB output): each takes its coarse voxel."""
    L, torch = env
    e, c = 512, 16
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(-128, 128, (e, e, e, c), generator=g, device="cuda", dtype=torch.int8).to(torch.bfloat16)
    y = torch.empty((e, 2, e, 2, e, 2, c), dtype=torch.bfloat16, device="cuda")
    assert y.numel() // 8 == 1 << 31
    assert L.mrtlbm_nn_up2(1, P(x), 1, e, e, e, c, P(y), None) == 0
    for z in range(0, e, 64):
        for d in range(8):
            assert torch.equal(y[z:z + 64, d >> 2, :, d >> 1 & 1, :, d & 1], x[z:z + 64]), (z, d)


@pytest.mark.parametrize("coarse,fine", [((8, 8, 8), (16, 16, 16)), ((1, 2, 3), (5, 4, 7)), ((9, 21, 40), (19, 33, 130)),
                                         ((16, 16, 48), (9, 11, 65)), ((40, 40, 40), (7, 6, 9)),
                                         ((64, 64, 64), (128, 96, 72))], ids=str)
def test_temperature_from_coarse_grid(env, coarse, fine):  # noqa: F811
    """Staged tiles, or for a finer coarse grid the gathering kernel, against
    the interpolation in FP64; the count of rejected values against the field."""
    L, torch = env
    c, scale, margin = 16, 3.0, 0.1
    g = torch.Generator(device="cuda").manual_seed(fine[2])
    pred = torch.randn(coarse + (c,), generator=g, device="cuda")
    T = torch.empty(fine, device="cuda")
    scratch = torch.empty(4096, dtype=torch.int32, device="cuda")
    bad = ctypes.c_longlong()
    assert L.mrtlbm_nn_to_temperature(P(pred), c, *coarse, *fine, scale, margin, P(T), P(scratch), ctypes.byref(bad),
                                      None) == 0
    ref = pred[..., 0].double()
    for a, (nc, n) in enumerate(zip(coarse, fine)):
        x = (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) * nc / n - 0.5
        lo = torch.floor(x)
        t = (x - lo).view([-1 if i == a else 1 for i in range(3)])
        lo = lo.long()
        lo, hi = (lo.clamp(0, nc - 1), (lo + 1).clamp(0, nc - 1)) if a == 2 else (lo % nc, (lo + 1) % nc)
        ref = (1 - t) * ref.index_select(a, lo) + t * ref.index_select(a, hi)
    W = fine[2]
    ref = ref / scale + 1 - (torch.arange(W, device="cuda", dtype=torch.float64) + 0.5) / W
    # FP32 coordinates: off by 2^-22 of the extent, times a difference of two
    # values, on each axis; and about sixteen roundings
    big = float(pred.abs().max())
    tol = (6 * max(coarse) * 2.0 ** -22 + 2.0 ** -20) * big / scale + 2.0 ** -21
    assert float((T.double() - ref).abs().max()) <= tol
    assert bad.value == int(((T < -margin) | (T > torch.tensor(1.0 + margin))).sum())


def test_adam_on_many_tensors_equals_one_by_one(env):  # noqa: F811
    """Bit for bit, over more tensors than a launch takes, an empty one and sizes
    around a block's values."""
    L, torch = env
    sizes = [1, 0, 1023, 1024, 1025, 5000] + [7 * k + 1 for k in range(40)]
    g = torch.Generator(device="cuda").manual_seed(1)

    def tensors():
        return [[torch.rand(max(n, 1), generator=g.manual_seed(9 * i + k), device="cuda") for i, n in enumerate(sizes)]
                for k in range(4)]

    a, b = tensors(), tensors()
    ab, bb = ([torch.zeros(max(n, 1), dtype=torch.bfloat16, device="cuda") for n in sizes] for _ in range(2))
    n = len(sizes)
    for t in (1, 2):
        ptrs = [(ctypes.c_void_p * n)(*(x.data_ptr() for x in xs)) for xs in a]
        wb = (ctypes.c_void_p * n)(*(None if i % 3 == 0 else x.data_ptr() for i, x in enumerate(ab)))
        assert L.mrtlbm_nn_adam_all(n, *ptrs, (ctypes.c_longlong * n)(*sizes), 1e-2, 0.9, 0.999, 1e-8, t, wb, None) == 0
        for i in range(n):
            assert L.mrtlbm_nn_adam(*(P(b[k][i]) for k in range(4)), sizes[i], 1e-2, 0.9, 0.999, 1e-8, t,
                                    None if i % 3 == 0 else P(bb[i]), None) == 0
    for x, y in zip(sum(a, []) + ab, sum(b, []) + bb):
        assert torch.equal(x, y)
