"""bench.py's command-line contract that needs no GPU."""

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120, cwd=ROOT)
    assert p.returncode == 2
    line = json.loads(p.stdout.strip().splitlines()[-1])
    assert "one GPU" in line["error"]


def test_help_lists_the_modes():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--help"], capture_output=True, text=True,
                       timeout=120, cwd=ROOT)
    assert p.returncode == 0
    for mode in ("throughput", "copy", "solve", "sweep", "warmstart", "paper", "network"):
        assert mode in p.stdout


def test_measured_traffic_is_that_of_the_kernel_and_shape():
    sys.path.insert(0, ROOT)
    import bench

    names = ("vec", "bx", "by", "nt", "map")
    tuned, other = dict(zip(names, (4, 64, 4, 2, 1))), dict(zip(names, (4, 32, 8, 0, 0)))
    assert bench.measured_traffic("braid256_f32", "moments", "k_step", tuned) == 563_201_378
    assert bench.measured_traffic("braid256_f32", "moments", "k_step", other) is None
    for launch in (tuned, other):
        assert bench.measured_traffic("braid256_f32", "moments", "k_step2", launch) == 580_211_342
    assert bench.measured_traffic("braid128_f32", "moments", "k_step2", tuned) is None
    assert bench.measured_traffic("braid256_f32", "moments", "k_box", tuned) is None


def test_network_flop_count():
    # the U-Net's convolutions at 64^3: level-0 layers carry sum C_in*C_out =
    # 8*16 + 16*16 + 32*16 + 16*16 + 16*16, level 1 (32^3) 16*32 + 32*32 +
    # 64*32 + 32*32, level 2 (16^3) 32*64 + 64*64 + 128*64 + 64*64, level 3
    # (8^3) 64*128 + 128*128; each voxel-channel pair costs 2 * 27 FLOPs
    import types

    from paper_1503_08718_amd import warmstart as ws

    cc = [(64 ** 3, 1408), (32 ** 3, 4608), (16 ** 3, 18432), (8 ** 3, 24576)]
    fwd = 54.0 * sum(v * c for v, c in cc)
    cube = (64, 64, 64)
    assert ws.forward_flops(types.SimpleNamespace(batch=1, n=64, grid=cube)) == fwd
    assert ws.forward_flops(types.SimpleNamespace(batch=4, n=64, grid=cube)) == 4 * fwd
    # training: forward + weight gradient everywhere, input gradient except the first layer
    first = 54.0 * 64 ** 3 * 8 * 16
    assert ws.iteration_flops(types.SimpleNamespace(batch=1, n=64, grid=cube)) == 3 * fwd - first
    # a 32 x 48 x 64 grid: every level has 32*48*64 / 64^3 of the cube's voxels
    assert ws.forward_flops(types.SimpleNamespace(batch=1, n=64, grid=(32, 48, 64))) == fwd * 0.375


def test_inference_grid():
    """One coarsening factor, max extent / 64, on every axis; extents rounded
    to multiples of 8: the sweep's shapes keep cubic (or, for a largest extent
    of 96, nearly cubic) voxels, and cubic cells map to 64^3."""
    from paper_1503_08718_amd.warmstart import inference_grid

    assert inference_grid((64, 64, 64), 64) == (64, 64, 64)
    assert inference_grid((128, 128, 128), 64) == (64, 64, 64)
    assert inference_grid((96, 96, 96), 64) == (64, 64, 64)
    assert inference_grid((128, 64, 96), 64) == (64, 32, 48)
    assert inference_grid((64, 96, 128), 64) == (32, 48, 64)
    assert inference_grid((96, 64, 64), 64) == (64, 40, 40)  # 42.7 -> 40
    assert inference_grid((16, 16, 512), 64) == (8, 8, 64)  # at least 8
    for shape in [(a, b, c) for a in (64, 96, 128) for b in (64, 96, 128) for c in (64, 96, 128)]:
        g = inference_grid(shape, 64)
        assert max(g) == 64 and all(e % 8 == 0 for e in g)
        f = [s / e for s, e in zip(shape, g)]
        assert max(f) / min(f) <= 1.07  # voxel aspect within 7 %


def test_mixed_training_cells():
    import workloads as w

    c = w.warmstart_cells_mixed(8721, 200)
    assert c == w.warmstart_cells_mixed(8721, 200)  # seeded
    assert {x["nx"] for x in c} == {32, 40, 48, 64} and {x["nz"] for x in c} == {32, 40, 48, 64}
    assert all(20.0 <= x["gamma"] <= 45.0 and 0.35 <= x["v"] <= 0.6 for x in c)
