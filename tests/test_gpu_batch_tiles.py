"""GPU tests of the batched two-step launch's tiles on members wider than those
of the batched workloads: the tall tiles (as many rows as the largest block
takes, where they fill every CU) in every storage mode, and x-split tiles in
FP16, where a value rounded twice differs once in some 2^13."""
import numpy as np
import pytest
import torch

from paper_2208_09267_amd import vanse
from paper_2208_09267_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(lat, dims, dtype, seed):
    dev = torch.device("cuda")
    s = vanse.Solver(lat, dims, 0.55 + 0.01 * seed, dtype)
    s.set_porosity(0.75, W.fourier_eps_device(dims, seed, dev), 60.0 + seed)
    s.set_force((1e-6, -2e-7, 3e-7))
    s.init(None, W.taylor_green_device(dims, 0.02, dev, 3))
    return s


def _equal(a, b):
    x, y = a.populations(), b.populations()
    return bool(((x == y) | (x.isnan() & y.isnan())).all())


def _check(lat, shapes, dtype, steps, tiles):
    members = [_solver(lat, d, dtype, 1 + k) for k, d in enumerate(shapes)]
    b = vanse.Batch(members)
    b.set_tuning(256, vanse.TUNE_TWO_STEP, 16)
    got = b.two_step_tiles()
    print("tiles", got, flush=True)
    tiles(got)
    b.step(steps)
    for k, m in enumerate(members):
        alone = _solver(lat, shapes[k], dtype, 1 + k)
        alone.step(steps)
        assert _equal(alone, m), k
        alone.close()
    b.close()
    for m in members:
        m.close()


# 20 x 8, 17 x 10 and 4 x 4 tiles of the largest block (FP32, FP16, FX16 D3Q19:
# 1024 threads; else 512) in segments of 32 planes: more than the 256 CUs
TALL = [(187, 96, 256), (150, 100, 300), (64, 64, 128)]


@pytest.mark.parametrize("lat,dtype,rows", [
    ("D3Q19", vanse.FP32_SHIFTED, [5, 6, 16]), ("D3Q19", vanse.FP16_SHIFTED, [5, 6, 16]),
    ("D3Q19", vanse.FX16_SHIFTED, [5, 6, 16]), ("D3Q19", vanse.FP64, [2, 3, 8]),
    ("D3Q27", vanse.FP64, [2, 3, 8]), ("D3Q27", vanse.FP16_SHIFTED, [2, 3, 8])])
def test_tall_tiles_equal_the_solves_alone_bitwise(lat, dtype, rows):
    print("case", lat, dtype, flush=True)

    def tiles(got):
        assert [r for _, r, _ in got] == rows
        assert [c for c, _, _ in got] == [d[0] for d in TALL]
        assert sum(-(-d[1] // r) * -(-d[2] // 32) for d, r in zip(TALL, rows)) >= 256

    _check(lat, TALL, dtype, 21, tiles)


@pytest.mark.parametrize("dtype", [vanse.FP16_SHIFTED, vanse.FP32_SHIFTED])
def test_x_split_tiles_equal_the_solve_alone_at_large(dtype):
    shapes = [(400, 60, 100), (70, 50, 30)]

    def tiles(got):
        assert got[0][0] <= 62 and got[1][0] == 70  # columns of a tile

    _check("D3Q19", shapes, dtype, 40, tiles)
