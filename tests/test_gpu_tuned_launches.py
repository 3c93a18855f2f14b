"""GPU tests of the launches that only the tuners and the batch layout choose.

The autotuner runs each of its candidates as real steps, so an autotuned solve
equals one that took as many single steps bit for bit: FP64 and D3Q27 tiles of
the largest blocks, ragged widths, and lattices at the edges of the range in
which it tries small blocks, ranges of blocks per XCD and nontemporal stores.
A batch whose tall tiles fill the chip, and small batches of single steps (each
XCD a range of blocks), equal the solves stepped alone.
"""
import numpy as np
import pytest
import torch

from paper_2208_09267_amd import vanse
from paper_2208_09267_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(lat, dims, dtype, seed):
    s = vanse.Solver(lat, dims, 0.55 + 0.01 * seed, dtype)
    d = 2 if lat == "D2Q9" else 3
    s.set_porosity(0.75, torch.from_numpy(W.fourier_eps(dims, seed=seed)).cuda(), 21.0 + seed)
    s.set_force((1e-6, -2e-7, 3e-7)[:d])
    s.init(None, torch.from_numpy(np.ascontiguousarray(W.taylor_green(dims, 0.03)[:d])).cuda())
    return s


def _bits(s):
    return s.populations().cpu().numpy()


def _same(x, y):
    """Every value equal (an FX16 code at its range's bound reads as NaN in both)."""
    return np.array_equal(x, y, equal_nan=True)


TUNED = [("D3Q27", (40, 24, 36), vanse.FP64), ("D3Q27", (100, 33, 17), vanse.FP64),
         ("D3Q19", (93, 37, 29), vanse.FP64), ("D3Q19", (187, 20, 11), vanse.FP32_SHIFTED),
         ("D3Q19", (32, 32, 16), vanse.FP32_SHIFTED), ("D3Q19", (31, 33, 16), vanse.FP64),
         ("D3Q19", (128, 128, 128), vanse.FX16_SHIFTED), ("D3Q27", (29, 29, 29), vanse.FP16_SHIFTED),
         ("D2Q9", (157, 131, 1), vanse.FP64)]


@pytest.mark.parametrize("case", range(len(TUNED)))
def test_autotuned_solve_equals_single_steps_bitwise(case):
    lat, dims, dtype = TUNED[case]
    print("case", lat, dims, dtype, flush=True)
    a, b = (_solver(lat, dims, dtype, 3 + case) for _ in range(2))
    a.autotune(3)
    a.step(11)
    b.step(a.time)
    assert _same(_bits(a), _bits(b))
    a.close()
    b.close()


@pytest.mark.parametrize("lat,dims,dtype", [
    ("D3Q19", (1, 1, 1), vanse.FP64), ("D3Q19", (31, 7, 5), vanse.FP32_SHIFTED),
    ("D3Q27", (64, 9, 11), vanse.FP64), ("D2Q9", (256, 33, 1), vanse.FP16_SHIFTED),
    ("D3Q19", (110, 110, 109), vanse.FP64), ("D3Q19", (110, 110, 110), vanse.FP64)])  # 192 MB
def test_untuned_launch_equals_plain_blocks_bitwise(lat, dims, dtype):
    print("case", lat, dims, dtype, flush=True)
    a, b = (_solver(lat, dims, dtype, 4) for _ in range(2))
    b.set_tuning(256, 0)
    a.step(7)
    b.step(7)
    assert _same(_bits(a), _bits(b))
    a.close()
    b.close()


# members, two-step or not
BATCHES = [("D3Q19", [(64, 96, 256), (70, 90, 250), (64, 96, 256)], vanse.FP32_SHIFTED, True),
           ("D3Q27", [(48, 120, 320), (50, 131, 310), (33, 97, 330)], vanse.FP64, True),
           ("D3Q19", [(33, 17, 9), (40, 40, 40), (1, 1, 1)], vanse.FP32_SHIFTED, False),
           ("D3Q27", [(20, 30, 40), (5, 3, 7)], vanse.FP16_SHIFTED, False)]


@pytest.mark.parametrize("case", range(len(BATCHES)))
def test_batch_equals_solves_alone_bitwise(case):
    lat, shapes, dtype, two = BATCHES[case]
    print("case", lat, shapes, dtype, two, flush=True)
    make = lambda: [_solver(lat, d, dtype, 5 + k) for k, d in enumerate(shapes)]
    want = []
    for s in make():
        s.step(21)
        want.append(_bits(s))
        s.close()
    members = make()
    b = vanse.Batch(members)
    b.set_tuning(256, vanse.TUNE_TWO_STEP if two else 0, 16)
    if two:
        tiles = b.two_step_tiles()
        # at 32 planes these tiles are more than the CUs
        assert sum(-(-d[1] // r) * -(-d[2] // 32) for d, (_, r, _) in zip(shapes, tiles)) >= 200
    b.step(21)
    for k, s in enumerate(members):
        assert _same(_bits(s), want[k]), k
    b.close()
    for s in members:
        s.close()
