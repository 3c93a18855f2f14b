"""GPU tests of D2Q9's launches of several steps (csrc/box.hip).

The autotuner runs every box kind as real steps, so a solve that has been
autotuned must equal one that took the same number of single steps bit for bit:
lattices smaller than a box, larger than several, of ragged sizes and one row;
trial lengths that end on fewer steps than a box takes; odd starts; a per-cell
force and every quadrature; every storage mode.  And one solve against the
oracle.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import oracle_run, rel_linf
from paper_2208_09267_amd import vanse
from paper_2208_09267_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(dims, dtype, seed, quad=0, force=False):
    n = int(np.prod(dims))
    rng = np.random.default_rng(seed)
    s = vanse.Solver("D2Q9", dims, 0.63, dtype)
    s.set_porosity(0.75, torch.from_numpy(W.fourier_eps(dims, seed=seed)).cuda(), 23.0, quad)
    s.set_force((1e-6, -2e-6))
    if force:
        s.set_force_field(torch.from_numpy(rng.uniform(-1e-4, 1e-4, (2, n))).cuda())
    s.init(torch.from_numpy(rng.uniform(0.98, 1.02, n)).cuda(),
           torch.from_numpy(np.ascontiguousarray(W.taylor_green(dims, 0.03)[:2])).cuda())
    return s


def _same(a, b):
    """Every population equal (an FX16 code at its range's bound reads as NaN
    in both: the force drives the longest of these runs there)."""
    return np.array_equal(a.populations().cpu().numpy(), b.populations().cpu().numpy(),
                          equal_nan=True)


CASES = [((1, 1, 1), 8, 0, 0), ((3, 5, 1), 8, 1, 1), ((64, 64, 1), 8, 0, 0), ((33, 29, 1), 7, 1, 2),
         ((130, 61, 1), 10, 0, 8), ((58, 10, 1), 2, 1, 0), ((59, 11, 1), 5, 0, 3), ((400, 1, 1), 8, 0, 0),
         ((1, 300, 1), 12, 1, 0), ((517, 203, 1), 9, 0, 0)]


@pytest.mark.parametrize("dtype", [vanse.FP64, vanse.FP32_SHIFTED, vanse.FP16_SHIFTED,
                                   vanse.FX16_SHIFTED])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_boxes_equal_single_steps_bitwise(case, dtype):
    dims, trial, pre, quad = CASES[case]
    print("case", dims, trial, pre, quad, dtype, flush=True)
    a, b = (_solver(dims, dtype, 40 + case, quad, force=case % 2 == 0) for _ in range(2))
    a.step(pre)
    launch = a.autotune(trial)
    assert launch.fused_rows == 0 and launch.fused_planes == 0
    assert a.time == pre + launch.steps_run
    a.step(29)
    b.step(a.time)
    assert _same(a, b)
    a.set_fused(0)  # back to single steps, at any level
    a.step(6)
    b.step(6)
    assert _same(a, b)
    a.close()
    b.close()


def test_boxes_vs_oracle():
    dims = (70, 45, 1)
    pert, u0 = W.fourier_eps(dims, seed=9), np.ascontiguousarray(W.taylor_green(dims, 0.03)[:2])
    s = vanse.Solver("D2Q9", dims, 0.7, vanse.FP64)
    s.set_porosity(0.75, torch.from_numpy(pert).cuda(), 17.0)
    s.set_force((1e-5, -2e-6))
    s.init(None, torch.from_numpy(u0).cuda())
    s.autotune(8)
    s.init(None, torch.from_numpy(u0).cuda())
    s.step(44)
    got = [t.cpu().numpy() for t in s.moments()]
    s.close()
    _, *want = oracle_run("D2Q9", dims, 0.7, 0.75, pert, 17.0, 44, u0=u0, force=(1e-5, -2e-6, 0))
    for a, b in zip(got, want):
        assert rel_linf(a, b) <= 1e-12
