"""GPU tests of library calls while their stream is being captured.

Captured steps replay in place: a launch of several steps moves a solve to its
second population array, and a graph holds pointers, so a captured call has to
end in the array it started from.
"""
import numpy as np
import pytest
import torch

from paper_2208_09267_amd import vanse
from paper_2208_09267_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(lat, dims, dtype):
    s = vanse.Solver(lat, dims, 0.7, dtype)
    d = 2 if lat == "D2Q9" else 3
    s.set_porosity(0.75, torch.from_numpy(W.fourier_eps(dims, seed=3)).cuda())  # static phi
    s.set_force((1e-6, -2e-7, 3e-7)[:d])
    s.init(None, torch.from_numpy(np.ascontiguousarray(W.taylor_green(dims, 0.03)[:d])).cuda())
    return s


@pytest.mark.parametrize("n", [2, 4, 8, 10, 16, 22])
@pytest.mark.parametrize("lat,dims,dtype,launch", [
    ("D2Q9", (64, 64, 1), vanse.FP64, "autotune"), ("D3Q19", (40, 24, 20), vanse.FP32_SHIFTED, (4, 4)),
    ("D3Q27", (64, 40, 10), vanse.FP64, (8, 8))])
def test_captured_steps_replay(lat, dims, dtype, launch, n):
    print("case", lat, dims, dtype, n, flush=True)
    a, b = (_solver(lat, dims, dtype) for _ in range(2))
    if launch == "autotune":
        a.autotune(8)
        a.init(None, torch.from_numpy(np.ascontiguousarray(W.taylor_green(dims, 0.03)[:2])).cuda())
    else:
        a.set_fused(*launch)
    for s in (a, b):
        s.step(6)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        a.step(n)
    done = 6
    for _ in range(4):  # with eager work and synchronisations in between
        g.replay()
        b.step(n)
        done += n
        torch.cuda.synchronize()
        x, y = (s.populations().cpu().numpy() for s in (a, b))
        assert np.array_equal(x, y), done
    # eager steps go on from the state of the last replay
    a.step(7)
    b.step(7)
    x, y = (s.populations().cpu().numpy() for s in (a, b))
    assert np.array_equal(x, y)
    a.close()
    b.close()


def test_calls_that_wait_are_refused_under_capture_and_leave_it_usable():
    s = _solver("D3Q19", (24, 20, 16), vanse.FP16_SHIFTED)
    r = _solver("D3Q19", (24, 20, 16), vanse.FP16_SHIFTED)
    n = 24 * 20 * 16
    eps, F = torch.zeros(n, dtype=torch.float64, device="cuda"), \
        torch.zeros((3, n), dtype=torch.float64, device="cuda")
    s.set_force_field(F)  # its first call allocates
    s.set_force_field(None)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    refused = 0
    with torch.cuda.graph(g):
        s.step(2)
        for call in (s.diagnostics, lambda: s.set_porosity(0.7, eps), lambda: s.set_force_field(F), s.init):
            for _ in range(20):
                with pytest.raises(vanse.VanseError) as e:
                    call()
                assert e.value.code == vanse.EDEVICE
                refused += 1
        s.step(2)
    assert refused == 80
    g.replay()
    r.step(4)
    assert np.array_equal(s.populations().cpu().numpy(), r.populations().cpu().numpy())
    assert s.diagnostics() == r.diagnostics()
    s.close()
    r.close()
