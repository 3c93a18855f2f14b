"""GPU tests of the two-step launch on z-planes of more than 2^28 cells.

The kernel addresses a plane by 32-bit byte offsets: planes of up to 2 GiB step
two levels per launch, larger ones are accepted and take single steps.
"""
import pytest
import torch

from paper_2208_09267_amd import vanse
from paper_2208_09267_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _free():
    yield
    torch.cuda.empty_cache()


def test_a_plane_of_more_than_2_28_cells_equals_single_steps():
    dims, dev = (256, (1 << 20) + 8, 1), torch.device("cuda")
    print("case", dims, flush=True)
    out = []
    for fused in (False, True):
        s = vanse.Solver("D3Q19", dims, 0.7, vanse.FX16_SHIFTED)
        one = s.device_bytes
        s.set_porosity(0.75, W.fourier_eps_device(dims, 4, dev), 20.0)
        s.init(None, W.taylor_green_device(dims, 0.02, dev, 3))
        if fused:
            s.set_fused(4, 1)
            assert s.device_bytes > one
        s.step(5)
        out.append(s.moments())
        s.close()
    for x, y in zip(*out):
        assert torch.equal(x, y)


def test_a_plane_past_the_offsets_takes_single_steps():
    dims = (256, (1 << 21) + 4, 1)  # 4 bytes a cell: just over 2 GiB
    print("case", dims, flush=True)
    s = vanse.Solver("D3Q19", dims, 0.7, vanse.FX16_SHIFTED)
    one = s.device_bytes
    s.set_porosity(0.75, None)
    s.init()
    s.set_fused(4, 1)
    assert s.device_bytes == one
    with pytest.raises(vanse.VanseError) as e:
        s.set_fused(9, 1)  # no such tile at any size
    assert e.value.code == vanse.EINVAL
    s.step(3)
    mass, momentum, force = s.diagnostics()
    n = dims[0] * dims[1]
    # the uniform state at rest: the code of every population is 0
    assert abs(mass - 0.75 * n) <= 1e-9 * n and s.time == 3
    s.close()
