"""GPU tests of vanse_autotune's trials and of what it keeps: which calls run
trials again, how many real steps a trial takes, and what a caller can do with
the launch it reports."""
import numpy as np
import pytest
import torch

from paper_2208_09267_amd import vanse
from paper_2208_09267_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(lat, dims, dtype, seed=3, period=31.0):
    s = vanse.Solver(lat, dims, 0.55 + 0.01 * seed, dtype)
    d = 2 if lat == "D2Q9" else 3
    s.set_porosity(0.75, torch.from_numpy(W.fourier_eps(dims, seed=seed)).cuda(), period)
    s.set_force((1e-6, -2e-7, 3e-7)[:d])
    s.init(None, torch.from_numpy(np.ascontiguousarray(W.taylor_green(dims, 0.03)[:d])).cuda())
    return s


def _bits(s):
    return s.populations().cpu().numpy()


# size classes that no other test tunes
@pytest.mark.parametrize("lat,dims,dtype", [("D2Q9", (211, 95, 1), vanse.FX16_SHIFTED),
                                            ("D3Q19", (53, 31, 23), vanse.FX16_SHIFTED)])
def test_longer_trials_run_again_and_replace_the_choice(lat, dims, dtype):
    print("case", lat, dims, dtype, flush=True)
    a = _solver(lat, dims, dtype)
    first = a.autotune(2)
    assert first.steps_run > 0
    assert a.autotune(1) == first._replace(steps_run=0)
    longer = a.autotune(8)
    assert longer.steps_run > first.steps_run
    assert a.autotune(8) == longer._replace(steps_run=0)
    assert a.autotune(3) == longer._replace(steps_run=0)
    a.close()


@pytest.mark.parametrize("trial,pre", [(1, 0), (3, 1), (8, 1), (8, 0)])
def test_d2q9_box_trials_are_whole_launches_from_an_even_level(trial, pre):
    dims = (64 + trial, 150 + pre, 1)  # a class of its own per case (nx is part of it)
    print("case", dims, trial, pre, flush=True)
    a, b = (_solver("D2Q9", dims, vanse.FX16_SHIFTED) for _ in range(2))
    a.step(pre)
    run = a.autotune(trial).steps_run
    # three boxes of 8 steps and two of 4, twice each, trials rounded up
    boxes = 2 * (3 * (-(-trial // 8) * 8) + 2 * (-(-trial // 4) * 4))
    singles = run - boxes
    assert singles > 0
    # n candidates of one step each, and a step to an even level where they end odd
    n, extra = divmod(singles, trial)
    if trial > 1:
        assert extra == (pre + n * trial) % 2
    assert (pre + run) % 2 == 0
    assert a.time == pre + run
    a.step(29)
    b.step(a.time)
    assert np.array_equal(_bits(a), _bits(b), equal_nan=True)
    a.close()
    b.close()


@pytest.mark.parametrize("lat,dims,dtype", [("D3Q19", (11, 9, 7), vanse.FP64), ("D2Q9", (61, 43, 1), vanse.FP64),
                                            ("D3Q27", (256, 6, 2), vanse.FP32_SHIFTED)])
def test_small_lattices_are_tried_in_the_untuned_order(lat, dims, dtype):
    """Their untuned launch gives each XCD a contiguous range of blocks, and so
    do the single-step launches they are tuned with."""
    print("case", lat, dims, dtype, flush=True)
    a, b = (_solver(lat, dims, dtype) for _ in range(2))
    assert a.autotune(4).flags & vanse.TUNE_XCD_REMAP
    a.step(7)
    b.step(a.time)
    assert np.array_equal(_bits(a), _bits(b))
    a.close()
    b.close()


def test_large_lattices_in_16_bits_try_the_untuned_launch():
    """2.3 M cells of 38 bytes (87 MB) run with ranges of blocks per XCD untuned:
    the tuner tries them as it does below 2^21 cells, 15 launches more than the
    those it has for every size (1024 threads and 64 to 512 with each choice of
    ranges and nontemporal stores; nx is no multiple of the tiled launches' 256)."""
    s = _solver("D3Q19", (160, 120, 121), vanse.FX16_SHIFTED)
    run = s.autotune(2).steps_run
    s.close()
    # flat: 256, 512, 1024 threads; two-step: as many tiles as at any size
    t = _solver("D3Q19", (160, 120, 321), vanse.FX16_SHIFTED)  # 234 MB: not remapped
    base = t.autotune(2).steps_run
    t.close()
    assert run - base == 2 * 15


def _big_plane():
    """D2Q9 FP64, 67 M cells: 4.8 GB of populations; boxes win by about 2."""
    dims, dev = (8192, 8192, 1), torch.device("cuda")
    s = vanse.Solver("D2Q9", dims, 0.7, vanse.FP64)
    s.set_porosity(0.75, W.fourier_eps_device(dims, 2, dev), 40.0)
    s.init(None, W.taylor_green_device(dims, 0.02, dev, 2))
    return s


def test_a_choice_without_memory_for_its_second_array_takes_single_steps():
    a = _big_plane()
    one = a.device_bytes
    a.autotune(8)
    boxes = a.device_bytes > one
    print("boxes chosen:", boxes, flush=True)
    a.close()
    b, c = _big_plane(), _big_plane()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    hog = torch.empty(free - (3 << 30), dtype=torch.uint8, device="cuda")  # 3 GB left
    assert b.autotune(8).steps_run == 0      # the class has its choice
    assert b.device_bytes == one
    short = b.autotune(16)                   # longer trials: without the boxes
    assert short.steps_run > 0 and b.device_bytes == one
    assert short.fused_rows == 0
    b.step(5)
    assert b.time == short.steps_run + 5
    del hog
    torch.cuda.empty_cache()
    again = c.autotune(16)                   # what was found without memory is not kept
    assert again.steps_run > short.steps_run
    assert (c.device_bytes > one) == boxes
    c.init(None, W.taylor_green_device((8192, 8192, 1), 0.02, torch.device("cuda"), 2))
    b.init(None, W.taylor_green_device((8192, 8192, 1), 0.02, torch.device("cuda"), 2))
    for s in (b, c):
        s.step(11)
    for x, y in zip(b.moments(), c.moments()):
        assert torch.equal(x, y)
    b.close()
    c.close()


# two-step tiles that are none of the general rules' (FP64, D3Q27, ragged widths)
TILES = [("D3Q27", (64, 40, 70), vanse.FP64, 8, 32), ("D3Q27", (64, 40, 10), vanse.FP64, 7, 8),
         ("D3Q19", (187, 17, 20), vanse.FP64, 2, 16), ("D3Q19", (187, 17, 20), vanse.FP32_SHIFTED, 5, 8),
         ("D3Q27", (100, 11, 9), vanse.FX16_SHIFTED, 5, 64), ("D3Q27", (256, 6, 5), vanse.FP64, 2, 8),
         ("D3Q19", (93, 37, 29), vanse.FP16_SHIFTED, 11, 128)]


@pytest.mark.parametrize("lat,dims,dtype,rows,planes", TILES)
def test_a_tile_the_autotuner_may_report_can_be_set(lat, dims, dtype, rows, planes):
    print("case", lat, dims, dtype, rows, planes, flush=True)
    a, b = (_solver(lat, dims, dtype) for _ in range(2))
    a.set_fused(rows, planes)
    for n in (2, 7, 4):
        a.step(n)
        b.step(n)
    assert np.array_equal(_bits(a), _bits(b), equal_nan=True)
    with pytest.raises(vanse.VanseError) as e:  # one row more than a block takes
        a.set_fused(1024 // dims[0] + 1, planes)
    assert e.value.code == vanse.EINVAL
    a.close()
    b.close()


@pytest.mark.parametrize("lat,dims,dtype", [("D3Q27", (160, 128, 128), vanse.FP64), ("D3Q19", (187, 141, 93), vanse.FP64),
                                            ("D3Q19", (250, 61, 64), vanse.FP32_SHIFTED)])
def test_the_reported_launch_can_be_restored(lat, dims, dtype):
    print("case", lat, dims, dtype, flush=True)
    a, b = (_solver(lat, dims, dtype) for _ in range(2))
    launch = a.autotune(4)
    print("chosen", launch, flush=True)
    b.set_tuning(256, launch.flags)
    b.set_tile(launch.tile_x, launch.tile_y)
    b.set_fused(launch.fused_rows, launch.fused_planes)
    assert a.device_bytes == b.device_bytes
    u0 = torch.from_numpy(np.ascontiguousarray(W.taylor_green(dims, 0.03))).cuda()
    for s in (a, b):  # the trials ran past the phase in which this flow is stable
        s.init(None, u0)
        s.step(11)
    assert np.array_equal(_bits(a), _bits(b))
    a.close()
    b.close()
