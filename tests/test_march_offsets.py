"""CPU check of the marching kernel's packed and scaled offsets (csrc/march.h):
the 16-bit modes keep a cell's distances to its x-neighbours in one register, 16
bits each, and phi offsets are derived from population offsets; lanes without a
cell store at an offset that the bounds check must refuse."""
import numpy as np
import pytest

MAX_WIDTH = 2 * 1024  # march_tile: nx * rows <= 2 nt, blocks of at most 1024 threads
NO_STORE = 0x80000000


def _i32(v):
    return np.asarray(v, dtype=np.int64).astype(np.uint64).astype(np.uint32).view(np.int32)


def _c_div(v, d):  # C's division truncates
    return np.trunc(np.asarray(v, dtype=np.float64) / d).astype(np.int64)


@pytest.mark.parametrize("nx", [1, 2, 3, 63, 64, 65, 127, 256, 511, 1000, 1023, 1024, 2047, MAX_WIDTH])
def test_packed_distances_to_the_x_neighbours(nx):
    x = np.arange(nx, dtype=np.int64)
    dm, dp = np.where(x == 0, nx - 1, -1), np.where(x + 1 == nx, 1 - nx, 1)
    packed = _i32((dm & 0xffff) | ((dp & 0xffff) << 16))
    low = (packed & 0xffff).astype(np.uint16).view(np.int16).astype(np.int64)
    high = (packed >> 16).astype(np.int64)  # arithmetic shift
    assert (low == dm).all() and (high == dp).all()
    assert ((x + low) % nx == (x - 1) % nx).all() and (0 <= x + low).all() and (x + low < nx).all()
    assert (0 <= x + high).all() and (x + high < nx).all()


@pytest.mark.parametrize("t,r", [(8, 8), (4, 4), (2, 4)])
def test_population_bytes_to_phi_bytes(t, r):
    cells = np.concatenate([np.arange(-MAX_WIDTH, 4 * MAX_WIDTH), [2 ** 28 - 1]])
    assert (_c_div(cells * t, t) * r == cells * r).all()


@pytest.mark.parametrize("t,r", [(8, 8), (4, 4), (2, 4)])
def test_lanes_without_a_cell_store_past_the_largest_plane(t, r):
    for nx in (1, 2, 256, MAX_WIDTH):
        nxy = ((1 << 31) - 1) // max(t, r) - 2 * nx  # march_plane's largest
        assert (nxy + 2 * nx) * max(t, r) < 1 << 31
        assert nxy * max(t, r) < 1 << 31          # plane_buffer's size is an int
        for step in (0, -1, 1, nx - 1, 1 - nx):   # with the x-neighbour added, in 32 bits
            assert (NO_STORE + step * t) % (1 << 32) >= nxy * t
