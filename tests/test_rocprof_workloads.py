"""CPU test: which workload of a bench.py run a traced two-step launch is
attributed to, by its template arguments (lattice, mode, passes over the
interior, with the outer rows, phi values per thread, threads, waves)."""
import pytest

from paper_2208_09267_amd import rocprof_summary as rs


@pytest.mark.parametrize("name,grid,workload", [
    ("fused2_kernel<D3Q19, 0, 1, 2, 2, 512, 2>", 131072, "D3Q19 128^3"),   # 4 rows of 128
    ("fused2_kernel<D3Q19, 0, 1, 2, 4, 512, 2>", 131072, "D3Q19 256^3"),   # 2 rows of 256
    ("fused2_kernel<D3Q19, 1, 1, 2, 4, 512, 4>", 131072, "D3Q19 256^3"),
    ("fused2_kernel<D3Q19, 3, 1, 2, 2, 1024, 4>", 262144, "D3Q19 256^3"),
    ("fused2_kernel<D3Q27, 0, 1, 2, 2, 512, 2>", 131072, "D3Q27 256^3"),
    ("fused2_kernel<D3Q27, 1, 2, 3, 4, 512, 2>", 131072, "D3Q27 256^3"),
    ("fused2_kernel<D3Q19, 0, 1, 2, 4, 1024, 2>", 131072, None)])
def test_two_step_launches_are_attributed_by_their_tile(name, grid, workload):
    assert rs._workload(name, grid)[0] == workload
