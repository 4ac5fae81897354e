"""The bytes that the benchmark credits a periodic relaxing-TVD step with: what its
launches have to move, the state read and written once by each (CPU only)."""
import bench


def test_two_launches_on_large_grids():
    # 256^3 and 1024^3: x and y together, then z
    for g in (16, 64):
        assert bench.rtvd_launches(g) == 2
        assert bench.rtvd_bytes_per_cell(g, 4) == 80 and bench.rtvd_bytes_per_cell(g, 8) == 160


def test_three_launches_on_small_grids():
    for g in (1, 2, 4, 8):
        assert bench.rtvd_launches(g) == 3
        assert bench.rtvd_bytes_per_cell(g, 4) == 120
