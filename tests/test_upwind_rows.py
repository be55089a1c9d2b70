"""Which kernel an upwind step takes (no GPU needed): whole tiles of 1, 2 or 4
rows, and one thread per cell (0) on tall grids of a few columns only."""
import pytest

from paper_1010_4124_amd import lbm


@pytest.mark.parametrize("nx,ny,first,second", [
    (400, 4, 1, 1), (4, 400, 1, 1), (64, 700, 2, 2), (2048, 2048, 4, 4), (100_000, 3, 4, 4),
    (1, 8000, 4, 4), (1, 16_000, 0, 0), (4, 40_000, 0, 0), (8, 480_000, 0, 4), (7, 480_000, 0, 0),
    (12, 480_000, 0, 4), (14, 480_000, 4, 4), (16, 16_000, 4, 4), (64, 200_000, 4, 4),
    (65, 500_000, 4, 4), (1, 900_000_000, 0, 0)])
def test_rows(nx, ny, first, second):
    rows = lbm.lib().lbmi_upwind_rows
    assert (rows(lbm.UPWIND1, nx, ny), rows(lbm.UPWIND2, nx, ny)) == (first, second)
