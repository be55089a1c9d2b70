"""The default step variant of a single grid (no GPU needed): fast tiles from
four rounds of 2048 tiles on where at most one tile in 128 lies at the grid's
edge, whole tiles everywhere else."""
import pytest

from paper_1010_4124_amd import lbm

FAST, NT = (4, 1, 2, 1, 1, 3), (4, 18, 6, 1, 1, 0)
P, F, R, O = 0, 1, 2, 3


@pytest.mark.parametrize("nx,ny,want", [
    (2048, 2048, FAST), (4096, 4096, FAST), (2048, 1024, FAST), (1024, 2048, FAST),
    (1536, 1408, FAST), (4096, 1024, FAST), (2048, 1023, FAST), (64, 32768, FAST),
    (2048, 1020, NT), (1536, 1024, NT), (1024, 1024, NT),  # fewer rounds
    (4096, 1020, NT), (8192, 256, NT), (65536, 32, NT),    # two tile rows of few
    (2050, 2050, NT), (3000, 1000, NT), (6000, 3000, NT),  # a partial tile column
    (20000, 20000, FAST), (512, 512, (4, 18, 6, 1, 0, 0)), (256, 256, (2, 18, 6, 1, 0, 0)),
    (400, 4, (1, 18, 6, 1, 0, 0)), (1, 1, (1, 18, 6, 1, 0, 0)), (1, 900_000_000, NT)])
def test_periodic_x(nx, ny, want):
    v = lbm.lib().lbmi_default_variant(nx, ny, P)
    assert lbm.lbm_step_variant_info(v) == want


@pytest.mark.parametrize("bc", [F, R, O])
@pytest.mark.parametrize("nx,ny", [(2048, 2048), (2048, 1536), (4096, 4096), (1024, 4096)])
def test_other_x_sides_take_whole_tiles(nx, ny, bc):
    """The first and last tile columns are at the edge there."""
    assert lbm.lbm_step_variant_info(lbm.lib().lbmi_default_variant(nx, ny, bc)) == NT
