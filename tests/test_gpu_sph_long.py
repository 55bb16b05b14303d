"""The SPH step on long grids (more than 256 cells along x, more than along y),
whose cell columns run along x: against the FP64 all-pairs oracle, with the
inputs, checks and tolerances of test_gpu_sph_cells.py.  257 and 256 cells lie
on the two sides of the rule."""
import pytest

import test_gpu_sph_cells as cells

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gx,gy,n,kernel", [(257, 3, 900, 0), (5000, 3, 1300, 1), (600, 7, 1500, 0), (257, 59, 1100, 1),
                                            (256, 59, 1100, 0), (3, 600, 700, 1)])
def test_long_grids_match_oracle(gx, gy, n, kernel):
    cells.test_cell_tiles_match_oracle(gx, gy, n, False, kernel)
