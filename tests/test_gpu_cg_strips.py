"""The CG solves on strips, whose blocks have tiles of their own: at the widths
and heights where the tile changes, at remainders, and with more tiles than
blocks; the references and bounds are those of the other grids."""
import pytest

import test_gpu_cg_levels as levels
from test_gpu_optical import q  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(2, 1025), (4, 1150), (5, 1027), (12, 1100), (13, 1030), (1025, 2), (1150, 4), (1030, 5),
                                   (2, 131300), (131300, 2)])
def test_tv(q, nx, ny):  # noqa: F811
    levels.test_tv_residual(q, nx, ny)


@pytest.mark.parametrize("nx,ny", [(1, 1024), (4, 1100), (11, 1026), (12, 1027), (1024, 1), (1027, 3), (1030, 4)])
def test_optical(q, nx, ny):  # noqa: F811
    levels.test_optical_batch_and_graph(q, nx, ny)
