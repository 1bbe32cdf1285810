"""The automatic launch shape of 3-D plans whose axes are transformed as matrix
products: what tiles() reports is what a single vector's launches use, on both
sides of each line of the rule, and fixing it changes nothing."""
import numpy as np
import pytest

import qpat_inputs as qi
from test_gpu_3d import N, T, problem, q  # noqa: F401  (q is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tiles", [
    ((18, 14, 12), (8, 1, 256, 1024)),   # matrix rows, FFT planes
    ((64, 20, 24), (8, 1, 256, 256)),    # FFT rows, matrix planes
    ((20, 32, 63), (8, 1, 256, 256)),    # 252 blocks of 8 lines: one per CU
    ((20, 33, 63), (16, 1, 256, 256)),   # 260
    ((53, 53, 53), (16, 1, 256, 256)),
    ((49, 49, 49), (16, 1, 256, 1024)),  # FFT planes
])
def test_reported_shape_is_used(q, shape, tiles):  # noqa: F811
    nx, ny, nz = shape
    prm, c0, rho0, p0 = problem(nx, ny, nz, 4)
    plan = q.Plan3D(prm, c0, rho0)
    assert plan.tiles() == tiles
    x = T(qi.gaussian_field(p0.shape, 61))
    auto = N(plan.jtjv(x))
    plan.set_tiles(*plan.tiles())
    assert plan.tiles() == tiles
    assert np.array_equal(N(plan.jtjv(x)), auto)
