"""3-D axes of 18 to 63 points, transformed as matrix products, against the
FP64 oracle (oracle/kspace3d.py) at the edges of the length classes (18, 31 |
32, 33 | 34, 49 | 50, 63), of the range (17, 64) and mixed with axes that take
the FFT stages.

Tolerances, from u = 2^-24: a transform of n white values sums n/2 folded
pairs, each rounded at the size of the running sum: relative L2 error at most
about u sqrt(n).  An operator is six of them, and a first derivative weighs the
(white) error of the first three with a symbol whose peak is sqrt(3) of its
rms: 3 (1 + sqrt(3)) u sqrt(63) = 3.9e-6.  Sensor data and gradients add the
time steps' 1e-5 each at most over the few iterates here."""
import numpy as np
import pytest

import qpat_inputs as qi
from oracle import kspace3d as K3
from test_gpu_3d import N, T, problem, q, rel  # noqa: F401  (q is the fixture)

pytestmark = pytest.mark.gpu

TOL_OP = 3.9e-6
TOL = 2e-5

SHAPES = [  # nx, ny, nz
    (18, 31, 32), (32, 33, 18), (33, 18, 34), (34, 50, 49), (49, 63, 50), (50, 49, 63), (63, 34, 31),
    (31, 32, 33), (63, 63, 63),
    (17, 20, 21), (64, 19, 20), (20, 17, 19), (22, 19, 64), (19, 49, 49), (49, 49, 48),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_spectral_operators(q, shape):
    nx, ny, nz = shape
    prm, c0, rho0, _ = problem(nx, ny, nz, 4)
    plan = q.Plan3D(prm, c0, rho0)
    o = K3.Operators(prm, c0, rho0)
    f = qi.gaussian_field((nz, ny, nx), 7)
    ref = f.astype(np.float32).astype(np.float64)
    for op, m in [("dx+", o.mp[0]), ("dy-", o.mm[1]), ("dz+", o.mp[2]), ("ydis", o.ldis), ("yabs", o.labs)]:
        assert rel(N(plan.apply(op, T(f))), o.spectral(m, ref)) <= TOL_OP, op


@pytest.mark.parametrize("a0", [0.0, 0.75])
@pytest.mark.parametrize("shape", SHAPES)
def test_forward_adjoint(q, shape, a0):
    nx, ny, nz = shape
    prm, c0, rho0, p0 = problem(nx, ny, nz, 6, alpha0_db=a0, pml=3)
    plan = q.Plan3D(prm, c0, rho0)
    ops = K3.Operators(prm, c0, rho0)
    x = qi.gaussian_field(p0.shape, 11).astype(np.float32)
    r = qi.gaussian_field((6, prm["sensor_xyz"].shape[0]), 12).astype(np.float32)
    assert rel(N(plan.forward(T(x))), K3.forward(prm, c0, rho0, x.astype(np.float64), ops=ops)) <= TOL
    assert rel(N(plan.adjoint(T(r))), K3.adjoint(prm, c0, rho0, r.astype(np.float64), ops=ops)) <= TOL


@pytest.mark.parametrize("shape", [(63, 20, 19), (50, 33, 63), (33, 49, 49), (32, 18, 33)])
def test_batch_and_shape_bitwise(q, shape):
    """Matrices in LDS (many blocks) and in registers, any rows, columns and
    threads per block, and captured launches: the same bits."""
    import torch
    nx, ny, nz = shape
    prm, c0, rho0, p0 = problem(nx, ny, nz, 5)
    plan = q.Plan3D(prm, c0, rho0)
    xs = qi.gaussian_field((12,) + p0.shape, 41)
    r = qi.gaussian_field((12, 5, 9), 42)
    d, g = N(plan.forward(T(xs))), N(plan.adjoint(T(r)))
    for b in (0, 11):
        assert np.array_equal(N(plan.forward(T(xs[b]))), d[b])
        assert np.array_equal(N(plan.adjoint(T(r[b]))), g[b])
    for tiles in [(2, 1, 64, 64), (18, 3, 512, 128), (16, 2, 128, 1024)]:
        plan.set_tiles(*tiles)
        assert np.array_equal(N(plan.forward(T(xs[:2]))), d[:2]), tiles
        assert np.array_equal(N(plan.adjoint(T(r[:2]))), g[:2]), tiles
    plan.set_graph(True)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for _ in range(3):
            dd, gg = plan.forward(T(xs), stream=s), plan.adjoint(T(r), stream=s)
            s.synchronize()
            assert np.array_equal(N(dd), d)
            assert np.array_equal(N(gg), g)
