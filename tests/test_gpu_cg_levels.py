"""The multigrid-preconditioned CG of the optical and TV solves where its launch
plan changes: a lone bottom level, all levels below 0 in one workgroup's LDS,
one to three tiled levels above it, strips, tile remainders, more tiles than
blocks; batched, single and captured runs to the bit.

TV: the residual of the returned z against the FP64 matrix M.  z is rounded to
FP32, which moves M z by at most 2^-24 |M| |z| elementwise; the solver stops at
tol |r|.  Optical: H against the oracle's direct solve.  The solve stops at
1e-10 of the right-hand side and H is FP32 (6e-8); the Robin problem's condition
number on these meshes is below 1e5: 1e-5."""
import numpy as np
import pytest

from oracle import optical as O
from oracle import recon as R
from test_gpu_optical import N, T, oracle_G, q, rel, tissue  # noqa: F401  (q is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 2), (31, 33), (64, 64), (70, 69), (98, 66), (129, 131), (2000, 3),
                                   (2, 700), (900, 700)])
def test_tv_residual(q, nx, ny):
    rng = np.random.default_rng(nx * ny)
    B, beta, gamma, tol = 3, 1e-2, 1e-1, 1e-8
    xs = rng.standard_normal((B, ny, nx)).astype(np.float32)
    r = rng.standard_normal((B, ny, nx)).astype(np.float32)
    tv = q.TV(nx, ny, B)
    tv.set_weights(T(xs), beta)
    z, it = tv.solve(T(r), gamma, tol=tol, max_iter=5000)
    assert 0 < it < 5000
    D = R.tv_difference(ny, nx)
    for b in range(B):
        M = R.tv_matrix(D, xs[b].astype(float), beta, gamma).tocsr()
        zb, rb = N(z)[b].ravel(), r[b].astype(float).ravel()
        bound = 2.0 ** -24 * np.linalg.norm(abs(M) @ np.abs(zb)) + tol * np.linalg.norm(rb)
        assert np.linalg.norm(M @ zb - rb) <= bound
    tv.close()
    one = q.TV(nx, ny, 1)
    one.set_weights(T(xs[2]), beta)
    # the batch stops with its slowest field: the same iterations, the same bits
    z1, it1 = one.solve(T(r[2]), gamma, tol=tol, max_iter=5000)
    assert it1 <= it
    assert np.array_equal(N(z1).ravel(), N(z)[2].ravel())
    one.close()


@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 1), (32, 31), (47, 49), (64, 64), (97, 65), (130, 129), (1, 300), (500, 2)])
def test_optical_batch_and_graph(q, nx, ny):
    import torch
    B, dx = 3, 1e-4
    m = O.Mesh(nx, ny, dx)
    kap, mu = tissue(m, B, 5)
    cur = np.array([[1.0, 0.0, 0.5, 0.0], [0.0, 2.0, 0.0, 1.0], [1.0, 1.0, 0.0, 0.0]])
    opt = q.Optical(nx, ny, dx, B)
    H = N(opt.forward(T(kap), T(mu), cur))
    for b in range(B):
        assert rel(H[b], O.forward(m, kap[b], mu[b], oracle_G(m, cur[b]))[0]) <= 1e-5
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for b in (0, 2):
            H1 = opt.forward(T(kap[b]), T(mu[b]), cur[b], stream=s)
            s.synchronize()
            assert np.array_equal(N(H1).ravel(), H[b])
