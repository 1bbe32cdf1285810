"""What the matrix-product transforms lose on smooth fields in the middle of the
grid (the phantoms of the benchmark), where a derivative's error is that of the
high wavenumbers: differences of large terms, so that the order of the sums counts.

Bound: the error of d/dx whose forward x transform is one FP32 sum per output in
growing order of the distance from the edge (emulated below; the order the prime
FFT stages use), and, for the other transforms, the error that the same operator
has on white noise, where order does not matter; 15% for two samples of noise."""
import numpy as np
import pytest

import qpat_inputs as qi
from oracle import kspace3d as K3
from test_gpu_3d import N, T, problem, q, rel  # noqa: F401  (q is the fixture)

pytestmark = pytest.mark.gpu


def rfft_ascending(f):
    """rfft along x of an FP32 field, each output one sum with fused multiply-adds."""
    n = f.shape[-1]
    k = np.arange(n // 2 + 1)
    a = np.repeat(f[..., :1], len(k), -1)
    b = np.zeros_like(a)
    for r in range(1, n // 2 + 1):
        w, m = 0.5 if 2 * r == n else 1.0, 2 * np.pi * (k * r % n) / n
        e = (f[..., r] + f[..., n - r])[..., None].astype(np.float64)
        o = (f[..., r] - f[..., n - r])[..., None].astype(np.float64)
        a = (e * np.float32(w * np.cos(m)) + a).astype(np.float32)
        b = (o * np.float32(w * np.sin(m)) + b).astype(np.float32)
    return a.astype(np.float64) - 1j * b


@pytest.mark.parametrize("n", [31, 37, 47, 53, 59, 61])
def test_derivative_of_blobs(q, n):  # noqa: F811
    prm, c0, rho0, _ = problem(n, n, n, 4)
    plan = q.Plan3D(prm, c0, rho0)
    o = K3.Operators(prm, c0, rho0)
    f = qi.blobs3d(n, n, n, n).astype(np.float32)
    ik = 2j * np.pi * np.fft.rfftfreq(n)
    exact = np.fft.irfft(ik * np.fft.rfft(f.astype(np.float64)), n)
    forward = rel(np.fft.irfft(ik * rfft_ascending(f), n), exact)
    w = qi.gaussian_field((n, n, n), 7).astype(np.float32)

    def error(field):
        return rel(N(plan.apply("dx+", T(field))), o.spectral(o.mp[0], field.astype(np.float64)))

    assert error(f) <= 1.15 * np.hypot(forward, error(w))
