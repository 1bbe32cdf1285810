"""Line lengths with pass kernels of their own, at the sizes where a plan, a
fused stage or a storage tile can go wrong: every length as rows and as
columns against the FP64 oracle, and bit for bit across launch shapes (row
tiles that do and do not divide the first-stage stride of the column pass),
batch sizes (global or LDS twiddles) and a launch over several lengths."""
import numpy as np
import pytest

import qpat_inputs as qi
from oracle import kspace as K

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_11685_amd as q
    return q


def T(x):
    import torch
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float32, device="cuda")


def N(t):
    return t.detach().double().cpu().numpy()


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def problem(nx, ny, nt, a0, ns=17):
    c0, rho0 = qi.medium(ny, nx, nx, ny + 1, sigma_cells=max(2.0, min(nx, ny) / 16))
    dx = 1e-4
    prm = qi.make_params(nx, ny, dx, 0.3 * dx / c0.max(), nt, c0.max(),
                         qi.ring_sensors(ns, 0.1 * min(nx, ny), dx, phase=0.05), pml_size=4, alpha0_db=a0)
    return prm, c0, rho0, qi.blobs(ny, nx, 5, count=4, radius_cells=0.2 * min(nx, ny))


# relative L2 of FP32 solves of a few dozen steps: the suite's bar on data and gradients
@pytest.mark.parametrize("nx,ny", [(32, 48), (48, 32), (64, 96), (96, 64), (192, 768), (768, 192), (384, 24), (12, 384)])
@pytest.mark.parametrize("a0", [0.75, 0.0])
def test_every_length_matches_oracle(q, nx, ny, a0):
    nt = 24
    prm, c0, rho0, p0 = problem(nx, ny, nt, a0)
    plan = q.Plan(prm, c0, rho0)
    ops = K.Operators(prm, c0, rho0)
    r = qi.gaussian_field((nt, 17), 3)
    assert rel(N(plan.forward(T(p0))), K.forward(prm, c0, rho0, p0, ops=ops)) <= 1e-4
    assert rel(N(plan.adjoint(T(r))), K.adjoint(prm, c0, rho0, r, ops=ops)) <= 1e-4


@pytest.mark.parametrize("n,shapes", [
    (32, [(2, 1, 64, 64), (8, 4, 64, 128), (32, 16, 512, 512)]),
    (48, [(2, 1, 64, 64), (16, 8, 256, 256), (8, 2, 512, 128)]),
    (64, [(2, 1, 64, 64), (64, 4, 512, 512), (16, 32, 128, 512)]),
    (96, [(2, 1, 64, 64), (32, 16, 512, 512), (16, 2, 256, 64)]),
    (192, [(2, 1, 64, 64), (16, 4, 512, 256), (8, 8, 256, 512)]),
    (384, [(2, 1, 128, 128), (8, 4, 512, 512), (4, 2, 256, 512)]),
    (768, [(2, 1, 256, 256), (4, 2, 512, 512)]),
])
def test_length_bitwise_over_shapes_and_batches(q, n, shapes):
    nt = 14
    for a0 in (0.75, 0.0):
        prm, c0, rho0, _ = problem(n, n, nt, a0)
        plan = q.Plan(prm, c0, rho0)
        nb = 2 * (512 // (n // 2) + 1) if n < 512 else 5   # more than two blocks per CU at two rows a block
        x = T(np.stack([qi.smooth_noise(n, n, 2.0, 70 + b) for b in range(nb)]))
        r = T(qi.gaussian_field((nb, nt, 17), 71))
        ref = None
        for shape in shapes:
            plan.set_tiles(*shape)
            one = (N(plan.forward(x[1])), N(plan.adjoint(r[1])))
            many = (N(plan.forward(x))[1], N(plan.adjoint(r))[1])
            ref = ref or one
            for a, b in ((one, ref), (many, ref)):
                assert all(np.array_equal(u, v) for u, v in zip(a, b)), (shape, a0)


def test_launch_over_several_lengths_bitwise(q):
    probs = []
    for nx, ny in ((192, 96), (384, 48), (48, 384), (768, 32)):
        prm, c0, rho0, p0 = problem(nx, ny, 12, 0.75)
        probs.append((q.Plan(prm, c0, rho0), T(p0)))
    xs = [x for _, x in probs]
    refs = [N(plan.jtjv(x)) for plan, x in probs]
    bat = q.Batch([plan for plan, _ in probs])
    for schedule in (0, 1):
        bat.set_schedule(schedule)
        for ref, g in zip(refs, bat.jtjv(xs)):
            assert np.array_equal(N(g), ref)


@pytest.mark.parametrize("nx,ny,b", [(64, 64, 40), (1024, 64, 9), (64, 1024, 9), (192, 256, 24), (12, 8, 3), (512, 512, 3)])
def test_shape_chosen_per_batch_size_is_bitwise(q, nx, ny, b):
    """Until a shape is set, a launch takes one chosen from its vector count."""
    prm, c0, rho0, _ = problem(nx, ny, 10, 0.75, ns=5)
    prm["pml_size"] = 3
    plan = q.Plan(prm, c0, rho0)
    x = T(qi.gaussian_field((b, ny, nx), 6))
    many = N(plan.jtjv(x))
    for i in (0, b - 1):
        assert np.array_equal(N(plan.jtjv(x[i])), many[i])
    one = plan.tiles()
    plan.set_tiles(*one)               # fixed from here on, the same shape for every count
    assert plan.tiles() == one
    assert np.array_equal(N(plan.jtjv(x)), many)


def test_launch_sequence_per_size_bitwise(q):
    """One launch sequence per grid size: groups of one problem (the shape of a
    single vector), of a few (two rows, one column a block) and, of 1024-point
    lines, of more blocks than four per CU along one axis."""
    import torch
    probs = []
    for i, (nx, ny) in enumerate([(96, 96), (64, 64), (64, 64)] + [(32, 1024)] * 3 + [(1024, 32)] * 3):
        prm, c0, rho0, _ = problem(nx, ny, 8 + i % 3, 0.75)
        probs.append((q.Plan(prm, c0 * (1 - 0.005 * i), rho0 * (1 + 0.005 * i)), T(qi.gaussian_field((ny, nx), 20 + i))))
    xs = [x for _, x in probs]
    refs = [N(plan.jtjv(x)) for plan, x in probs]
    bat = q.Batch([plan for plan, _ in probs])
    bat.set_schedule(1)
    for ref, g in zip(refs, bat.jtjv(xs)):
        assert np.array_equal(N(g), ref)
    bat.set_graph(True)
    s = torch.cuda.Stream()
    for _ in range(2):
        out = bat.jtjv(xs, stream=s)
        s.synchronize()
        for ref, g in zip(refs, out):
            assert np.array_equal(N(g), ref)
