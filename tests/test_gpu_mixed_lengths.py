"""One launch over problems of every line length: the kernels that hold all
lengths give the bits of each length's own kernels, lossy and lossless, with
short lengths (run-time plans) among them."""
import numpy as np
import pytest

import qpat_inputs as qi
from test_gpu_lengths import N, T, problem, q  # noqa: F401  (q is the fixture)

pytestmark = pytest.mark.gpu

LENGTHS = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024)


@pytest.mark.parametrize("a0", [0.75, 0.0])
@pytest.mark.parametrize("across", ["rows", "columns"])
def test_all_lengths_in_one_launch_bitwise(q, a0, across):
    probs = []
    for i, n in enumerate(LENGTHS):
        other = (16, 24, 32, 48)[i % 4]
        nx, ny = (n, other) if across == "rows" else (other, n)
        prm, c0, rho0, _ = problem(nx, ny, 7 + i % 3, a0, ns=5)
        prm["pml_size"] = 2
        probs.append((q.Plan(prm, c0, rho0), T(qi.gaussian_field((ny, nx), 30 + i))))
    xs = [x for _, x in probs]
    refs = [(N(plan.forward(x)), N(plan.jtjv(x))) for plan, x in probs]
    bat = q.Batch([plan for plan, _ in probs])
    assert bat.schedule() == 0
    for (d, g), db, gb in zip(refs, bat.forward(xs), bat.jtjv(xs)):
        assert np.array_equal(N(db), d) and np.array_equal(N(gb), g)
