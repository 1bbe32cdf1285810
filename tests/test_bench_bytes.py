"""CPU check of the byte count behind the benchmark's optical rate: what each
launch of a CG iteration reads and writes (cg_mg.hpp), 8 bytes a value."""
import pytest


def test_optical_iteration_moves_what_its_launches_move():
    import bench
    stencil = 4
    dir_q = 2 + stencil + 2                       # z, p; stencil; p, q
    update = 5 + stencil + 2 + 1 / 4              # x, p, r, q, 1/d; stencil; x, r and the coarse right-hand side
    post = 2 + 1 / 4 + stencil + 1                # r, 1/d and the coarse correction; stencil; z
    restrict = 2 + stencil + 1 / 4                # b, 1/d; stencil; the coarse right-hand side
    coarse = sum(4.0 ** -level for level in range(1, 30))
    assert bench.OPT_MOVED_BYTES_PER_NODE_ITER == pytest.approx(8 * (dir_q + update + post + coarse * (restrict + post)))
