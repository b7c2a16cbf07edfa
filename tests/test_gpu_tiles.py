"""GPU: the plane-ring kernel's tile shapes (64 x 8, 32 x 16, 32 x 8, 16 x 16)
at the edges of their tiles and of their runs of planes.  A face flux does not
depend on the tile that computed it, so the state after two steps, the time
step, the totals and max |R_rho| are bitwise those of the simple per-cell
kernel."""
import numpy as np
import pytest

from gpu_util import say
from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu

# one cell short of, at and past the tiles' extents; thin blocks; k runs with and without remainder
DIMS = [(16, 16, 5), (17, 15, 7), (31, 17, 4), (33, 16, 9), (64, 8, 3), (65, 9, 11), (48, 33, 6), (4, 4, 4)]


def _run(case, tuning):
    from paper_1710_09995_amd.binding import Solver
    s = Solver(case, tuning=tuning)
    h = s.step(2, hist=True).cpu().numpy()
    q = s.state()
    s.close()
    return h, q


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("viscous", [0, 1])
@pytest.mark.parametrize("dims", DIMS)
def test_ring_tile_shapes_match_the_simple_kernel(dims, viscous, fp32):
    case = cases.bump_ns_case(*dims, seed=5, reynolds=5e3, viscous=viscous).with_params(flux_fp32=fp32)
    h0, q0 = _run(case, {"kernel": 1, "tile_j": 4, "tile_k": 8})
    for tj, tk in ((8, 32), (8, 3), (4, 4), (4, 2)):
        say("ring tiles", dims, viscous, fp32, tj, tk)
        h, q = _run(case, {"kernel": 2, "tile_j": tj, "tile_k": tk})
        for a, b in zip(q, q0):
            assert np.array_equal(a, b)
        exact = [0, 6, 7, 8, 9, 10, 11]
        assert np.array_equal(h[:, exact], h0[:, exact])
