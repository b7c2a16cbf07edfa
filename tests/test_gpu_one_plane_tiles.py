"""GPU: one-plane tiles of the tiled kernel (kernel 0, tile_k 1) where they do not
run as bricks, FP64 inviscid flow on a grid of more than seven bricks a CU, at
ragged tile edges: state, time step, totals and max |R_rho| bitwise the simple
kernel's."""
import numpy as np
import pytest

from gpu_util import say
from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_j", [2, 4, 8])
def test_one_plane_tiles_match_the_simple_kernel(tile_j):
    from paper_1710_09995_amd.binding import Solver
    case = cases.channel_case(130, 67, 61, mach=0.7, hb=0.06, local_dt=tile_j == 4)     # 17 x 17 x 16 bricks
    out = []
    for tun in ({"kernel": 0, "tile_j": tile_j, "tile_k": 1}, {"kernel": 1, "tile_j": 4, "tile_k": 8}):
        say("one-plane tiles", tun)
        s = Solver(case, tuning=tun)
        h = s.step(2).cpu().numpy()
        s.step(9, hist=False)
        out.append((h, s.state()[0]))
        s.close()
    exact = [0, 6, 7, 8, 9, 10, 11]
    assert np.array_equal(out[0][0][:, exact], out[1][0][:, exact])
    assert np.isfinite(out[0][1]).all() and np.array_equal(out[0][1], out[1][1])
