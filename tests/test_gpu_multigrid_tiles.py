"""GPU: V-cycles with every level, or the coarse levels alone, on each stage kernel
and tile size: bricks, the tiled kernel's marching tiles (whose stages apply a
level's forcing themselves), the simple kernel and the plane-ring kernel's two
sizes give bitwise the same states and history rows (but for the finest level's L2
norms, summed in tile order)."""
import numpy as np
import pytest

from gpu_util import say
from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu

TUNINGS = [(0, 4, 1), (0, 4, 2), (0, 2, 2), (0, 8, 4), (0, 4, 16), (2, 8, 4), (2, 4, 4), (2, 4, 3)]


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("name", ["channel", "bump_ns"])
def test_levels_on_every_kernel_and_tile_size(name, fp32):
    from paper_1710_09995_amd.binding import Multigrid, Solver
    case = cases.channel_case(72, 24, 20, mach=0.7, hb=0.06) if name == "channel" else \
        cases.bump_ns_case(40, 24, 12, seed=2, reynolds=5e3)
    case = case.with_params(flux_fp32=fp32)
    exact = [0, 6, 7, 8, 9, 10, 11]

    def run(tun, first):
        s = Solver(case)
        mg = Multigrid(s, 3, 1, 2)
        for lv in mg.levels[first:]:
            lv.set_tuning(kernel=tun[0], tile_j=tun[1], tile_k=tun[2])
        h = mg.cycles(3).cpu().numpy()
        q = s.state()
        mg.close()
        s.close()
        return h, q
    ref = run((1, 4, 8), 0)
    assert all(np.isfinite(q).all() for q in ref[1])
    for tun in TUNINGS:
        for first in (0, 1):
            say("multigrid levels", name, fp32, tun, first)
            h, q = run(tun, first)
            assert np.array_equal(h[:, exact], ref[0][:, exact]), tun
            assert all(np.array_equal(a, b) for a, b in zip(q, ref[1])), tun
