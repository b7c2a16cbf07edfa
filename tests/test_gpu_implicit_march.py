"""The implicit step's Jacobi sweep where its marches take more than one plane
(grids of 12 k row chunks and more): a thin channel against the oracle, with the
gates of the implicit parity tests (state within 1e-12 of max |Q|, update within
1e-10 of its own maximum), and a box whose extents leave remainders of the row
groups and of the marches, bitwise the same cut into blocks whose marches start
at other planes."""
import numpy as np
import pytest

from gpu_util import max_rel, say
from oracle import implicit as oim
from oracle import solver as osol
from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu


def test_marched_sweeps_match_the_oracle():
    from paper_1710_09995_amd.binding import Solver
    case = cases.channel_case(8, 114, 111, mach=0.7, hb=0.02).with_params(limiter_eps=1e-4, local_dt=1)
    say("marched sweeps", case.dims)
    s = Solver(case)
    s.step_implicit(1, 3, 5.0, hist=False)
    got = s.state()
    s.close()
    st = osol.setup(case.with_params(cfl=5.0))
    oim.implicit_step(st, 3, record=False)
    want = osol.interior_state(st)
    assert max_rel(got, want) <= 1e-12
    assert max_rel([g - q for g, q in zip(got, case.q0)], [w - q for w, q in zip(want, case.q0)]) <= 1e-10


@pytest.mark.parametrize("local", [0, 1])
def test_marched_sweeps_do_not_depend_on_the_cut(local):
    from paper_1710_09995_amd.binding import Solver
    box = cases.vortex_case(114, nz=111, seed=6, curvilinear=True).with_params(local_dt=local)
    split = cases.split_periodic_box(box, (2, 1, 3))
    say("marched sweeps, cut", box.dims, split.dims)
    out = []
    for c in (box, split):
        s = Solver(c)
        s.step_implicit(2, 3, 8.0, hist=False)
        out.append(s.state())
        s.close()
    W = out[0][0]
    for b, m in enumerate(split.dims):
        o = ((b % 2) * m[0], 0, (b // 2) * m[2])
        assert np.array_equal(out[1][b], W[:, o[2]:o[2] + m[2], o[1]:o[1] + m[1], o[0]:o[0] + m[0]]), b
