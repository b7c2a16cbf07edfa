"""GPU: the implicit step on blocks of very unequal sizes in one context.  The
sweep's workgroups are numbered over the blocks: independent channels side by
side take bitwise the steps that each takes alone."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_util import say
from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [[(5, 3, 2), (128, 80, 80), (64, 4, 9), (70, 5, 33)],
                                  [(65, 9, 2), (2, 2, 2), (2, 2, 2), (12, 17, 3), (4, 4, 4)]])
def test_unequal_blocks_step_as_each_alone(dims):
    from paper_1710_09995_amd.binding import Solver
    one = [cases.channel_case(*d, mach=0.6, hb=0.05) for d in dims]      # local steps: nothing couples the blocks
    conns = [replace(k, blk=b, nbr=b) for b, c in enumerate(one) for k in c.conns]
    bcs = [replace(k, blk=b) for b, c in enumerate(one) for k in c.bcs]
    together = cases.Case("channels", one[0].params, [c.dims[0] for c in one], [c.nodes[0] for c in one], conns, bcs,
                          [c.q0[0] for c in one])

    def run(case):
        s = Solver(case)
        s.step_implicit(2, 3, 8.0, hist=False)
        q = s.state()
        s.close()
        return q
    say("unequal blocks", dims)
    for got, c in zip(run(together), one):
        want = run(c)[0]
        assert np.isfinite(want).all() and np.array_equal(got, want)
