"""GPU: blocks of one to seven cells along i, alone and joined to larger ones, take
the same one-pass inviscid WCNS-E-5 kernels as any other: bitwise the three-pass
path, and bitwise the unsplit block.  Blocks whose marches take chunks of one and
two cells, with remainders: within 1e-12 of the oracle's largest entry."""
import numpy as np
import pytest

from gpu_util import say
from oracle import highorder as ho
from test_gpu_highorder import _smooth_state
from test_gpu_zcurvilinear import _curv_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,curved", [((1, 40, 50), False), ((2, 30, 31), True), ((3, 26, 25), False),
                                      ((5, 20, 20), True), ((7, 17, 16), False), ((7, 31, 9), True),
                                      ((12, 13, 13), True), ((100, 3, 6), True), ((11, 11, 11), False)])
def test_narrow_rows_are_the_three_pass_path_bitwise(n, curved):
    """A periodic block (three passes along j and k) and the same flow three periods
    deep (one pass)."""
    import torch
    from paper_1710_09995_amd.binding import (wcns5_euler_residual_curv_periodic, wcns5_euler_residual_periodic,
                                              wcns5_metrics_periodic)
    assert n[0] * n[1] * n[2] < 2048 <= 3 * n[0] * n[1] * n[2]
    say("narrow rows", n, curved)
    q = torch.from_numpy(_smooth_state(n, seed=3)).cuda()
    deep = lambda t: torch.cat([t] * 3, dim=t.dim() - 3).contiguous()
    if curved:
        Xv, P = _curv_grid(n, "wavy")
        S, J = wcns5_metrics_periodic(torch.from_numpy(Xv).cuda(), P)
        one = wcns5_euler_residual_curv_periodic(deep(q), deep(S), deep(J))
        three = wcns5_euler_residual_curv_periodic(q, S, J)
    else:
        h = (0.1, 0.2, 0.3)
        one, three = wcns5_euler_residual_periodic(deep(q), h), wcns5_euler_residual_periodic(q, h)
    assert torch.equal(one, deep(three))


@pytest.mark.parametrize("n,cuts", [((45, 40, 24), ([5, 40], [17], [])), ((37, 33, 32), ([5, 11, 30], [], [9]))])
def test_narrow_blocks_among_others_match_the_unsplit_block(n, cuts):
    import torch
    from paper_1710_09995_amd.binding import (wcns5_euler_residual_blocks, wcns5_euler_residual_curv_periodic,
                                              wcns5_metrics_periodic)
    from test_oracle_highorder import _split_box
    Xv, P = _curv_grid(n, "wavy")
    say("narrow blocks", n, cuts)
    S, J = wcns5_metrics_periodic(torch.from_numpy(Xv).cuda(), P)
    q = torch.from_numpy(_smooth_state(n, seed=5)).cuda()
    lo, m, nbr = _split_box(n, cuts)
    sls = [(slice(o[2], o[2] + e[2]), slice(o[1], o[1] + e[1]), slice(o[0], o[0] + e[0])) for o, e in zip(lo, m)]
    parts = wcns5_euler_residual_blocks([q[(slice(None),) + sl].contiguous() for sl in sls],
                                        [S[(slice(None), slice(None)) + sl].contiguous() for sl in sls],
                                        [J[sl].contiguous() for sl in sls], nbr)
    whole = wcns5_euler_residual_curv_periodic(q, S, J)
    for part, sl in zip(parts, sls):
        assert torch.equal(part, whole[(slice(None),) + sl])


@pytest.mark.parametrize("n", [(40, 41, 43), (64, 43, 16), (33, 31, 33), (100, 19, 18)])
def test_short_chunks_match_the_oracle(n):
    import torch
    from paper_1710_09995_amd.binding import wcns5_euler_residual_periodic
    q = _smooth_state(n, seed=sum(n))
    h = (1.0 / n[0], 1.0 / n[1], 1.0 / n[2])
    say("short chunks", n)
    got = wcns5_euler_residual_periodic(torch.from_numpy(q).cuda(), h).cpu().numpy()
    want = ho.wcns5_euler_residual_periodic(q, h, 1.4, 0.1)
    assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want))
