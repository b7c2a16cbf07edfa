"""GPU: blocks of one to seven cells along i, alone and joined to larger ones, take
the same one-pass inviscid WCNS-E-5 kernels as any other: bitwise the three-pass
path, and bitwise the unsplit block."""
import pytest

from gpu_util import say
from test_gpu_highorder import _smooth_state
from test_gpu_zcurvilinear import _curv_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,curved", [((1, 128, 100), False), ((2, 90, 70), True), ((3, 99, 101), False),
                                      ((5, 64, 64), True), ((7, 61, 60), False), ((7, 31, 65), True)])
def test_narrow_rows_are_the_three_pass_path_bitwise(n, curved):
    """A periodic block (three passes) and the same flow three periods deep (one pass)."""
    import torch
    from paper_1710_09995_amd.binding import (wcns5_euler_residual_curv_periodic, wcns5_euler_residual_periodic,
                                              wcns5_metrics_periodic)
    assert n[0] * n[1] * n[2] < 32768 <= 3 * n[0] * n[1] * n[2]
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
