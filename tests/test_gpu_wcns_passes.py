"""The one-pass inviscid WCNS-E-5 kernels (row runs along i, marches along j and
k), which take blocks of 32 k cells in all, at the sizes where their work is cut
unevenly: rows of eight cells, runs that end inside or at the end of a row,
chunks of one to thirty-two faces, planes, and more joined blocks than one launch
holds.  Against the oracle within 1e-12 of the largest entry (the bar of the
three-pass kernels' parity tests); bitwise between the one-pass and three-pass
kernels and between split and unsplit blocks (the same operations on every
path)."""
import numpy as np
import pytest

from gpu_util import say
from oracle import highorder as ho
from test_gpu_highorder import _smooth_state
from test_gpu_zcurvilinear import _curv_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(8, 64, 64), (9, 61, 60), (54, 25, 25), (108, 19, 16), (109, 7, 43), (118, 139, 2),
                               (256, 33, 4), (300, 5, 37), (33, 31, 33), (182, 181, 1)])
def test_one_pass_residual_matches_the_oracle(n):
    import torch
    from paper_1710_09995_amd.binding import wcns5_euler_residual_periodic
    assert n[0] * n[1] * n[2] >= 32768
    q = _smooth_state(n, seed=sum(n))
    h = (1.0 / n[0], 1.0 / n[1], 1.0 / n[2])
    say("one-pass residual", n)
    got = wcns5_euler_residual_periodic(torch.from_numpy(q).cuda(), h).cpu().numpy()
    want = ho.wcns5_euler_residual_periodic(q, h, 1.4, 0.1)
    assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want))


@pytest.mark.parametrize("n,axis,curved", [((24, 24, 24), 2, False), ((24, 24, 24), 2, True), ((64, 1, 171), 2, False),
                                           ((8, 1366, 1), 1, False)])
def test_one_pass_is_the_three_pass_path_bitwise(n, axis, curved):
    """A periodic block (three passes) and the same flow three periods long (one
    pass)."""
    import torch
    from paper_1710_09995_amd.binding import (wcns5_euler_residual_curv_periodic, wcns5_euler_residual_periodic,
                                              wcns5_metrics_periodic)
    q = torch.from_numpy(_smooth_state(n, seed=7)).cuda()
    say("one pass and three passes", n, curved)
    deep = lambda t: torch.cat([t] * 3, dim=t.dim() - 1 - axis).contiguous()
    if curved:
        Xv, P = _curv_grid(n, "wavy")
        S, J = wcns5_metrics_periodic(torch.from_numpy(Xv).cuda(), P)
        one, three = wcns5_euler_residual_curv_periodic(deep(q), deep(S), deep(J)), \
            wcns5_euler_residual_curv_periodic(q, S, J)
    else:
        h = (0.1, 0.2, 0.3)
        one, three = wcns5_euler_residual_periodic(deep(q), h), wcns5_euler_residual_periodic(q, h)
    assert torch.equal(one, deep(three))


@pytest.mark.parametrize("n,cuts", [((48, 36, 24), ([17], [8, 20], [11])), ((60, 24, 30), ([10, 25, 33], [5], [25]))])
def test_batched_blocks_match_the_unsplit_block(n, cuts):
    """12 and 16 joined blocks (two launches of up to eight a pass), down to five
    cells deep: residual, viscous terms and two RK3 steps bitwise the unsplit
    block's."""
    import torch
    from paper_1710_09995_amd.binding import (c4_viscous_add_blocks, c4_viscous_add_curv_periodic,
                                              wcns5_euler_residual_blocks, wcns5_euler_residual_curv_periodic,
                                              wcns5_metrics_periodic, wcns5_ns_steps_blocks,
                                              wcns5_ns_steps_curv_periodic)
    from test_oracle_highorder import _split_box
    Xv, P = _curv_grid(n, "wavy")
    say("batched blocks", n, cuts)
    S, J = wcns5_metrics_periodic(torch.from_numpy(Xv).cuda(), P)
    qt = torch.from_numpy(_smooth_state(n, seed=31)).cuda()
    lo, m, nbr = _split_box(n, cuts)
    sls = [(slice(o[2], o[2] + e[2]), slice(o[1], o[1] + e[1]), slice(o[0], o[0] + e[0])) for o, e in zip(lo, m)]
    qs = [qt[(slice(None),) + sl].contiguous() for sl in sls]
    Ss = [S[(slice(None), slice(None)) + sl].contiguous() for sl in sls]
    Js = [J[sl].contiguous() for sl in sls]
    same = lambda parts, whole: all(torch.equal(p, whole[(slice(None),) + sl]) for sl, p in zip(sls, parts))
    whole = wcns5_euler_residual_curv_periodic(qt, S, J)
    parts = wcns5_euler_residual_blocks(qs, Ss, Js, nbr)
    assert same(parts, whole)
    gas = (1.4, 0.72, 0.02, 0.38)
    assert same(c4_viscous_add_blocks(qs, parts, Ss, Js, nbr, *gas), c4_viscous_add_curv_periodic(qt, whole, S, J, *gas))
    step = (1e-3, 2, 1.4, 0.1, 1e-6, 0.72, 0.02, 0.38)
    assert same(wcns5_ns_steps_blocks([t.clone() for t in qs], Ss, Js, nbr, *step),
                wcns5_ns_steps_curv_periodic(qt.clone(), S, J, *step))
