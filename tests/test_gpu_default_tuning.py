"""GPU: the default tuning's line between bricks and the plane-ring kernel: seven
8 x 4 x 4 bricks a CU, 13 with FP32 flux (blocks of 128 bricks and more); on either
side the state is bitwise the simple kernel's."""
import numpy as np
import pytest

from gpu_util import say
from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("viscous", [0, 1])
@pytest.mark.parametrize("fp32", [0, 1])
def test_bricks_up_to_their_line(fp32, viscous):
    import torch
    from paper_1710_09995_amd.binding import Solver
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    most = (13 if fp32 else 7) * cu
    for bricks in (most, most + 1):
        # one layer of bricks a few cells deep, and one brick more for the far side
        dims = [(8 * (bricks // 8), 31, 3)] + ([(8, 4, 4)] if bricks % 8 else [])
        one = [cases.bump_ns_case(*d, seed=2, reynolds=5e3, viscous=viscous) for d in dims]
        from dataclasses import replace
        conns = [replace(k, blk=b, nbr=b) for b, c in enumerate(one) for k in c.conns]
        bcs = [replace(k, blk=b) for b, c in enumerate(one) for k in c.bcs]
        case = cases.Case("line", one[0].params, [c.dims[0] for c in one], [c.nodes[0] for c in one], conns, bcs,
                          [c.q0[0] for c in one]).with_params(flux_fp32=fp32)
        out = []
        for tun in (None, {"kernel": 1, "tile_j": 4, "tile_k": 8}):
            s = Solver(case, tuning=tun)
            if tun is None:
                t = s.get_tuning()
                say("default tuning", fp32, viscous, bricks, t)
                assert ((t["kernel"], t["tile_k"]) == (0, 1)) == (bricks == most) and t["kernel"] in (0, 2)
            s.step(2, hist=False)
            out.append(s.state())
            s.close()
        assert all(np.isfinite(a).all() and np.array_equal(a, b) for a, b in zip(*out))
