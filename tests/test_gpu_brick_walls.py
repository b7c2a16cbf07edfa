"""GPU: every boundary kind on every face of a block whose stages run as bricks and
form their ghost states themselves (inviscid flow): state, time step, totals and
max |R_rho| bitwise the simple kernel's, whose ghost cells are filled, and the FP64
state within 1e-12 of the oracle's."""
import numpy as np
import pytest

from gpu_util import max_rel, oracle_steps, say
from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu

KINDS = {"farfield": cases.FARFIELD, "slip": cases.SLIPWALL, "noslip": cases.NOSLIP_ADIABATIC, "extrap": cases.EXTRAP}


def _box(kind, face, dims=(18, 11, 9)):
    """A curved box of far-field faces but one, the flow crossing every face at an angle."""
    case = cases.vortex_case(max(dims), seed=4, curvilinear=True)
    ni, nj, nk = dims
    nodes = np.ascontiguousarray(case.nodes[0][:, :nk + 1, :nj + 1, :ni + 1])
    q0 = np.ascontiguousarray(case.q0[0][:, :nk, :nj, :ni])
    bcs = [cases.full_bc(0, dims, f, KINDS[kind] if f == face else cases.FARFIELD) for f in range(6)]
    return cases.Case("box", case.params, [dims], [nodes], [], bcs, [q0]).with_params(beta=0.3, alpha=0.2)


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("face", range(6))
@pytest.mark.parametrize("kind", list(KINDS))
def test_ghost_states_of_every_kind_and_face(kind, face, fp32):
    from paper_1710_09995_amd.binding import Solver
    case = _box(kind, face).with_params(flux_fp32=fp32, local_dt=face % 2)
    out = []
    for tun in ({"kernel": 0, "tile_j": 4, "tile_k": 1}, {"kernel": 1, "tile_j": 4, "tile_k": 8}):
        say("brick walls", kind, face, fp32, tun)
        s = Solver(case, tuning=tun)
        h = s.step(3).cpu().numpy()
        out.append((h, s.state()))
        s.close()
    exact = [0, 6, 7, 8, 9, 10, 11]
    assert np.isfinite(out[0][1][0]).all() and np.array_equal(out[0][1][0], out[1][1][0])
    assert np.array_equal(out[0][0][:, exact], out[1][0][:, exact])
    if not fp32:
        assert max_rel(out[0][1], oracle_steps(case, 3)[0]) <= 1e-12
