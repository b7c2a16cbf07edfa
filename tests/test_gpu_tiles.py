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


BRICK = {"kernel": 0, "tile_j": 4, "tile_k": 1}


def _extrap_case():
    """A channel whose outflow face extrapolates."""
    case = cases.channel_case(19, 9, 7, mach=0.7, hb=0.08, local_dt=0)
    for bc in case.bcs:
        if bc.face == 1:
            bc.kind = cases.EXTRAP
    return case


BRICK_CASES = {
    "channel_local": lambda: cases.channel_case(21, 11, 6, mach=0.7, hb=0.08),
    "channel_thin": lambda: cases.channel_case(9, 2, 5, mach=0.6, hb=0.05),
    "extrap": _extrap_case,
    "chain": lambda: cases.batched_euler_case(nblk=4, seed=6, lo=2, hi=19, flux_fp32=0),
    "chain_fp32": lambda: cases.batched_euler_case(nblk=3, seed=7, lo=5, hi=14),
    "periodic": lambda: cases.vortex_case(10, nz=3, seed=1, curvilinear=True),
    "split": lambda: cases.split_periodic_box(cases.vortex_case(8, nz=8, seed=2), (4, 2, 2)),
    "ns": lambda: cases.bump_ns_case(19, 7, 5, seed=3, reynolds=5e3),
}


@pytest.mark.parametrize("name", list(BRICK_CASES))
def test_bricks_match_the_simple_kernel(name):
    """Bricks form their inviscid ghost states from the cells they depend on;
    every boundary kind and connection gives bitwise the filled ghosts' steps,
    with a history and without, as single launches and as a graph of eight."""
    from paper_1710_09995_amd.binding import Solver
    case = BRICK_CASES[name]()
    say("bricks", name)
    h0, q0 = _run(case, {"kernel": 1, "tile_j": 4, "tile_k": 8})
    h, q = _run(case, BRICK)
    for a, b in zip(q, q0):
        assert np.array_equal(a, b)
    exact = [0, 6, 7, 8, 9, 10, 11]
    assert np.array_equal(h[:, exact], h0[:, exact])
    runs = []
    for tun in (BRICK, dict(BRICK, use_graph=0), {"kernel": 1, "tile_j": 4, "tile_k": 8}):
        s = Solver(case, tuning=tun)
        for _ in range(3):
            s.step(9, hist=False)
            s.torch.cuda.synchronize()
        runs.append(s.state())
        s.close()
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("name", ["channel_local", "chain", "ns"])
def test_residual_reads_the_callers_ghosts(name):
    """cfd_residual takes the arena as it is, ghost cells included, on bricks as
    on the simple kernel."""
    from paper_1710_09995_amd.binding import Solver
    case = BRICK_CASES[name]()
    out = []
    for tun in (BRICK, {"kernel": 1, "tile_j": 4, "tile_k": 8}):
        s = Solver(case, tuning=tun)
        s.fill_ghosts()
        for v, (ni, nj, nk) in zip(s.views(), s.dims):      # ghost states no fill would give
            v[:, :2] *= 1.01
            v[:, :, nj + 2:] *= 0.99
            v[:, :, :, :2] *= 1.02
        r = s.residual(fill=False)
        out.append([t.cpu().numpy() for t in s.interior_views(r)])
        s.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
