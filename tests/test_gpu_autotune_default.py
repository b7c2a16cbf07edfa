"""GPU: the tile autotuner with its own candidates on a grid that takes bricks by
default times that default first and ends on the fastest tuning it timed, the
solver's state untouched."""
import numpy as np
import pytest

from paper_1710_09995_amd import cases

pytestmark = pytest.mark.gpu


def test_default_tuning_is_a_candidate():
    from paper_1710_09995_amd.autotune import autotune
    from paper_1710_09995_amd.binding import Solver
    s = Solver(cases.vortex_case(24, nz=20, seed=1))
    start, before = s.get_tuning(), s.state()
    assert (start["kernel"], start["tile_k"]) == (0, 1)
    res = autotune(s, use_cache=False, verify=True)
    assert {k: res["table"][0][k] for k in start} == start
    least = min(res["table"], key=lambda r: r["ms_per_step"])
    assert s.get_tuning() == res["tuning"] == {k: least[k] for k in start}
    assert res["ms_per_step"] <= res["table"][0]["ms_per_step"]
    assert all(np.array_equal(a, b) for a, b in zip(s.state(), before))
    s.close()
