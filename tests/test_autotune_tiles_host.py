"""Host logic of the tile autotuner (autotune) on a stand-in solver: what it
times and what it keeps."""
import types

import pytest

from paper_1710_09995_amd import autotune as at


class _Solver:
    """Steps cost a table of milliseconds by (kernel, tile_j, tile_k), 1 by default;
    `capture`: tunings whose first call with a new step count costs 100 more."""
    stream = None
    device = "cpu"
    dims = [(8, 8, 8)]
    q = object()
    case = types.SimpleNamespace(params=types.SimpleNamespace(viscous=1, flux_fp32=0, local_dt=0))

    def __init__(self, current, costs, capture=()):
        self.now, self.costs, self.capture, self.seen = 0.0, costs, capture, set()
        self.t = dict(zip(("kernel", "tile_j", "tile_k"), current), use_graph=1, order=1)
        solver = self

        class Event:
            def __init__(self, **kw):
                self.t = None

            def record(self, stream):
                self.t = solver.now

            def elapsed_time(self, other):
                return other.t - self.t
        cuda = types.SimpleNamespace(Event=Event, synchronize=lambda device=None: None,
                                     current_stream=lambda device=None: None, is_available=lambda: False)
        self.torch = types.SimpleNamespace(cuda=cuda)

    def key(self):
        return self.t["kernel"], self.t["tile_j"], self.t["tile_k"]

    def get_tuning(self):
        return dict(self.t)

    def set_tuning(self, **t):
        self.t.update(t)
        self.seen = set()

    def new_arena(self):
        return types.SimpleNamespace(copy_=lambda src: None)

    def step(self, n, hist=True, arena=None):
        assert arena is not None and not hist
        self.now += n * self.costs.get(self.key(), 1.0)
        if self.key() in self.capture and n not in self.seen:
            self.now += 100.0
        self.seen.add(n)


def test_timed_steps_follow_a_call_of_their_own_length():
    """A run's graphs are captured on its first call; a run of another length has others."""
    s = _Solver((2, 8, 32), {(2, 8, 16): 0.5, (0, 4, 8): 0.9}, capture=[(2, 8, 32), (2, 8, 16)])
    res = at.autotune(s, candidates=[(2, 8, 16), (0, 4, 8)], use_cache=False)
    assert s.key() == (2, 8, 16) and abs(res["ms_per_step"] - 0.5) < 1e-12


def test_keeps_the_current_tuning_when_nothing_is_faster():
    s = _Solver((2, 8, 23), {(2, 8, 23): 0.4, (0, 4, 8): 0.5})
    before = s.get_tuning()
    res = at.autotune(s, candidates=[(0, 4, 8)], use_cache=False)
    assert res["tuning"] == before == s.get_tuning() and abs(res["ms_per_step"] - 0.4) < 1e-12
    assert [r["ms_per_step"] for r in res["table"]] == pytest.approx([0.4, 0.5])


@pytest.mark.parametrize("fastest", [(0, 4, 1), (2, 4, 16), (2, 8, 16), (0, 8, 8)])
def test_default_candidates_hold_every_kind_of_default_tuning(fastest):
    """Bricks, both sizes of plane-ring tiles, tiled tiles."""
    s = _Solver((2, 8, 32), {fastest: 0.5})
    at.autotune(s, use_cache=False)
    assert s.key() == fastest


def test_cached_winners_belong_to_the_library_that_timed_them(tmp_path, monkeypatch):
    from paper_1710_09995_amd import binding
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"one")
    monkeypatch.setenv("CFD_TUNE_CACHE", str(tmp_path / "tune.json"))
    monkeypatch.setattr(binding, "LIBPATH", str(lib))
    kept = at.autotune(_Solver((2, 8, 32), {(0, 4, 8): 0.5}), candidates=[(0, 4, 8)])
    again = at.autotune(_Solver((2, 8, 32), {}), candidates=[(0, 4, 8)])
    assert not kept["cached"] and again["cached"] and again["tuning"] == kept["tuning"]
    lib.write_bytes(b"two")
    s = _Solver((2, 8, 32), {(0, 4, 8): 2.0})
    other = at.autotune(s, candidates=[(0, 4, 8)])
    assert not other["cached"] and s.key() == (2, 8, 32)
