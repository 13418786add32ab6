"""bench.py measures the vertex repulsion against one run without it (host only,
with a stand-in for the simulation)."""
import types

from tests.test_bench_host import _bench


def test_repulsion_is_measured_on_and_off_once(monkeypatch):
    b = _bench()
    made = []

    class Sim:
        step_mode = 2

        def __init__(self, wl, **kw):
            made.append(wl.repulsion > 0.0)

        def set_step_mode(self, m):
            pass

        def step(self, n):
            pass

        def diagnostics(self):
            return {"nonfinite": 0, "bin_overflow": 0, "sync_timeouts": 0}

        def close(self):
            pass

    monkeypatch.setattr(b, "_timed", lambda torch, sim, steps: steps * (0.03 if made[-1] else 0.02))
    res = b.repulsion_cost(types.SimpleNamespace(Sim=Sim), None, "channel-256x64", (64, 4), 10, 10)
    assert made == [True, False]
    assert abs(res["repulsion_us_per_step"] - 10.0) < 1e-9
