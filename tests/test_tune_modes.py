"""The autotuner times what differs: the step modes are names of one launch
form, so each choice of tile, hints and graph chunk is timed once and listed
under every mode (host only, with a stand-in for the batch)."""
import paper_1907_00080_amd as pkg
from paper_1907_00080_amd import tune
from workloads import configs


class _Batch:
    log = []

    def __init__(self, workloads, dtype, tile, device=None, graph_steps=0, streaming=None):
        self.tile, self.g, self.sm = tuple(tile), graph_steps, streaming
        self.mode, self.cache_hints, self.launch = 0, 0, 0

    def set_step_mode(self, m):
        self.mode = m

    @property
    def step_mode(self):
        return self.mode or 2

    def set_cache_hints(self, h):
        self.cache_hints = h

    def set_graph_steps(self, g):
        self.g = g

    def set_lattice_launch(self, w):
        self.launch = w

    def step(self, n):
        pass

    def close(self):
        pass


def test_step_modes_share_one_timing(monkeypatch):
    timed = []

    def time_steps(b, steps):
        timed.append((b.tile, b.g, b.cache_hints, b.launch, b.sm))
        # the later of two timings of one form is the faster, as noise may have it
        return 100.0 + 10.0 * (b.cache_hints != 1) + 5.0 * (b.tile != (128, 2)) - 0.01 * len(timed)

    monkeypatch.setattr(pkg, "Batch", _Batch)
    monkeypatch.setattr(tune, "_time_steps", time_steps)
    monkeypatch.setattr(tune, "_device_name", lambda d: "none")
    ws = [configs.small_case(nx=48, ny=24, n_rbc=1, seed_offset=31)]
    rec = tune.autotune(ws, "f32", cache=None)
    first = len(tune.TILES) * len(tune.CACHE_HINTS) * len(tune.GRAPH_STEPS)
    assert len(timed) == first + 4 + 1 and len(set(timed[:first])) == first
    # listed under every mode with the one time, and the first mode picked
    assert len(rec["candidates"]) == first * len(tune.STEP_MODES)
    for c in rec["candidates"]:
        same = [d["ms_per_step"] for d in rec["candidates"]
                if (d["tile"], d["graph_steps"], d["cache_hints"])
                == (c["tile"], c["graph_steps"], c["cache_hints"])]
        assert len(same) == len(tune.STEP_MODES) and len(set(same)) == 1
    assert rec["tile"] == [128, 2] and rec["cache_hints"] == 1 and rec["step_mode"] == tune.STEP_MODES[0]
