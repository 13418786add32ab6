"""Body kernel: how the chunks of particles and red cells share workgroups.
Rigid bodies of one to four chunks are packed whole, larger ones and soft
particles by chunks, each with a wave that samples the fluid at its vertices;
red cells fill workgroups of their own.  Every mix must follow the oracle to
the round-off of the float64 path (1e-9)."""
import numpy as np
import pytest

import oracle
import paper_1907_00080_amd as pkg
from workloads import configs

pytestmark = pytest.mark.gpu

RIGID, SOFT, RBC = configs.PARTICLE_RIGID, configs.PARTICLE_SOFT, configs.RBC_KINEMATIC
MIXES = {
    # (kind, vertices): a body that does not fit the rest of its workgroup opens the next
    "rigid": [(RIGID, n) for n in (16, 61, 181, 60, 240, 120, 121, 59, 17, 180)],
    "large": [(RIGID, 241), (SOFT, 61), (RIGID, 300), (SOFT, 240), (RIGID, 62)],
    "mixed": [(RBC, 130), (SOFT, 60), (RIGID, 45), (RBC, 61), (SOFT, 121), (RBC, 600), (RIGID, 182)],
    "soft": [(SOFT, 40)],
}


def _workload(mix, transfer):
    bodies = []
    for k, (kind, n) in enumerate(MIXES[mix]):
        t = 2.0 * np.pi * (np.arange(n) + 0.3 * k) / n
        xy = np.stack([7.0 * np.cos(t) + 12.0 + 24.0 * k, 5.0 * np.sin(t) + 14.0 + (k % 3)], axis=1)
        bodies.append(configs.Body(kind, xy, ks=0.0 if kind == RIGID else 1e-3, ka=1e-3, kb=0.0))
    return configs.Workload("packing", 24 * len(bodies), 31, gx=2e-5, bodies=bodies, transfer=transfer,
                            u0=np.stack([np.full((31, 24 * len(bodies)), 0.02), np.zeros((31, 24 * len(bodies)))]))


@pytest.mark.parametrize("transfer", ["roma", "mls"])
@pytest.mark.parametrize("mix", sorted(MIXES))
def test_packed_bodies_match_oracle(mix, transfer):
    print(f"[gpu-packing] {mix} {transfer}", flush=True)
    wl = _workload(mix, transfer)
    sim = pkg.Sim(wl, dtype="f64")
    ref = oracle.Sim(wl)
    sim.step(6)
    ref.step(6)
    assert np.max(np.abs(sim.all_markers() - ref.all_markers())) < 1e-9
    _, ux, uy = sim.fields()
    scale = np.sqrt(np.sum(ref.ux ** 2 + ref.uy ** 2))
    assert np.sqrt(np.sum((ux - ref.ux) ** 2 + (uy - ref.uy) ** 2)) < 1e-9 * scale
    assert sim.diagnostics()["sync_timeouts"] == 0
    sim.close()
