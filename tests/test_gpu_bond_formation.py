"""Bond formation with many eligible ligands: the wave that draws for 64 of
them together must give the ascending one-by-one order of the oracle, through
conflicts (ligands after the same receptor), several waves' worth of ligands,
uneven receptors and walls without receptors."""
import numpy as np
import pytest

import oracle
import paper_1907_00080_amd as pkg
from workloads import configs

pytestmark = pytest.mark.gpu


def _flat_body(nv, stride):
    """A long ellipse lying along the lower wall: most of its lower side within y_cr."""
    t = 2.0 * np.pi * np.arange(nv) / nv
    xy = np.stack([60.0 * np.cos(t) + 90.0, 4.0 * np.sin(t)], axis=1)
    xy[:, 1] += -0.5 + 0.3 - xy[:, 1].min()
    return configs.Body(configs.PARTICLE_RIGID, xy, sigma=1e-3, ligand_stride=stride)


RECEPTORS = {
    "sparse": np.linspace(20.0, 170.0, 9),                       # far fewer than ligands: conflicts
    "uneven": np.cumsum(np.tile([0.1, 3.0, 0.2, 1.7], 30)),      # off the evenly spaced guess
    "dense": np.arange(180, dtype=np.float64),
    "none": np.zeros(0),
}


@pytest.mark.parametrize("receptors", sorted(RECEPTORS))
@pytest.mark.parametrize("nv,stride,kf", [(300, 1, 5.0), (300, 2, 0.3), (131, 1, 1.0)])
def test_formation_order_matches_oracle(receptors, nv, stride, kf):
    print(f"[gpu-bonds] {receptors} nv {nv} stride {stride} kf0 {kf}", flush=True)
    rec = RECEPTORS[receptors]
    rec = rec[rec < 180.0]
    wl = configs.Workload("formation", 180, 32, gx=1e-6, bodies=[_flat_body(nv, stride)],
                          receptors=[rec, np.zeros(0)],
                          adhesion=configs.Adhesion(y_cr=6.0, y_eq=1.0, kf0_dt=kf, kr0_dt=0.05,
                                                    sigma_ts_frac=0.5, kbt=1e-3))
    sim = pkg.Sim(wl, dtype="f64")
    ref = oracle.Sim(wl)
    for _ in range(4):
        sim.step(1)
        ref.step(1)
        assert np.array_equal(sim.bonds(), ref.l2r)
    assert ref.ties == 0
    if rec.size:
        assert (ref.l2r >= 0).sum() >= min(5, rec.size)
    d = sim.diagnostics()
    assert d["sync_timeouts"] == 0 and d["bin_overflow"] == 0
