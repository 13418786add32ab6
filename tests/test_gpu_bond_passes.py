"""Bond kinetics of an instance with more ligands than one pass of the bond
workgroup takes (1024): three passes, so that a set of counts is used again, the
last one ragged, with eligible ligands in every pass, more than 64 of them in
all or fewer (the two ways they are handed to the formation).  Every step's bond
table must be the oracle's."""
import numpy as np
import pytest

import oracle
import paper_1907_00080_amd as pkg
from workloads import configs

pytestmark = pytest.mark.gpu

PASS = 1024
BODIES, NV = 8, 290


def _workload(y_cr, kf, kr):
    bodies = []
    t = 2.0 * np.pi * np.arange(NV) / NV
    for k in range(BODIES):
        xy = np.stack([60.0 * np.cos(t) + 70.0 + 137.0 * k, 4.0 * np.sin(t)], axis=1)
        xy[:, 1] += -0.5 + 0.3 - xy[:, 1].min()
        bodies.append(configs.Body(configs.PARTICLE_RIGID, xy, sigma=1e-3, ligand_stride=1))
    nx = 137 * BODIES
    return configs.Workload("bond passes", nx, 32, gx=1e-6, bodies=bodies,
                            receptors=[np.arange(0.25, nx, 0.5), np.zeros(0)],
                            adhesion=configs.Adhesion(y_cr=y_cr, y_eq=1.0, kf0_dt=kf, kr0_dt=kr,
                                                      sigma_ts_frac=0.5, kbt=1e-3))


# y_cr 6: most of the lower sides; 0.315: a few ligands of each body
@pytest.mark.parametrize("y_cr,kf,kr", [(6.0, 0.3, 0.2), (0.315, 1.0, 0.3)])
def test_three_passes_match_oracle(y_cr, kf, kr):
    print(f"[gpu-bonds] passes y_cr {y_cr}", flush=True)
    wl = _workload(y_cr, kf, kr)
    nlig = BODIES * NV
    assert 2 * PASS < nlig < 3 * PASS and nlig % (PASS // 2) != 0
    eligible = np.concatenate([0.5 * (b.xy[:, 1] + np.roll(b.xy[:, 1], -1)) + 0.5 < y_cr for b in wl.bodies])
    assert (eligible.sum() > 64) == (y_cr > 1.0)
    for lo in range(0, nlig, PASS):
        assert eligible[lo:lo + PASS].any()
    sim = pkg.Sim(wl, dtype="f64")
    ref = oracle.Sim(wl)
    formed = np.zeros(nlig, dtype=bool)
    ruptured = 0
    for _ in range(5):
        before = ref.l2r.copy()
        sim.step(1)
        ref.step(1)
        assert np.array_equal(sim.bonds(), ref.l2r)
        formed |= ref.l2r >= 0
        ruptured += int(((before >= 0) & (ref.l2r != before)).sum())
    assert ref.ties == 0 and ruptured > 0
    for lo in range(0, nlig, PASS):
        assert formed[lo:lo + PASS].any()
    d = sim.diagnostics()
    assert d["sync_timeouts"] == 0 and d["bin_overflow"] == 0
    sim.close()
