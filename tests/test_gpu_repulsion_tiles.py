"""Repulsion kernel: which tiles, entries and candidates a chunk looks at.
Cut-offs from one lattice unit to several tiles, on lattices narrower than the
reach, with the reach across the seam, and with more than 64 tiles per chunk;
the float64 path must agree with the oracle to round-off (1e-9)."""
import numpy as np
import pytest

import oracle
import paper_1907_00080_amd as pkg
from workloads import configs, geometry

pytestmark = pytest.mark.gpu


def _row(nx, ny, pery, cutoff):
    """Rings 1.2 apart in a row from the seam on, turned and shifted against each other."""
    bodies, x = [], 1.5
    while x + 6.0 < nx:
        k = len(bodies)
        kind = (configs.RBC_KINEMATIC, configs.PARTICLE_RIGID, configs.PARTICLE_SOFT)[k % 3]
        xy = geometry.place(geometry.circle(2.4, 17 + k % 5), 0.3 * k, [x, 0.5 * ny + (k % 3) - 1.0])
        bodies.append(configs.Body(kind, xy, ks=0.0 if kind == configs.PARTICLE_RIGID else 0.02))
        x += 6.0
    return configs.Workload("row", nx, ny, 1.0, gx=1e-6, periodic_y=pery, bodies=bodies,
                            repulsion=configs.REPULSION_COEFF, repulsion_cutoff=cutoff)


@pytest.mark.parametrize("tile", pkg.TILES)
@pytest.mark.parametrize("nx,ny,pery,cutoff", [(300, 60, 0, 1.0), (300, 60, 1, 5.0), (131, 40, 0, 16.0),
                                               (40, 71, 1, 16.0), (19, 12, 0, 7.0)])
def test_reach_matches_oracle(tile, nx, ny, pery, cutoff):
    print(f"[gpu-repulsion] {nx}x{ny} periodic_y={pery} cutoff {cutoff} tile {tile}", flush=True)
    wl = _row(nx, ny, pery, cutoff)
    sim = pkg.Sim(wl, dtype="f64", tile=tile)
    ref = oracle.Sim(wl)
    sim.step(3)
    ref.step(3)
    assert np.max(np.abs(sim.all_markers() - ref.all_markers())) < 1e-9
    d = sim.diagnostics()
    assert d["bin_overflow"] == 0
    sim.close()
