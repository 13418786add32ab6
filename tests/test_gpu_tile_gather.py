"""Spreading into a tile with one row of one marker per lane: bins of up to a
wave's worth of rows (21 markers), beyond it, and beyond one pass of the
workgroup (85 markers), on tiles cut by the seam and by both walls, against
the float64 oracle."""
import numpy as np
import pytest

import oracle
import paper_1907_00080_amd as pkg
from workloads import configs, geometry

pytestmark = pytest.mark.gpu


def _ring(x, y, r, n, kind=configs.RBC_KINEMATIC):
    return configs.Body(kind, geometry.place(geometry.circle(r, n), 0.1, [x, y]), ks=0.02, kb=1e-3)


# vertices of one ring of radius 3.2: all of them meet in one or two tiles
@pytest.mark.parametrize("nv", [3, 20, 22, 64, 86, 180, 300])
@pytest.mark.parametrize("tile", [(64, 4), (256, 1)])
@pytest.mark.parametrize("nx,periodic_y", [(65, 0), (257, 0), (70, 1)])
def test_crowded_tile_matches_oracle(nv, tile, nx, periodic_y):
    print(f"[gpu-gather] nv {nv} tile {tile} nx {nx} periodic_y {periodic_y}", flush=True)
    ny, r = 21, 3.2
    y = ny / 2.0 if periodic_y else (r + 0.4 if nv % 2 else ny - 1.4 - r)
    wl = configs.Workload("gather", nx, ny, gx=1e-5, periodic_y=periodic_y,
                          bodies=[_ring(nx - 1.0, y, r, nv), _ring(0.4 * nx, 0.55 * ny, r, nv)])
    for b in wl.bodies:   # out of its rest shape, so that forces act from the first step
        b.ks = 0.02
    sim = pkg.Sim(wl, dtype="f64", tile=tile)
    ref = oracle.Sim(wl)
    stretched = [1.02 * (b.xy - b.xy.mean(0)) + b.xy.mean(0) for b in wl.bodies]
    for k, xy in enumerate(stretched):
        sim.set_markers(k, xy)
        ref.bodies[k].X = xy.copy()
        ref.bodies[k].Xm = xy.copy()
    sim.step(5)
    ref.step(5)
    _, ux, uy = sim.fields()
    scale = np.sqrt((ref.ux ** 2 + ref.uy ** 2).sum())
    assert scale > 0
    assert np.sqrt(((ux - ref.ux) ** 2 + (uy - ref.uy) ** 2).sum()) <= 1e-9 * scale
    assert np.abs(sim.all_markers() - ref.all_markers()).max() <= 1e-9
    assert sim.diagnostics()["bin_overflow"] == 0
