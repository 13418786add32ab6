"""Reverse sweep of particles around the sizes where its split over lanes and
waves changes (21 items to a wave, 63 to a workgroup, larger bodies one lane
per item): gradients against central differences of the float64 forward."""
import numpy as np
import pytest

import paper_1907_00080_amd as pkg
from paper_1907_00080_amd.adjoint import AdjointWindow
from workloads import configs, geometry

pytestmark = pytest.mark.gpu


def _workload(nv, rigid):
    wl = configs.adjoint_channel(nx=96, ny=32, n_rbc=0, rigid=rigid)
    b = wl.bodies[0]
    r = max(2.0, nv / (2.0 * np.pi * 1.1))
    p0 = geometry.circle(r, nv)
    b.xy = geometry.place(p0, 0.05, [30.3, 0.0])
    b.xy[:, 1] += -0.5 + 0.25 - b.xy[:, 1].min()
    if not rigid:
        b.kb = 0.05 * b.ks * r * r
    return wl


@pytest.mark.parametrize("rigid", [False, True])
@pytest.mark.parametrize("nv", [5, 21, 22, 42, 43, 63, 64, 84])
def test_gradient_matches_finite_differences(nv, rigid):
    print(f"[gpu-adjoint-sizes] nv {nv} rigid {rigid}", flush=True)
    wl = _workload(nv, rigid)
    sim = pkg.Sim(wl, dtype="f64")
    sim.step(1)
    state = sim.get_state()
    bonds = int((sim.bonds() >= 0).sum())
    win = AdjointWindow(sim, 30, 7)
    P0 = np.array([wl.bodies[0].ks, wl.bodies[0].kb, wl.bodies[0].sigma])

    def J(P):
        sim.set_state(state)
        sim.set_body_params(0, *P)
        return win.forward()[0]

    J(P0)
    g = win.backward(1.0)[0]
    again = win.backward(1.0)[0]
    assert np.array_equal(g, again)
    for q in ([2] if rigid else [0, 1, 2]):
        if q == 2 and bonds == 0:
            continue
        h = 1e-3 * P0[q]
        d = np.zeros(3)
        d[q] = h
        fd = (J(P0 + d) - J(P0 - d)) / (2 * h)
        # the bound of the existing float64 gradient test
        assert abs(g[q] - fd) <= 1e-5 * abs(fd) + 1e-12, (q, g[q], fd)
