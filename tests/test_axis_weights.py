"""The three weights of a point along one axis with their first and second
derivatives (axis_weights in roma.h: what the reverse kernels use), against the
kernel taken node by node and against central differences (host build)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def fns(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("axis") / "libaxis.so")
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1907_00080_amd", "csrc"), "-o", out,
                    os.path.join(ROOT, "tests", "native", "axis_weights_check.cpp")], check=True)
    lib = ctypes.CDLL(out)
    D = ctypes.POINTER(ctypes.c_double)
    lib.t_axis.argtypes = [ctypes.c_double, ctypes.c_int, D]
    lib.t_node.argtypes = [ctypes.c_double, D]

    def axis(d, second=True):
        o = np.full(9, np.nan)
        lib.t_axis(float(d), int(second), o.ctypes.data_as(D))
        return o.reshape(3, 3)

    def node(r):
        o = np.full(3, np.nan)
        lib.t_node(float(r), o.ctypes.data_as(D))
        return o

    return axis, node


def test_three_nodes_match_the_kernel_node_by_node(fns):
    axis, node = fns
    # the node form rounds 1 - |d +- 1| to 2^-53; its effect grows with the next
    # derivative, at most 3, 24 and 144 in size on this range
    tol = np.array([4e-16 * 4, 4e-16 * 24, 4e-16 * 144])
    for d in np.concatenate([np.linspace(-0.5, 0.5, 1001)[1:-1], [1e-300, -1e-9, 0.5 - 1e-12]]):
        got = axis(d)
        want = np.array([node(d + a - 1) for a in range(3)]).T
        assert np.all(np.abs(got - want) <= tol[:, None]), (d, got - want)


def test_second_derivatives_are_differences_of_the_first(fns):
    axis, _ = fns
    h = 1e-6
    for d in np.linspace(-0.5 + 1e-5, 0.5 - 1e-5, 401):
        fd = (axis(d + h)[1] - axis(d - h)[1]) / (2 * h)
        # |phi''''| <= 3000 on this range: h^2 / 6 of it, and rounding / h
        assert np.all(np.abs(axis(d)[2] - fd) <= 5e-10 + 1e-9), d


def test_ends_and_switch(fns):
    axis, _ = fns
    for d in (0.5, np.nextafter(-0.5, 0.0)):
        # the one-sided values of the pieces the weights are taken from
        assert np.allclose(axis(d)[2], [4.0, -8.0, 4.0], rtol=1e-12)
    for d in np.linspace(-0.49, 0.5, 23):
        w, dw, ddw = axis(d)
        assert abs(w.sum() - 1.0) < 1e-15 and abs(dw.sum()) < 1e-15 and abs(ddw.sum()) < 1e-14
        off = axis(d, second=False)
        assert np.array_equal(off[:2], [w, dw]) and np.all(off[2] == 0.0)
