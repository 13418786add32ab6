"""Contexts beside each other: what one does must not wait for, or be changed
by, another one's run."""
import ctypes
import threading

import numpy as np
import pytest

import paper_1907_00080_amd as pkg
from workloads import configs

pytestmark = pytest.mark.gpu


def _small(k):
    return configs.small_case(nx=96 + 8 * k, ny=24, n_rbc=1, particles=(configs.PARTICLE_RIGID,),
                              seed_offset=60 + k)


def test_closing_a_context_does_not_wait_for_another_run():
    """A run of tens of milliseconds is still under way after another context,
    which has been read, is closed."""
    import torch
    print("[gpu-contexts] close", flush=True)
    big = pkg.Sim(configs.capillary_2000x200(), graph_steps=100)
    big.step(200)
    small = pkg.Sim(_small(0))
    small.step(2)
    small.fields()
    small.markers(0)
    small.stream.synchronize()
    big.stream.synchronize()
    big.step(4000)
    done = torch.cuda.Event()
    done.record(big.stream)
    assert not done.query()
    small.close()
    assert not done.query()
    done.synchronize()
    big.close()


def test_readbacks_on_threads_of_their_own():
    """Six contexts, each stepped and read by its own thread at the same time,
    give what they give one after the other, bit for bit."""
    print("[gpu-contexts] threads", flush=True)

    def job(k):
        s = pkg.Sim(_small(k))
        out = []
        for _ in range(5):
            s.step(4)
            out += [*s.fields(), s.markers(0), s.markers(1), s.marker_forces(1)]
            s.set_state(s.get_state())   # the blob itself has unused bytes (row padding)
        s.close()
        return out

    want = [job(k) for k in range(6)]
    got = [None] * 6
    ts = [threading.Thread(target=lambda k=k: got.__setitem__(k, job(k))) for k in range(6)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(6):
        assert got[k] is not None
        for a, b in zip(want[k], got[k]):
            assert np.array_equal(a, b)


def test_marker_reads_after_a_refused_call_of_the_program():
    """A HIP call of the program's own that the runtime refused (and whose error
    it still holds for this thread) is not an error of the next marker read."""
    print("[gpu-contexts] refused call", flush=True)
    s = pkg.Sim(_small(0))
    s.step(2)
    want = [s.markers(1), s.marker_forces(1)]
    hip_set_device = s.lib.hipSetDevice   # the runtime the library is linked to
    hip_set_device.argtypes, hip_set_device.restype = [ctypes.c_int], ctypes.c_int
    try:
        for k, read in enumerate((s.markers, s.marker_forces)):
            assert hip_set_device(999) != 0
            assert np.array_equal(read(1), want[k])
    finally:
        s.lib.hipGetLastError()   # taken back: other calls of this process look at it
    s.close()


@pytest.mark.parametrize("handle", [0, 1, 2])
def test_default_legacy_and_per_thread_streams(handle):
    """A context on the null stream, the legacy or the per-thread one."""
    import torch
    print(f"[gpu-contexts] stream handle {handle}", flush=True)

    class Stream:
        cuda_stream = handle

    ref = pkg.Sim(_small(0))
    torch.cuda.synchronize()
    s = pkg.Sim(_small(0), stream=Stream())
    for a in (ref, s):
        a.step(3)
    for a, b in zip([*ref.fields(), ref.markers(1)], [*s.fields(), s.markers(1)]):
        assert np.array_equal(a, b)
    ref.close()
    s.close()
