"""Host side of the readbacks and the step modes (no GPU): the built library on a HIP runtime that
works on host memory and runs copies only when something waits for them
(tests/native/fake_hip.h)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1907_00080_amd")
ROCM = "/opt/rocm"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("g++ or the HIP headers not available")
    if not os.path.exists(os.path.join(PKG, "liblbib.so")):
        pytest.skip("liblbib.so not built")
    exe = str(tmp_path_factory.mktemp("readback") / "readback_host")
    subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-pthread", "-D__HIP_PLATFORM_AMD__", "-w", "-rdynamic",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "native", "readback_host.cpp"), "-L", PKG, "-llbib",
                    f"-Wl,-rpath,{PKG}", f"-Wl,-rpath-link,{os.path.join(ROCM, 'lib')}"], check=True)
    return exe


# device: a stream of another device than the current one; close: contexts
# closed beside others; threads: more of them than rings; refused, failed: no
# pinned memory, a copy that fails; error: one left behind by the program;
# pinned: a state blob in pinned memory; modes: the step modes' names
@pytest.mark.parametrize("case", ["device", "close", "threads", "refused", "failed", "error", "pinned", "modes"])
def test_host_side(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
