"""The library's memory handling and dispatch on a stand-in for the HIP runtime (CPU only).

The built liblbm3.so is linked with tests/fake_device/fake_hip.cpp, whose definitions take the
place of the runtime's: device memory is address space with a settable capacity, launches and
copies are recorded and do nothing, any call can be made to fail.  The library's host code runs
unchanged; no kernel does."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "fake_device")
PKG = os.path.join(ROOT, "paper_1808_08555_amd")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    """Builds a driver (its main file's name) and returns a function that runs it."""
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("g++ or the HIP headers are not available")
    if not os.path.exists(os.path.join(PKG, "liblbm3.so")):
        from paper_1808_08555_amd import build
        build.build()
    built = {}

    def run(main, *args):
        if main not in built:
            exe = str(tmp_path_factory.mktemp("fake") / main)
            r = subprocess.run(["g++", "-std=c++17", "-O1", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                                "-I", HERE, os.path.join(HERE, main + ".cpp"), os.path.join(HERE, "fake_hip.cpp"),
                                os.path.join(PKG, "liblbm3.so"), "-Wl,-rpath," + PKG, "-Wl,-rpath-link,/opt/rocm/lib",
                                "-rdynamic", "-o", exe], capture_output=True, text=True)
            assert r.returncode == 0, r.stderr[-3000:]
            built[main] = exe
        r = subprocess.run([built[main], *args], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
        return r.stdout

    return run


@pytest.mark.parametrize("what", ["pool", "retry", "faults"])
def test_memory(driver, what):
    """pool: what the pool of workspaces keeps and gives back; retry: every allocation of the
    library finds the memory that the pool keeps; faults: each runtime call of a reverse sweep
    failing in turn leaves no work, event or memory behind."""
    assert driver("memory_main", what).strip() == "ok"


def test_a_cleared_shape_brings_the_default_launches_back(driver):
    assert driver("dispatch_main", "clear").strip() == "ok"
