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


def _check(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]


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
            inc = ["-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), "-I", HERE]
            src = os.path.join(HERE, main + ".cpp")
            if main == "grids_main":  # includes a header with device functions: only their host side is compiled
                obj = exe + ".o"
                _check(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-host-only", "-fPIC", "-std=c++17", "-O1", *inc, "-c", src,
                        "-o", obj])
                src = obj
            _check(["g++", "-std=c++17", "-O1", *inc, src, os.path.join(HERE, "fake_hip.cpp"),
                    os.path.join(PKG, "liblbm3.so"), "-Wl,-rpath," + PKG, "-Wl,-rpath-link,/opt/rocm/lib", "-rdynamic",
                    "-o", exe])
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


def test_block_grids_cover_the_lattice(driver):
    """The grids of the one-step and two-step blocks, for lattices around the sides of a block and
    devices of different numbers of compute units."""
    assert driver("grids_main").strip() == "ok"


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("cell,times", [((45, 19, 8), (5, 5, 1)), ((28, 24, 9), (8, 4, 1)), ((31, 5, 60), (3, 7, 3))])
def test_a_box_and_its_repetition_take_different_tiles(driver, cell, times, precision, q):
    """The pairs of boxes that tests/test_gpu_d3.py compares bit for bit (small and large tiles) do
    take different tiles on 256 compute units."""
    large = 24 if precision == 2 else 16
    rows = [int(driver("dispatch_main", "box", *(str(c * t) for c, t in zip(cell, n)), str(q), str(precision)))
            for n in ((1, 1, 1), times)]
    assert rows == [8, large]
