"""What the library's host code asks of the HIP runtime, call by call, on a stand-in that keeps account (no GPU):
tests/host_path_model.cpp, linked with the host side of the library's own sources.  And the work items that it cuts
maps into: tests/band_geometry_model.cpp with the host side of the headers."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1611_06256_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = tmp_path_factory.mktemp("host_path")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objects, running = [], []
    for name, flags in (("ga3c.hip", ["--cuda-host-only", "--offload-arch=gfx950"]), ("sched.hip", ["--cuda-host-only", "--offload-arch=gfx950"]),
                        ("tuner.cpp", [])):
        objects.append(str(out / (name + ".o")))
        running.append(subprocess.Popen([hipcc, *flags, "-O1", "-w", "-std=c++17", "-fPIC", "-c", os.path.join(CSRC, name), "-o", objects[-1]]))
    assert all(p.wait() == 0 for p in running)
    exe = str(out / "host_path_model")
    # the device code is not there: nothing but its registration refers to it
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-no-pie", "-o", exe,
                           os.path.join(ROOT, "tests", "host_path_model.cpp"), *objects, "-Wl,--unresolved-symbols=ignore-all"])
    return exe


@pytest.mark.parametrize("check", [
    "streams",      # calls on streams that come and go: every read and write of a parameter copy in order, no handle kept
    "capture",      # a stream that is being captured
    "packets",      # what predictions and updates leave in the queues besides their launches
    "ticks",        # a scheduler's tick allocates nothing and waits for nothing
    "memory",       # host memory that runs out in the scheduler's queues
    "workspace",    # partial sums of updates of any size, and no more memory for them than those need
    "fragments",    # the any-size layers' filters, as terms or rounded
    "order",        # results of several batches, oldest first
    "failures",     # launches and event records that fail in a scheduler's tick
])
def test_host_path(model, check):
    r = subprocess.run([model, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and " 0 problems" in r.stdout, r.stdout[-3000:] + r.stderr[-1000:]


def test_work_items_of_maps_of_any_proportion(tmp_path):
    # rows that a staging unit's packed place cannot hold would be another row's, at a byte that is no vector's
    hipcc, obj, exe = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), str(tmp_path / "model.o"), str(tmp_path / "model")
    subprocess.check_call([hipcc, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-w", "-std=c++17", "-c",
                           os.path.join(ROOT, "tests", "band_geometry_model.cpp"), "-o", obj])
    subprocess.check_call(["g++", "-no-pie", "-o", exe, obj, "-Wl,--unresolved-symbols=ignore-all"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and " 0 problems" in r.stdout, r.stdout[-3000:] + r.stderr[-1000:]
