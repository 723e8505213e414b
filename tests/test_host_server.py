"""The library's host code without a GPU: every csrc/*.hip file's host side (hipcc
--offload-host-only) over a stand-in for the HIP runtime (tests/host/fake_hip.cpp) whose
kernels do nothing and whose streams, events and graphs are watched, so that a call naming a
destroyed one, or asking about an event whose stream was destroyed, is an error.  The driver
(tests/host/server_driver.cpp) sends bursts of jobs to servers that come and go, makes calls
on streams of its own that come and go, lets every allocation of a call fail, and looks at
the route of batches near the LDS limit."""
import concurrent.futures as cf
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


def _run(cmd, **kw):
    r = subprocess.run(cmd, capture_output=True, text=True, **kw)
    return r.returncode, r.stdout + r.stderr


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or shutil.which("g++") is None:
        pytest.skip("hipcc or g++ is not installed")
    d = tmp_path_factory.mktemp("host_server")
    srcs = sorted(glob.glob(os.path.join(ROOT, "paper_1606_02162_amd", "csrc", "*.hip")))

    def compile_one(src):
        obj = str(d / (os.path.basename(src) + ".o"))
        rc, out = _run([hipcc, "-std=c++17", "-O1", "-fPIC", "--offload-arch=gfx950",
                        "--offload-host-only", "-Wno-unused-result", "-c", src, "-o", obj])
        assert rc == 0, out
        return obj

    with cf.ThreadPoolExecutor(4) as ex:
        objs = list(ex.map(compile_one, srcs))
    # the device code that each file would carry
    rc, out = _run(["nm", "-u", *objs])
    assert rc == 0, out
    names = sorted(set(re.findall(r"__hip_fatbin_\w+", out)))
    stub = d / "fatbin.cpp"
    stub.write_text("".join(f'extern "C" const char {n}[8] = {{0}};\n' for n in names))
    exe = str(d / "server_driver")
    rc, out = _run(["g++", "-std=c++17", "-O1", "-Wall", str(stub), os.path.join(HOST, "fake_hip.cpp"),
                    os.path.join(HOST, "server_driver.cpp"), *objs, "-o", exe, "-lpthread"])
    assert rc == 0, out
    return exe


def test_no_event_outlives_its_stream(driver):
    rc, out = _run([driver, "streams"], timeout=240)
    assert rc == 0 and out.strip().endswith("OK"), out


def test_positions_stay_when_memory_runs_out(driver):
    """gila_layout_components with the i-th device allocation and all after it failing, for
    every i: ENOMEM, and no kernel that writes the caller's positions was launched."""
    rc, out = _run([driver, "memory"], timeout=240)
    assert rc == 0 and out.strip().endswith("OK"), out


def test_batch_route_near_the_lds_limit(driver):
    """A batch takes one workgroup of 1024 threads, or of 512, per unit of a graph as long as
    the graph and three bitmaps per wavefront fit in LDS."""
    rc, out = _run([driver, "batch"], timeout=240)
    assert rc == 0 and out.strip().endswith("OK"), out
