"""The order of a state's device work over its own and its callers' streams, on
the CPU: the host code of dc_runtime.hip and the kernels' launch code, linked
with tests/order_driver.cpp, whose model of the HIP runtime's streams, events
and captures checks that every operation comes after the one before it."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_35115_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not installed")
    from paper_2609_35115_amd import _build
    kernels = os.path.join(ROOT, "paper_2609_35115_amd", "_build", "libdc_so_dc_kernels.o")
    if not os.path.exists(kernels):
        _build.build()
    out = tmp_path_factory.mktemp("order")
    objs = []
    for src in (os.path.join(CSRC, "dc_runtime.hip"), os.path.join(ROOT, "tests", "order_driver.cpp")):
        o = str(out / (os.path.basename(src) + ".o"))
        subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC",
                        "-I", os.path.join(ROOT, "include"), "-c", src, "-o", o], check=True, capture_output=True)
        objs.append(o)
    exe = str(out / "driver")
    # (host-only objects name a code object that is not there: nothing reads it)
    subprocess.run([HIPCC, "-no-hip-rt", "-o", exe, *objs, kernels, "-Wl,--unresolved-symbols=ignore-all", "-lpthread"],
                   check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("scenario", ["several_streams", "settle", "capture", "failing_wait", "same_handle",
                                      "callers_error"])
def test_device_work_is_in_order(driver, scenario):
    r = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr
