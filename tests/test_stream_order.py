"""The order of a state's device work over its own and its callers' streams, on
the CPU: the host code of dc_runtime.hip and the kernels' launch code, linked
with tests/order_driver.cpp, whose model of the HIP runtime's streams, events
and captures checks that every operation comes after the one before it; and the
binding's share, the calls that Decoder.decode makes around a decode."""
from __future__ import annotations

import os
import subprocess
from types import SimpleNamespace as NS

import numpy as np
import pytest

import paper_2609_35115_amd as dc

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


def test_a_held_stream_is_settled_around_every_decode(monkeypatch):
    """Once a program has read Decoder.stream, each decode on another stream is
    ordered with it both ways (what dc_settle does: the `settle` scenario above);
    before, none is."""
    calls = []
    monkeypatch.setattr(dc, "dc_decode_chunk_on", lambda *a: calls.append("decode") or dc.DC_OK)
    monkeypatch.setattr(dc, "dc_settle", lambda h: calls.append("settle") or dc.DC_OK)
    monkeypatch.setattr(dc, "dc_free", lambda h: None)
    dec = dc.Decoder.__new__(dc.Decoder)
    current = NS(cuda_stream=7)
    dec.torch = NS(cuda=NS(current_device=lambda: 0, is_current_stream_capturing=lambda: False,
                           current_stream=lambda: current),
                   from_numpy=lambda a: NS(to=lambda d: a), empty=lambda *a, **k: object(), float32=None)
    dec.h, dec.host, dec.device, dec.batch, dec.max_tokens, dec.spt, dec.has_source = 1, False, 0, 1, 8, 4, False
    dec.arch, dec._stream, dec._shared = {"frames_per_token": 1}, object(), False
    ids = np.zeros((1, 8), np.int32)
    dec.decode(ids)
    assert calls == ["decode"]
    held = dec.stream
    assert held is dec._stream and calls == ["decode", "settle"]
    del calls[:]
    dec.decode(ids)
    dec.decode(ids)
    assert calls == ["settle", "decode", "settle"] * 2
