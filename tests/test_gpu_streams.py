"""Decoder.decode runs on the caller's current stream (dc_decode_chunk_on):
calls from several streams and threads, mixed with C calls and resets on the
state's own stream and work of the caller's there, none of them waited for, give
the bits of the same calls made one after the other on the state's stream; so
does a decode captured after an uncaptured one."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import paper_2609_35115_amd as dc
from paper_2609_35115_amd import synth
from tests.gpu_common import bits_equal

pytestmark = pytest.mark.gpu

CASES = [("tiny", synth.TINY_ARCH, "f32", 2, 8), ("tiny source", synth.TINY_NSF_ARCH, "f32", 2, 8),
         ("tiny bf16 fused batch", synth.TINY_ARCH, "bf16", 8, 5),
         ("real bf16", synth.REAL_ARCH, "bf16", 16, 25)]   # calls ten times longer than their submission
PER_THREAD = 2   # hipStreamPerThread


def _inputs(arch, B, sizes):
    """Every call's tokens and f0 on the device."""
    fpt = arch["frames_per_token"]
    ids = synth.make_tokens(arch, B, sum(sizes))
    f0 = synth.make_f0(arch, B, sum(sizes)) if "n_harmonics" in arch else None
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    out, at = [], 0
    for n in sizes:
        out.append((cuda(ids[:, at:at + n]), None if f0 is None else cuda(f0[:, at * fpt:(at + n) * fpt])))
        at += n
    return out


def _home(dec, tok, f0, out):
    """One C call on the state's own stream, not waited for."""
    n = tok.shape[1]
    st = (dc.dc_decode_chunk_f0(dec.h, tok, f0, n, out) if dec.has_source else dc.dc_decode_chunk(dec.h, tok, n, out))
    assert st == dc.DC_OK


def _reference(arch, dtype, blob, B, chunk, inputs, resets=()):
    """The calls one after the other on the state's stream, each waited for."""
    ref = dc.Decoder(arch, dtype, blob, B, chunk, chunk, rng_seed=7)
    want = []
    for i, (tok, f0) in enumerate(inputs):
        if i in resets:
            ref.reset_stream(1)
        out = torch.empty((B, tok.shape[1] * ref.spt), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        _home(ref, tok, f0, out)
        ref.sync()
        want.append(out.cpu().numpy())
    ref.close()
    return want


@pytest.mark.parametrize("name,arch,dtype,B,chunk", CASES, ids=[c[0] for c in CASES])
def test_calls_from_several_streams_are_in_order(name, arch, dtype, B, chunk):
    blob = synth.make_weights(arch, 0)
    sizes = [chunk, chunk, 3, chunk, 1, chunk, chunk, 2, chunk, chunk, chunk, chunk, 3, chunk]   # replays, direct launches
    inputs, resets = _inputs(arch, B, sizes), (6, 9)
    want = _reference(arch, dtype, blob, B, chunk, inputs, resets)
    dec = dc.Decoder(arch, dtype, blob, B, chunk, chunk, rng_seed=7)
    got = [torch.empty(w.shape, dtype=torch.float32, device="cuda") for w in want]
    side = [torch.cuda.Stream() for _ in range(2)]

    def raw(stream, i):
        tok, f0 = inputs[i]
        assert dc.dc_decode_chunk_on(dec.h, stream, tok, f0, tok.shape[1], got[i]) == dc.DC_OK

    torch.cuda.synchronize()
    for i, (tok, f0) in enumerate(inputs):      # nothing is waited for from here
        if i in resets:
            dec.reset_stream(1)
        how = i % 7
        if how == 3:
            _home(dec, tok, f0, got[i])
        elif how == 5:
            raw(PER_THREAD, i)
        elif how == 6:
            t = threading.Thread(target=raw, args=(PER_THREAD, i))
            t.start()
            t.join()
        else:
            with torch.cuda.stream([torch.cuda.default_stream(), side[0], side[1], None, dec._stream][how]):
                got[i] = dec.decode(tok, f0)
    dec.sync()
    torch.cuda.synchronize()
    for i, (w, g) in enumerate(zip(want, got)):
        assert bits_equal(g.cpu().numpy(), w), f"call {i}"
    assert dec.stats()["staged_tokens"] == dec.stats()["calls"] == len(sizes)
    # a reset on the state's stream comes after the caller's calls
    got = dec.decode(*inputs[0])
    dec.reset()
    again = dec.decode(*inputs[0])
    torch.cuda.synchronize()
    assert bits_equal(again.cpu().numpy(), want[0]) and not bits_equal(got.cpu().numpy(), want[0])
    dec.close()


@pytest.mark.parametrize("name,arch,dtype,B,chunk", [CASES[0], CASES[3]], ids=["tiny", "real bf16"])
def test_work_on_a_held_stream_is_in_order_with_decodes(name, arch, dtype, B, chunk):
    """A program that keeps Decoder.stream writes each call's tokens and reads its
    PCM there, while the decodes run on its current stream; nothing is waited for."""
    blob = synth.make_weights(arch, 0)
    inputs = _inputs(arch, B, [chunk] * 8)
    want = _reference(arch, dtype, blob, B, chunk, inputs)
    dec = dc.Decoder(arch, dtype, blob, B, chunk, chunk, rng_seed=7)
    held = dec.stream
    tok = torch.zeros_like(inputs[0][0])
    got = [torch.empty(w.shape, dtype=torch.float32, device="cuda") for w in want]
    torch.cuda.synchronize()
    pcm = []                                    # (kept: their memory is not handed out again)
    for (t, _), g in zip(inputs, got):
        with torch.cuda.stream(held):
            tok.copy_(t)
        pcm.append(dec.decode(tok))
        with torch.cuda.stream(held):
            g.copy_(pcm[-1])
            tok.zero_()
    torch.cuda.synchronize()
    for i, (w, g) in enumerate(zip(want, got)):
        assert bits_equal(g.cpu().numpy(), w), f"call {i}"
    dec.close()


def test_a_captured_decode_after_an_uncaptured_one():
    """decode under torch's graph capture (a decoder without graphs of its own; in
    relaxed mode, as the call allocates its PCM on the state's stream), after a
    decode on the caller's stream; replays between eager decodes."""
    arch, B, n = synth.TINY_ARCH, 2, 8
    blob = synth.make_weights(arch, 0)
    inputs = _inputs(arch, B, [n] * 8)
    want = _reference(arch, "f32", blob, B, n, inputs)
    dec = dc.Decoder(arch, "f32", blob, B, n, n, flags=dc.DC_NO_GRAPH, rng_seed=7)
    tok = torch.zeros_like(inputs[0][0])
    first = dec.decode(inputs[0][0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        pcm = dec.decode(tok)
    got = [first]
    for i in range(1, 8):
        if i % 3 == 0:
            got.append(dec.decode(inputs[i][0]))
        else:
            tok.copy_(inputs[i][0])
            g.replay()
            got.append(pcm.clone())
        if i % 2:
            torch.cuda.synchronize()
    torch.cuda.synchronize()
    for i, (w, o) in enumerate(zip(want, got)):
        assert bits_equal(o.cpu().numpy(), w), f"call {i}"
    del g
    dec.close()


def test_refused_calls_launch_nothing():
    arch = synth.TINY_ARCH
    blob = synth.make_weights(arch, 0)
    dec = dc.Decoder(arch, "f32", blob, 1, 8)
    tok = torch.zeros((1, 8), dtype=torch.int32, device="cuda")
    out = torch.empty((1, 8 * dec.spt), device="cuda")
    f0 = torch.zeros((1, 8), device="cuda")
    assert dc.dc_decode_chunk_on(dec.h, 0, tok, f0, 8, out) == dc.DC_EINVAL     # no source
    assert dc.dc_decode_chunk_on(dec.h, 0, None, None, 8, out) == dc.DC_EINVAL
    assert dc.dc_decode_chunk_on(dec.h, 0, tok, None, 9, out) == dc.DC_ERANGE
    assert dc.dc_decode_chunk_on(ctypes.c_void_p(None), 0, tok, None, 8, out) == dc.DC_EINVAL
    assert dec.stats()["calls"] == 0 and dec.stats()["rejected"] == 3
    host = dc.Decoder(arch, "f32", blob, 1, 8, flags=dc.DC_HOST_PTRS)
    assert dc.dc_decode_chunk_on(host.h, 0, tok, None, 8, out) == dc.DC_EINVAL
    nsf = dc.Decoder(synth.TINY_NSF_ARCH, "f32", synth.make_weights(synth.TINY_NSF_ARCH, 0), 1, 8)
    assert dc.dc_decode_chunk_on(nsf.h, 0, tok, None, 8, out) == dc.DC_EINVAL   # f0 missing
    for d in (dec, host, nsf):
        d.close()
