"""The decode loop's calls in native code: what they hand to the library, what they make, and what they leave to ctypes."""
import os
import subprocess
import sys
import threading

import pytest
import torch

from paper_2605_08317_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def b():
    from paper_2605_08317_amd import binding
    return binding


class _NoCache:
    def __init__(self, h):
        import types
        self.h, self.cfg = h, types.SimpleNamespace(seq_lens=[5], hq=2, d=128)


def test_errors_are_those_of_the_library_and_of_ctypes(b, monkeypatch):
    import ctypes
    monkeypatch.setattr(b, "_stream", lambda: 0)
    q = torch.zeros(1, 2, 128, dtype=torch.bfloat16)
    for h in (None, 0, ctypes.c_void_p()):
        with pytest.raises(b.RdkvError, match="RDKV_ERR_INVALID_ARG"):
            b.rdkv_decode_attn(_NoCache(h), q)
        for k in (q, None):
            with pytest.raises(b.RdkvError, match="RDKV_ERR_INVALID_ARG"):
                b.rdkv_cache_append(_NoCache(h), k, k)
    odd = torch.zeros(1, 2, 256, dtype=torch.bfloat16)[:, :, ::2]
    for args in ((odd,), (q, odd), (q, None, odd)):
        with pytest.raises(AssertionError):
            b.rdkv_decode_attn(_NoCache(0), *args)
    with pytest.raises(AssertionError):
        b.rdkv_cache_append(_NoCache(0), q, odd)
    with pytest.raises((AttributeError, TypeError)):
        b.rdkv_decode_attn(_NoCache("no handle"), q)


def test_a_subclass_is_asked_for_its_memory(b, monkeypatch):
    asked = []

    class Own(torch.Tensor):
        def data_ptr(self):
            asked.append(1)
            return super().data_ptr()
    monkeypatch.setattr(b, "_stream", lambda: 0)
    q = torch.zeros(1, 2, 128, dtype=torch.bfloat16)
    for args in ((q.as_subclass(Own),), (q, q.float().as_subclass(Own)), (q, None, q.float().as_subclass(Own))):
        with pytest.raises(b.RdkvError):
            b.rdkv_decode_attn(_NoCache(None), *args)
    with pytest.raises(b.RdkvError):
        b.rdkv_cache_append(_NoCache(None), q, q.as_subclass(Own))
    assert len(asked) == 4


@pytest.mark.gpu
def test_results_made_or_given_on_any_stream_and_thread(b):
    wl = W.scaled(W.CONFIGS["tiny"], seq_lens=(700,))
    inp = {k: v.cuda() for k, v in W.make_inputs(wl, device="cpu").items() if k in ("K", "V", "q", "Q_obs")}
    cfg = b.Config([700], wl.hq, wl.hkv, budget_bits=[3.0], s_obs=wl.s_obs)
    cache = b.rdkv_compress(cfg, inp["K"], inp["V"], inp["Q_obs"])
    out, lse = b.rdkv_decode_attn(cache, inp["q"])
    for t, shape in ((out, (1, wl.hq, 128)), (lse, (1, wl.hq))):
        assert t.shape == shape and t.dtype == torch.float32 and t.is_contiguous() and t.device == inp["q"].device and not t.requires_grad
    given = [torch.full_like(out, 7.0), torch.full_like(lse, 7.0)]
    for o, l in ((None, given[1]), (given[0], None), given):
        r = b.rdkv_decode_attn(cache, inp["q"], o, l)
        assert isinstance(r, tuple) and (o is None or r[0] is o) and (l is None or r[1] is l)
        assert torch.equal(r[0], out) and torch.equal(r[1], lse)
    torch.cuda.synchronize()
    bad = []

    def loop():
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(20):
                o, l = b.rdkv_decode_attn(cache, inp["q"])
                stream.synchronize()
                if not (torch.equal(o, out) and torch.equal(l, lse)):
                    bad.append(1)
    thread = threading.Thread(target=loop)
    thread.start()
    thread.join()
    assert not bad
    cache.free()


def test_ctypes_serves_where_the_native_calls_do_not_load():
    """The same errors, and a warning, without _rdkv_call: a missing or unfit one is not needed to import the binding."""
    code = """
import sys, types, warnings
sys.modules["paper_2605_08317_amd._rdkv_call"] = None
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    from paper_2605_08317_amd import binding as b
assert any("_rdkv_call" in str(x.message) for x in w), w
import torch
b._stream = lambda: 0
q = torch.zeros(1, 2, 128, dtype=torch.bfloat16)
cache = types.SimpleNamespace(h=None, cfg=types.SimpleNamespace(seq_lens=[5], hq=2, d=128))
for call in (lambda: b.rdkv_decode_attn(cache, q), lambda: b.rdkv_cache_append(cache, q, q)):
    try:
        call()
    except b.RdkvError as e:
        assert e.status == 1
    else:
        raise SystemExit("no error")
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
