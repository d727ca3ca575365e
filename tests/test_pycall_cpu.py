"""The CPython module between the binding and the C ABI: every argument arrives where the header says, for tensors, absent tensors,
views, numbers of other types; what is no descriptor is refused; an error of a tensor comes through.  The C functions are
replaced by callbacks that note what they get."""
import ctypes
import os
import sysconfig

import numpy as np
import pytest
import torch

import paper_2602_01053_amd as lra
from paper_2602_01053_amd import binding as B
from paper_2602_01053_amd import build

vp, i32 = ctypes.c_void_p, ctypes.c_int32


@pytest.fixture(params=["module", "ctypes"])
def noted(request, monkeypatch):
    """The binding bound to callbacks, through the CPython module and by ctypes: (list of calls, status to return)."""
    lib = lra.load_library()
    calls, status = [], [0]

    def note(name):
        def f(*args):
            calls.append((name, args))
            return status[0]
        return f

    P = ctypes.POINTER
    fd = ctypes.CFUNCTYPE(ctypes.c_int, P(B.LraShape), P(B.LraCache), P(B.LraAdapters), vp, vp, vp, i32, i32, vp, vp, ctypes.c_size_t,
                          vp, vp)(lambda sh, c, ad, *r: note("decode")(sh[0].rank, c[0].max_seq_len, ad[0].b_k, ad[0].b_v, ad[0].n_adapters, *r))
    fp = ctypes.CFUNCTYPE(ctypes.c_int, P(B.LraShape), P(B.LraCache), P(B.LraAdapters), vp, i32, i32, i32, vp, vp, ctypes.c_size_t,
                          vp, vp)(lambda sh, c, ad, *r: note("prefill")(sh[0].rank, c[0].max_seq_len, ad[0].b_k, ad[0].b_v, ad[0].n_adapters, *r))
    fa = ctypes.CFUNCTYPE(ctypes.c_int, P(B.LraShape), P(B.LraCache), P(B.LraProjection), vp, i32, i32, vp, ctypes.c_size_t, vp, vp)(
        lambda sh, c, pr, *r: note("append")(sh[0].rank, c[0].max_seq_len, pr[0].w, pr[0].d_model, pr[0].rope_theta, *r))
    if request.param == "ctypes":
        monkeypatch.setattr(B, "_calls", B._CtypesCalls(fd, fp, fa))
        monkeypatch.setattr(B, "_stream_ptr", lambda s: 4003 if s is None else s.cuda_stream)
        yield calls, status
        return
    mod = B._entry_points()
    mod.bind(*[ctypes.cast(f, vp).value for f in (fd, fp, fa)], ctypes.addressof(B._tuning), B.LraShape, B.LraCache,
             lambda: 3, lambda dev: 4000 + dev, lambda: True)
    yield calls, status
    monkeypatch.undo()
    B._lib = None
    lra.load_library()
    assert lib is not None


def _descriptors():
    q = torch.zeros(6, 4, 64)
    k = torch.zeros(50, 4, 64)
    lens = torch.tensor([50], dtype=torch.int32)
    return q, lra.make_shape(q, 4, 8), lra.make_cache(k, k, torch.zeros(50, 8), lens, 50), lens


def test_arguments_arrive(noted):
    calls, status = noted
    q, shape, cache, lens = _descriptors()
    b = torch.zeros(3, 8, 256)
    out, ws = torch.empty_like(q), torch.empty(512, dtype=torch.uint8)
    tun = ctypes.addressof(B._tuning)
    lra.lra_attn_decode(shape, cache, b, b[1:], 3, q, lens, lens[:1], np.int64(2), out, ws)
    lra.lra_attn_decode(shape, cache, None, b, 2.0, q[2:], lens, lens, 1, out, None, stream=type("S", (), {"cuda_stream": 77})())
    lra.lra_attn_prefill(shape, cache, b, None, 1, q, 5, 1, out, ws[256:], None)
    x, w = torch.zeros(7, 128), torch.zeros(520, 128)
    lra.lra_cache_append(shape, cache, w, 10000, x, 0, workspace=ws)
    lra.lra_cache_append(shape, cache, w, 0.5, x[3:], True)
    p = lambda t: t.data_ptr()
    assert calls == [
        ("decode", (8, 50, p(b), p(b) + 8192, 3, p(q), p(lens), p(lens), 6, 2, p(out), p(ws), 512, tun, 4003)),
        ("decode", (8, 50, None, p(b), 2, p(q) + 2048, p(lens), p(lens), 4, 1, p(out), None, 0, tun, 77)),
        ("prefill", (8, 50, p(b), None, 1, p(q), 5, 1, 6, p(out), p(ws) + 256, 256, tun, 4003)),
        ("append", (8, 50, p(w), 128, 10000.0, p(x), 0, 7, p(ws), 512, tun, 4003)),
        ("append", (8, 50, p(w), 128, 0.5, p(x) + 3 * 512, 1, 4, None, 0, tun, 4003)),
    ]
    status[0] = 5
    with pytest.raises(lra.LraError, match="workspace"):
        lra.lra_attn_prefill(shape, cache, b, b, 1, q, 0, 0, out, None)


def test_what_is_refused(noted):
    calls, _ = noted
    q, shape, cache, lens = _descriptors()
    good = dict(shape=shape, cache=cache, b_k=None, b_v=None, n_adapters=1, q=q, query_adapter=lens, seq_query_start=lens,
                max_queries_per_seq=1, out=q, workspace=None)
    for name, value, error in [("shape", cache, TypeError), ("shape", None, TypeError), ("cache", shape, TypeError), ("q", None, AttributeError),
                               ("q", 7, AttributeError), ("n_adapters", None, TypeError), ("workspace", 4096, AttributeError),
                               ("b_v", object(), AttributeError),
                               ("max_queries_per_seq", "x", ValueError)]:
        with pytest.raises((error, ctypes.ArgumentError)):
            lra.lra_attn_decode(**{**good, name: value})
    x = torch.zeros(4, 128)
    with pytest.raises(lra.LraError):
        lra.lra_cache_append(shape, cache, x[:, :64], 0.0, x, 0)
    with pytest.raises(TypeError):
        lra.lra_cache_append(shape, cache, x, None, x, 0)
    assert not calls


def test_library_without_the_module(monkeypatch, tmp_path, capfd):
    """No module for this interpreter: the library is loaded and called by ctypes; a build without its headers makes none
    and leaves no stale one."""
    lra.load_library()
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_calls", None)
    monkeypatch.setattr(B, "PYCALL_PATH", str(tmp_path / "none.so"))
    assert lra.lra_status_string(0) == "ok" and isinstance(B._entry_points(), B._CtypesCalls)
    q, shape, cache, lens = _descriptors()
    with pytest.raises(lra.LraError):  # (refused before any launch: no adapter)
        lra.lra_attn_decode(shape, cache, None, None, 0, q, lens, lens, 1, q, None, stream=type("S", (), {"cuda_stream": 0})())
    stale = tmp_path / "stale.so"
    stale.write_bytes(b"x")
    monkeypatch.setattr(build, "PYCALL_PATH", str(stale))
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert not build.build_pycall("hipcc") and not stale.exists() and "ctypes" in capfd.readouterr().out


def test_stream_hooks_come_as_a_pair(monkeypatch):
    """Without the current device the raw stream of some device would be another stream than the caller's."""
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("S", (), {"cuda_stream": 99})())
    both = type("C", (), {"_cuda_getCurrentRawStream": staticmethod(lambda d: 10 + d), "_cuda_getDevice": staticmethod(lambda: 3)})
    raw, device = B._stream_hooks(both)
    assert raw(device()) == 13
    for missing in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        one = type("C", (), {k: staticmethod(getattr(both, k)) for k in ("_cuda_getCurrentRawStream", "_cuda_getDevice") if k != missing})
        raw, device = B._stream_hooks(one)
        assert raw(device()) == 99


def test_module_is_this_interpreters():
    """Its name carries the interpreter's ABI, so that another one finds no module rather than a foreign binary."""
    lra.load_library()
    assert B.PYCALL_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and len(sysconfig.get_config_var("EXT_SUFFIX")) > len(".so")
    assert os.path.realpath(B._entry_points().__file__) == os.path.realpath(B.PYCALL_PATH)
