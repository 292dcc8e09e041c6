"""The decode step's native argument marshalling: what is not plainly an accepted call goes to the Python path, which converts or
refuses it as ever; both give the same."""
import contextlib
import ctypes
import sys

import pytest
import torch

import paper_2506_15545_amd
from paper_2506_15545_amd import binding as rb


def tensors(dev, N=2, Hq=4, Hkv=2, D=64, W=16, dtype=torch.float32):
    g = torch.Generator().manual_seed(5900)
    r = lambda *s, dt=dtype: torch.randn(*s, generator=g).to(device=dev, dtype=dt)
    return dict(q=r(N, Hq, D), k_new=r(N, Hkv, D), v_new=r(N, Hkv, D), pos=torch.tensor([3, 40], dtype=torch.int32, device=dev),
                k_ring=r(N, Hkv, W, D), v_ring=r(N, Hkv, W, D), state=r(N, Hkv, D, D, dt=torch.float32))


def native(t, gs=None, gr=None, scale=0.125, eps=1e-6, out=None, phi="softmax"):
    return rb._decode_native(*t.values(), gs, gr, scale, eps, out, phi)


@contextlib.contextmanager
def step_replaced(f):
    """The native path with `f`, a function of libpython that takes nothing and returns an int, in the step's place: nothing is
    launched, and what f returns is the status."""
    rb._load_decode_native()
    lib = rb.lib()
    from paper_2506_15545_amd import _marshal
    addr = lambda g: ctypes.cast(g, ctypes.c_void_p).value
    try:
        _marshal.bind(addr(f), addr(lib.rattn_decode_workspace_bytes))
        yield
    finally:
        _marshal.bind(addr(lib.rattn_decode_step_ws), addr(lib.rattn_decode_workspace_bytes))


def test_host_tensors_are_refused_as_ever():
    t = tensors("cpu")
    assert native(t) is None
    with pytest.raises(ValueError, match="q must be a contiguous device tensor"):
        rb.rattn_decode_step(**t)
    with pytest.raises((ValueError, AttributeError)):
        rb.rattn_decode_step(None, **{k: v for k, v in t.items() if k != "q"})
    with pytest.raises(TypeError):
        rb._decode_native(t["q"])


def test_only_the_decode_step_needs_the_extension(monkeypatch):
    """Without it (or with one built for another torch) everything else loads, and a decode step says what to run."""
    monkeypatch.setitem(sys.modules, "paper_2506_15545_amd._marshal", None)   # importing it raises ImportError
    monkeypatch.delattr(paper_2506_15545_amd, "_marshal", raising=False)
    monkeypatch.setattr(rb, "_lib", None)
    monkeypatch.setattr(rb, "_decode_native", lambda *a: rb._load_decode_native())
    assert rb.rattn_cache_bytes(4, 0, 100, 16, 1, 2, 64, 2) > 0
    with pytest.raises(RuntimeError, match="_marshal.so is not built"):
        rb.rattn_decode_step(**tensors("cpu"))


@pytest.mark.gpu
def test_forms_that_python_converts_or_refuses():
    t = tensors("cuda")
    gain = torch.full((4, 64), 1.25, device="cuda")
    refused = [dict(q=t["q"].transpose(1, 2)), dict(pos=t["pos"].long()), dict(state=t["state"].bfloat16()),
               dict(k_ring=t["k_ring"][:, :, :8].contiguous()), dict(v_new=t["v_new"].bfloat16()), dict(q=t["q"].half()),
               dict(pos=t["pos"][:1].contiguous()), dict(k_new=t["k_new"].cpu())]
    for change in refused:
        bad = {**t, **change}
        assert native(bad) is None, change.keys()
        with pytest.raises(ValueError):
            rb.rattn_decode_step(**bad)
    # the library's own refusals come out as its status
    with pytest.raises(rb.RattnError):
        rb.rattn_decode_step(**t, rms_eps=0.0)
    with pytest.raises(ValueError):
        rb.rattn_decode_step(**t, gamma_swa=gain[:3])
    with pytest.raises(KeyError):
        rb.rattn_decode_step(**t, feature_map="cosine")
    fresh = lambda: {k: v.clone() for k, v in t.items()}
    out = torch.empty_like(t["q"])
    x = fresh()
    assert native(x, gain, None, out=out) is out
    for phi in ("softmax", "relu", "identity"):
        want = rb.rattn_decode_step(**fresh(), gamma_swa=gain, softmax_scale=0.125, feature_map=phi)
        for gs, scale in ((gain.double(), 0.125), (gain.bfloat16(), 0.125), (gain.t().contiguous().t(), 0.125),
                          (gain, torch.tensor(0.125)), (gain.cpu(), 0.125)):
            x = fresh()
            assert native(x, gs, None, scale, phi=phi) is None
            got = rb.rattn_decode_step(**x, gamma_swa=gs, softmax_scale=scale, feature_map=phi)
            assert torch.equal(got, want)
    assert torch.equal(out, rb.rattn_decode_step(**fresh(), gamma_swa=gain, softmax_scale=0.125))
    assert not torch.equal(rb.rattn_decode_step(**fresh(), softmax_scale=1), out)


@pytest.mark.gpu
def test_out_that_cannot_take_the_result_is_refused():
    """The step writes N Hq D elements of q's type: an `out` that does not hold them is refused ahead of any launch (nothing here
    is launched through it), one of another shape that does is taken."""
    t = tensors("cuda")
    N, Hq, D = t["q"].shape
    keep = {k: v.clone() for k, v in t.items()}
    for out in (torch.empty(N, Hq, D), torch.empty(N - 1, Hq, D, device="cuda"), torch.empty(0, device="cuda"),
                torch.empty(N, Hq, D, device="cuda", dtype=torch.bfloat16), torch.empty(N, D, Hq, device="cuda").transpose(1, 2),
                torch.empty(N, Hq, 2 * D, device="cuda")[..., :D]):
        with step_replaced(ctypes.pythonapi.Py_IsInitialized):   # (1)
            assert native(t, out=out) is None
        for scale in (0.125, torch.tensor(0.125)):   # the native path's refusal, the Python path's own
            with pytest.raises(ValueError, match="out must be"):
                rb.rattn_decode_step(**t, softmax_scale=scale, out=out)
    torch.cuda.synchronize()
    assert all(torch.equal(t[k], keep[k]) for k in t)
    want = rb.rattn_decode_step(**{k: v.clone() for k, v in t.items()}, softmax_scale=0.125)
    for scale in (0.125, torch.tensor(0.125)):
        out = torch.empty(N * Hq * D + 8, device="cuda")
        x = {k: v.clone() for k, v in t.items()}
        assert rb.rattn_decode_step(**x, softmax_scale=scale, out=out) is out
        assert torch.equal(out[:N * Hq * D].view(N, Hq, D), want)


@pytest.mark.gpu
@pytest.mark.parametrize("W", [16, 1024])   # without a workspace, with one
def test_other_threads_run_during_the_step(W):
    """The interpreter lock is not held while the step is enqueued, which can wait for the device."""
    t = tensors("cuda", D=128, W=W, dtype=torch.bfloat16)
    with step_replaced(ctypes.pythonapi.PyGILState_Check):   # 1 with the lock held
        assert torch.is_tensor(native(t))


@pytest.mark.gpu
def test_a_result_that_cannot_be_made_stops_the_step():
    """No memory for the result's object: the error comes ahead of the step (whose stand-in would return 1), not behind it."""
    testcapi = pytest.importorskip("_testcapi")
    t = tensors("cuda")
    args = (*t.values(), None, None, 0.125, 1e-6, None, "softmax")
    got = None
    with step_replaced(ctypes.pythonapi.Py_IsInitialized):
        f = rb._decode_native
        assert f(*args) == 1
        testcapi.set_nomemory(0, 0)
        try:
            got = f(*args)
        except MemoryError:
            got = "refused"
        finally:
            testcapi.remove_mem_hooks()
    assert got == "refused"
