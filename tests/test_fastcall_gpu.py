"""The binding's native call path: what it takes gives the bits of the step-by-step path, and what it does not take it leaves to that
(views, streams, outputs to allocate, scalars of other types) or to its errors."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _tensors(dev, dt):
    g = torch.Generator(device=dev).manual_seed(3)
    n = lambda *s: torch.randn(s, generator=g, device=dev, dtype=torch.float32).to(dt)
    return dict(A=n(33, 72), B=n(72, 48), Bt=n(48, 72), bias=n(48), Q=n(2, 3, 20, 64), K=n(2, 3, 33, 64), V=n(2, 3, 33, 64),
                q=n(2, 3, 64), Kc=n(6, 3, 16, 64), Vc=n(6, 3, 16, 64), table=torch.arange(6, device=dev, dtype=torch.int32).reshape(2, 3),
                lens=torch.tensor([40, 17], device=dev, dtype=torch.int32))


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
def test_native_and_python_paths_agree(dt, monkeypatch):
    from paper_2503_14985_amd import binding as b
    dev = torch.device("cuda:0")
    t = _tensors(dev, dt)
    s = 1 / math.sqrt(64)
    empty = lambda *shape: torch.empty(shape, device=dev, dtype=dt)
    wide = empty(33, 60)
    c32 = torch.randn(33, 48, device=dev)
    calls = [lambda: b.mlt_gemm(t["A"], t["B"], C=empty(33, 48)), lambda: b.mlt_gemm(t["A"], t["Bt"], C=empty(33, 48), transB=True),
             lambda: b.mlt_gemm(t["A"][::2], t["B"], C=wide[:17, 5:53]), lambda: b.mlt_gemm(t["A"][:1], t["B"], C=empty(1, 48)),
             lambda: b.mlt_gemm_bias_act(t["A"], t["B"], t["bias"], 2, C=empty(33, 48)), lambda: b.mlt_gemm_bias_act(t["A"], t["B"], None, 1, C=empty(33, 48)),
             lambda: b.mlt_gemm_acc(t["A"], t["Bt"], c32.clone(), transB=True),
             lambda: b.mlt_mha_fwd(t["Q"], t["K"], t["V"], s, causal=True, O=torch.empty_like(t["Q"])), lambda: b.mlt_mha_fwd(t["Q"], t["K"], t["V"], -s, O=torch.empty_like(t["Q"])),
             lambda: b.mlt_paged_attn_decode(t["q"], t["Kc"], t["Vc"], t["table"], t["lens"], s, O=torch.empty_like(t["q"]))]
    taken = []
    native = {f: getattr(b._fast, f) for f in ("gemm", "gemm_bias_act", "gemm_acc", "mha_fwd", "paged_attn_decode")}

    class Fast:
        def __getattr__(self, f):
            def call(*a):
                r = native[f](*a)
                taken.append(r is not None)
                return r
            return call

    class Off:
        def __getattr__(self, f):
            return lambda *a: None

    monkeypatch.setattr(b, "_fast", Fast())
    got = [c().clone() for c in calls]
    assert taken == [True] * len(calls)
    monkeypatch.setattr(b, "_fast", Off())
    for c, g in zip(calls, got):
        w = c()
        assert torch.equal(w.view(torch.int16), g.view(torch.int16))


def test_what_the_native_path_leaves_alone():
    from paper_2503_14985_amd import binding as b
    dev = torch.device("cuda:0")
    t = _tensors(dev, torch.bfloat16)
    f, C, side = b._fast, torch.empty(33, 48, device=dev, dtype=torch.bfloat16), torch.cuda.Stream(device=dev)
    O = torch.empty_like(t["Q"])

    class Sub(torch.Tensor):
        pass

    for args in ((t["A"], t["B"], None, False, None), (t["A"], t["B"], C, False, side), (t["A"], t["B"], C, 0, None), (t["A"].cpu(), t["B"], C, False, None),
                 (t["A"].half(), t["B"], C, False, None), (t["A"], t["Bt"], C, False, None), (t["A"].t(), t["B"], C, False, None), (t["A"], t["B"].t().contiguous().t(), C, False, None),
                 (t["A"].as_subclass(Sub), t["B"], C, False, None), (t["A"], t["B"], C.float(), False, None), (t["A"][:32], t["B"], C, False, None), (1, 2, 3, False, None)):
        assert f.gemm(*args) is None
    assert f.gemm_bias_act(t["A"], t["B"], t["bias"][:40], 2, C, False, None) is None
    assert f.gemm_bias_act(t["A"], t["B"], t["bias"], 7, C, False, None) is None
    assert f.gemm_acc(t["A"], t["B"], C, False, None) is None
    assert f.mha_fwd(t["Q"], t["K"], t["V"], 1, False, O, None) is None                       # an int scale
    with pytest.raises(b.MltError):
        f.mha_fwd(t["Q"], t["K"], t["V"], float("nan"), False, O, None)                        # the library's refusal
    assert f.mha_fwd(t["Q"].transpose(1, 2), t["K"], t["V"], 1.0, False, O, None) is None
    assert f.paged_attn_decode(t["q"], t["Kc"], t["Vc"], t["table"].long(), t["lens"], 1.0, torch.empty_like(t["q"])) is None
    with pytest.raises(b.MltError):
        b.mlt_mha_fwd(t["Q"], t["K"], t["V"], float("nan"), O=O)
    with pytest.raises(ValueError):
        b.mlt_gemm(t["A"], t["Bt"], C=C)
    with torch.cuda.stream(side):                             # the current stream is the one that is used
        side.wait_stream(torch.cuda.default_stream())
        torch.cuda._sleep(20_000_000)
        A2 = t["A"] * 2
        b.mlt_gemm(A2, t["B"], C=C)
    side.synchronize()
    assert torch.equal(C, b.mlt_gemm(A2, t["B"]))


def test_a_failed_call_is_made_once():
    import ctypes
    from paper_2503_14985_amd import binding as b
    t = _tensors(torch.device("cuda:0"), torch.bfloat16)
    C = torch.zeros(33, 48, device="cuda:0")
    calls = []
    refuse = ctypes.CFUNCTYPE(ctypes.c_int, *b.raw().mlt_gemm_acc.argtypes)(lambda *a: calls.append(a) or b.MLT_ERR_LAUNCH)
    names = ("mlt_gemm", "mlt_gemm_bias_act", "mlt_gemm_acc", "mlt_mha_fwd", "mlt_paged_attn_decode")
    own = {f: ctypes.cast(getattr(b.raw(), f), ctypes.c_void_p).value for f in names}
    try:
        b._fast.bind(b.MltError, *({**own, "mlt_gemm_acc": ctypes.cast(refuse, ctypes.c_void_p).value}[f] for f in names))
        with pytest.raises(b.MltError) as e:
            b.mlt_gemm_acc(t["A"], t["B"], C)
    finally:
        b._fast.bind(b.MltError, *(own[f] for f in names))
    assert e.value.status == b.MLT_ERR_LAUNCH and str(e.value).startswith("mlt_gemm_acc:")
    assert len(calls) == 1 and not C.any()
