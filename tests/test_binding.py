"""The native argument marshalling of the binding: it declines (-1) every call
that is not an ordinary one, so that the general Python path raises the same
errors as ever, and an ordinary call gives what the general path gives (which
an explicit stream argument takes)."""
import ctypes
import importlib.util
import shutil

import numpy as np
import pytest
import torch

from paper_2406_08552_amd import build, dfa


class _Sub(torch.Tensor):
    pass


def test_declines_cpu_tensors():
    """Whatever the other arguments are: each is looked at without a fault, and
    the general path raises.  What each check alone declines is in
    test_each_check_alone_declines, which needs GPU tensors."""
    n = dfa._native()
    t = torch.zeros(1, 2, 64, 64, dtype=torch.bfloat16)
    assert n.attn(0, t, t, t, t, None, 3) == -1
    assert n.plan_step(0, t, t, t, t, None, None, 3) == -1
    assert n.attn(0, None, t, t, t, None, 3) == -1
    assert n.attn(0, t.as_subclass(_Sub), t, t, t, None, 3) == -1
    assert n.attn(0, t, t, t, t, None, 3.0) == -1
    assert n.attn(0, t, t, t, t, None, 1 << 40) == -1
    assert n.attn(3, t, t, t, t, None, 3) == -1
    assert n.qkv_proj(t, t, None, t, t, t) == -1
    assert n.out_proj(t, t, None, None) == -1
    assert n.module_step(0, *[t] * 12, 3, 2) == -1
    assert n.mrae(t, t, t, t) == -1
    assert n.plan_step() == -1
    with pytest.raises(ValueError, match="GPU"):
        dfa.dfa_plan_step(0, t, t, t, t, None, None, 3)
    with pytest.raises(TypeError, match="bf16|bfloat16"):
        dfa.dfa_attn_full(t.float(), t, t, t)


_vp, _int = ctypes.c_void_p, ctypes.c_int
_TYPES = {   # the library functions' arguments, in the order init takes them
    "full": [_vp] * 5 + [_int] * 5 + [_vp], "refresh": [_vp] * 5 + [_int] * 5 + [_vp],
    "window": [_vp] * 5 + [_int] * 5 + [_vp], "plan": [_int] + [_vp] * 6 + [_int] * 5 + [_vp],
    "qkv": [_vp] * 6 + [_int] * 4 + [_vp], "out": [_vp] * 4 + [_int] * 4 + [_vp],
    "module": [_int] + [_vp] * 12 + [_int] * 5 + [_vp],
    "mrae": [_vp, _vp, ctypes.c_size_t, _vp, _vp, _vp],
}


@pytest.fixture
def recorder(tmp_path):
    """A copy of the extension bound to functions that record their arguments
    and launch nothing, and the list of what they recorded."""
    path = tmp_path / "_dfa_binding.so"
    shutil.copy(dfa.BINDING_PATH, path)   # a file of its own: the functions it is bound to are per loaded file
    spec = importlib.util.spec_from_file_location("_dfa_binding", str(path))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    calls, keep = [], []
    for name, types in _TYPES.items():
        keep.append(ctypes.CFUNCTYPE(_int, *types)(lambda *a, name=name: calls.append((name, *a)) or 0))
    mod.init(torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, *[ctypes.cast(f, _vp).value for f in keep])
    mod.keep = keep
    return mod, calls


def _ordinary():
    """name -> (function, arguments, positions that may be None, what the
    library is called with but for the stream)."""
    B, H, L, d, w = 2, 16, 10, 72, 3
    C = H * d
    bf = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    f32 = lambda *s: torch.zeros(s, device="cuda")  # noqa: E731
    Q, K, V, O, Oc, R = *(bf(B, H, L, d) for _ in range(5)), f32(B, H, L, d)
    X, Y, Yc, Wq, bq, Wo, bo = bf(B, L, C), bf(B, L, C), bf(B, L, C), bf(3 * C, C), f32(3 * C), bf(C, C), f32(C)
    ws, res = torch.zeros(8192, dtype=torch.uint8, device="cuda"), torch.zeros(2, dtype=torch.float64, device="cuda")
    p = lambda *ts: [t.data_ptr() for t in ts]  # noqa: E731
    at = [Q, K, V, O, R]
    cases = {f"attn {i}": ("attn", [i, *at, w], (2, 3, 4, 5), [name, *p(*at), B, H, L, d, w])
             for i, name in enumerate(("full", "refresh", "window"))}
    cases["plan"] = ("plan_step", [1, *at, Oc, w], (1, 2, 3, 5, 6), ["plan", 1, *p(*at, Oc), B, H, L, d, w])
    cases["qkv"] = ("qkv_proj", [X, Wq, bq, Q, K, V], (1, 2), ["qkv", *p(X, Wq, bq, Q, K, V), B, H, L, d])
    cases["out"] = ("out_proj", [O, Wo, bo, Y], (1, 2), ["out", *p(O, Wo, bo, Y), B, H, L, d])
    m = [X, Wq, bq, Wo, bo, Q, K, V, O, R, Y, Yc]
    cases["module"] = ("module_step", [1, *m, w, H], (*range(1, 11), 12), ["module", 1, *p(*m), B, H, L, d, w])
    cases["mrae"] = ("mrae", [Q, K, ws, res], (), ["mrae", *p(Q, K), Q.numel(), *p(ws, res)])
    return cases


@pytest.mark.gpu
def test_native_calls_hand_over_addresses_sizes_and_stream(recorder):
    mod, calls = recorder
    side = torch.cuda.Stream()
    for name, (fn, args, nullable, want) in _ordinary().items():
        for stream in (torch.cuda.current_stream(), side):
            with torch.cuda.stream(stream):
                assert getattr(mod, fn)(*args) == 0, name
            assert calls == [(*want, stream.cuda_stream or None)], name
            calls.clear()
        off = 2 if isinstance(want[1], int) and fn in ("plan_step", "module_step") else 1
        for i in nullable:   # a null pointer in its place; the library says whether it may be
            assert getattr(mod, fn)(*args[:i], None, *args[i + 1:]) == 0, (name, i)
            lib = list(want)
            lib[off + i - (0 if fn in ("qkv_proj", "out_proj") else 1)] = None
            assert calls == [(*lib, torch.cuda.current_stream().cuda_stream or None)], (name, i)
            calls.clear()
    code = _ordinary()["plan"]
    assert mod.plan_step(np.int32(2), *code[1][1:]) == 0 and calls.pop()[1] == 2   # a plan's element


@pytest.mark.gpu
def test_each_check_alone_declines(recorder):
    """Every argument of an ordinary call in turn is made unordinary in one way:
    the call is declined, and the library is not called."""
    mod, calls = recorder
    for name, (fn, args, nullable, _) in _ordinary().items():
        f = getattr(mod, fn)

        def declined(i, value, why):
            status = f(*args[:i], value, *args[i + 1:])
            assert status == -1 and not calls, (name, i, why)

        for i, a in enumerate(args):
            if isinstance(a, torch.Tensor):
                workspace = a.dtype == torch.uint8      # any type and size from 8 KiB
                spread = torch.zeros((*a.shape, 2), dtype=a.dtype, device=a.device)[..., 0]
                assert spread.shape == a.shape and not spread.is_contiguous()
                declined(i, spread, "not contiguous")
                if not workspace:
                    declined(i, a.to(torch.float16), "type")
                smaller = a[:0] if a.dtype == torch.float64 else a[..., :-8].contiguous()
                declined(i, smaller, "shape")
                declined(i, a.as_subclass(_Sub), "subclass")
                declined(i, a.cpu(), "CPU")
                declined(i, a.data_ptr(), "no tensor")
                if i not in nullable:
                    declined(i, None, "None")
            else:
                for value in (float(a), 1 << 40, -(1 << 40), 1 << 80, None, "1"):
                    declined(i, value, value)
        if fn == "attn":
            declined(0, 3, "no such function")
            declined(0, -1, "no such function")
        if fn == "module_step":
            for heads in (0, -1, 7):
                declined(14, heads, "heads")
        assert f(*args[:-1]) == -1 and f(*args, args[-1]) == -1 and f() == -1 and not calls, (name, "number of arguments")


def test_library_builds_with_hipcc_alone(monkeypatch):
    made = []
    monkeypatch.setattr(build, "_compile", lambda cmd, path, verbose: made.append((cmd[0], path)))
    assert build.build_library() == build.LIB_PATH
    assert made == [(build.hipcc(), build.LIB_PATH)]
    assert build.build_binding() == build.BINDING_PATH
    assert [p for _, p in made] == [build.LIB_PATH, build.BINDING_PATH]


def test_calls_without_the_extension(monkeypatch, tmp_path):
    """A library built alone is enough for the binding: its general path makes
    the same checks and calls."""
    monkeypatch.setattr(dfa, "BINDING_PATH", str(tmp_path / "missing.so"))
    monkeypatch.setattr(dfa, "_NATIVE", None)
    t = torch.zeros(1, 2, 64, 64, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="GPU"):
        dfa.dfa_plan_step(0, t, t, t, t, None, None, 3)
    with pytest.raises(ValueError, match="GPU"):
        dfa.dfa_attn_full(t, t, t, t)
    if torch.cuda.is_available():
        Q, K, V = (torch.randn(1, 2, 64, 64, device="cuda").to(torch.bfloat16) for _ in range(3))
        O = torch.zeros_like(Q)
        dfa.dfa_attn_full(Q, K, V, O)
        assert bool(O.any())


def test_torch_without_gpu_support(monkeypatch):
    """CPU tensors are refused with the general path's message there too."""
    for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
        monkeypatch.delattr(torch._C, name)
    monkeypatch.setattr(dfa, "_NATIVE", None)
    t = torch.zeros(1, 2, 64, 64, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="GPU"):
        dfa.dfa_plan_step(0, t, t, t, t, None, None, 3)


@pytest.mark.gpu
def test_native_calls_match_the_general_path(monkeypatch):
    dev = torch.device("cuda")
    B, H, L, d, w = 2, 16, 100, 72, 20
    C = H * d
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    r = lambda shape, dt=torch.bfloat16: torch.randn(shape, generator=g, device=dev).to(dt)  # noqa: E731
    Q, K, V = (r((B, H, L, d)) for _ in range(3))
    X, Wq, bq, Wo, bo = r((B, L, C)), r((3 * C, C)), r((3 * C,), torch.float32), r((C, C)), r((C,), torch.float32)
    stream = torch.cuda.current_stream()

    native, made = dfa._native(), []

    class Spy:
        def __getattr__(self, name):
            return lambda *a: made.append(getattr(native, name)(*a)) or made[-1]

    monkeypatch.setattr(dfa, "_NATIVE", Spy())

    def both(call):
        outs = []
        made.clear()
        for st in (None, stream):
            O, R = torch.zeros((B, H, L, d), dtype=torch.bfloat16, device=dev), torch.ones((B, H, L, d), device=dev)
            Y, res = torch.zeros((B, L, C), dtype=torch.bfloat16, device=dev), torch.zeros(1, dtype=torch.float64, device=dev)
            call(O, R, Y, res, st)
            torch.cuda.synchronize()
            outs.append((O, R, Y, res))
        assert made == [0]   # the native call was made, the explicit stream took the general path
        assert all(torch.equal(a, b) for a, b in zip(*outs))
        assert any(bool(t.any()) for t in (outs[0][0], outs[0][2], outs[0][3]))

    both(lambda O, R, Y, res, st: dfa.dfa_attn_full(Q, K, V, O, stream=st))
    both(lambda O, R, Y, res, st: dfa.dfa_attn_full_and_residual(Q, K, V, O, R, w, stream=st))
    both(lambda O, R, Y, res, st: dfa.dfa_attn_window_plus_residual(Q, K, V, O, R, w, stream=st))
    both(lambda O, R, Y, res, st: dfa.dfa_attn_window_plus_residual(Q, K, V, O, None, w, stream=st))
    for code in (dfa.FULL, dfa.WARS_REFRESH, np.int32(dfa.WARS_REUSE), dfa.ASC_REUSE, dfa.WARS_ASC_REFRESH):
        both(lambda O, R, Y, res, st: dfa.dfa_plan_step(code, Q, K, V, O, R, None, w, stream=st))
        q, k, v, o = (torch.empty_like(Q) for _ in range(4))
        both(lambda O, R, Y, res, st: dfa.dfa_module_step(code, X, Wq, bq, Wo, None, q, k, v, o, R, Y, None, w, H, stream=st))
    both(lambda O, R, Y, res, st: dfa.dfa_qkv_proj(X, Wq, bq, O, torch.empty_like(O), torch.empty_like(O), stream=st))
    both(lambda O, R, Y, res, st: dfa.dfa_out_proj(Q, Wo, bo, Y, stream=st))
    ws = torch.empty(dfa.MRAE_WORKSPACE_BYTES, dtype=torch.uint8, device=dev)
    both(lambda O, R, Y, res, st: dfa.dfa_mrae(Q, K, ws, res, stream=st))
    # a refused call raises the library's error on both paths
    for st in (None, stream):
        with pytest.raises(dfa.DfaError, match="overlaps"):
            dfa.dfa_attn_full(Q, K, V, Q, stream=st)
        with pytest.raises(dfa.DfaError, match="even batch"):
            dfa.dfa_plan_step(dfa.ASC_REUSE, Q[:1], K[:1], V[:1], torch.empty_like(Q[:1]), None, None, w, stream=st)
