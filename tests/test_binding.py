"""The native argument marshalling of the binding: it declines (-1) every call
that is not an ordinary one, so that the general Python path raises the same
errors as ever, and an ordinary call gives what the general path gives (which
an explicit stream argument takes)."""
import numpy as np
import pytest
import torch

from paper_2406_08552_amd import build, dfa


class _Sub(torch.Tensor):
    pass


def test_declines_unusual_arguments():
    n = dfa._native()
    t = torch.zeros(1, 2, 64, 64, dtype=torch.bfloat16)
    assert n.plan_step(0, t, t, t, t, None, None, 3) == -1                 # CPU tensors
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
def test_native_calls_match_the_general_path():
    dev = torch.device("cuda")
    B, H, L, d, w = 2, 16, 100, 72, 20
    C = H * d
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    r = lambda shape, dt=torch.bfloat16: torch.randn(shape, generator=g, device=dev).to(dt)  # noqa: E731
    Q, K, V = (r((B, H, L, d)) for _ in range(3))
    X, Wq, bq, Wo, bo = r((B, L, C)), r((3 * C, C)), r((3 * C,), torch.float32), r((C, C)), r((C,), torch.float32)
    stream = torch.cuda.current_stream()

    def both(call):
        outs = []
        for st in (None, stream):
            O, R = torch.zeros((B, H, L, d), dtype=torch.bfloat16, device=dev), torch.ones((B, H, L, d), device=dev)
            Y, res = torch.zeros((B, L, C), dtype=torch.bfloat16, device=dev), torch.zeros(1, dtype=torch.float64, device=dev)
            call(O, R, Y, res, st)
            torch.cuda.synchronize()
            outs.append((O, R, Y, res))
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
    # the current stream is the one of the caller's context
    side = torch.cuda.Stream()
    O, ref = torch.empty_like(Q), torch.empty_like(Q)
    dfa.dfa_attn_full(Q, K, V, ref)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        dfa.dfa_attn_full(Q, K, V, O)
    side.synchronize()
    assert torch.equal(O, ref)
