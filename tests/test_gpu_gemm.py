"""GPU parity of the projections at the edges of their tile shapes, against
float64 matrix products of the same bf16 operands.

The bar: one rounding to bf16 (at most 2^-8 of the value, twice the half-ulp,
so that an fp32 sum next to a rounding boundary may fall on its other side)
plus 1e-4 for the fp32 accumulation of N(0, 1) sums over at most 1152 terms
(a random walk of 1152 roundings of 2^-24 is about 2e-6)."""
import pytest
import torch

from paper_2406_08552_amd import dfa
from tests.test_gpu_parity import Guarded, say

pytestmark = pytest.mark.gpu


def _randn(g, shape, scale=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale).to(dtype)


def _check(name, got, ref):
    assert torch.isfinite(got).all(), f"{name}: non-finite output"
    err = (got.double() - ref).abs()
    bad = err > 2.0 ** -8 * ref.abs() + 1e-4
    assert not bad.any(), f"{name}: {int(bad.sum())} outputs off, max abs {float(err.max()):.3e}"


def _route(N, M):
    """The tile shape that the library's rule gives N output features of M
    tokens (features x tokens of a workgroup, "ring" or "stream")."""
    tiles = lambda f, t: -(-N // f) * -(-M // t)  # noqa: E731
    n128, n192 = tiles(128, 128), tiles(192, 256)
    if tiles(64, 64) <= 256:
        return "64x64 ring"
    if n128 <= 256:
        return "128x128 ring"
    last = n128 % 512
    rounds = 100 * (n128 // 512) + (0 if last == 0 else 65 if last <= 256 else 100)
    return "192x256 stream" if 125 * -(-n192 // 256) < rounds else "128x128 stream"


R64, R128, S128, S192 = "64x64 ring", "128x128 ring", "128x128 stream", "192x256 stream"


# (B, H, L, d), the tile shape of the QKV projection, then of the output
# projection.  A QKV projection's 3C features are a multiple of 192 (C is one of
# 128); output features need not be.
@pytest.mark.parametrize("B,H,L,d,qkv,out", [
    (1, 2, 1, 64, R64, R64),            # one token, K = 128 (two k-tiles)
    (3, 2, 37, 64, R64, R64),           # ragged token tile, tokens of one tile in several batch entries
    (5, 16, 63, 72, R128, R64),
    (2, 6, 701, 64, R128, R64),         # K = 384
    (3, 16, 683, 72, S128, R128),       # one round, ragged
    (2, 16, 2050, 72, S128, S128),      # last token tile of 4
    (1, 2, 170001, 64, S192, S128),     # K = 128 over many tiles per workgroup
    (1, 6, 60003, 64, S192, S192),      # K = 384, output features a multiple of 192, many tiles, ragged
    (2, 10, 9001, 64, S192, S128),      # K = 640
    (4000, 16, 2, 72, S128, S192),      # a new batch entry every other token
    # output features not a multiple of 192: a last feature tile of 64 (whole and
    # ragged last token tile) and of 128, with further tiles of the same workgroup behind it
    (2, 16, 16384, 64, S192, S192),
    (2, 16, 16350, 64, S192, S192),
    (1, 8, 65003, 64, S192, S192),
])
@pytest.mark.parametrize("bias", [True, False])
def test_projection_tile_edges(B, H, L, d, qkv, out, bias):
    assert (_route(3 * H * d, B * L), _route(H * d, B * L)) == (qkv, out), "not the tile shapes this case is for"
    C = H * d
    g = torch.Generator(device="cuda")
    g.manual_seed(B + 7 * L)
    X, Wqkv, Wo = _randn(g, (B, L, C)), _randn(g, (3 * C, C), C ** -0.5), _randn(g, (C, C), C ** -0.5)
    bqkv = _randn(g, (3 * C,), 0.1, torch.float32) if bias else None
    bo = _randn(g, (C,), 0.1, torch.float32) if bias else None
    dev = torch.device("cuda")
    Q, K, V = (Guarded((B, H, L, d), dev) for _ in range(3))
    say(f"qkv_proj B={B} H={H} L={L} d={d} bias={bias}")
    dfa.dfa_qkv_proj(X, Wqkv, bqkv, Q.t, K.t, V.t)
    torch.cuda.synchronize()
    xd = X.double().view(B * L, C)
    for i, (name, got) in enumerate((("Q", Q), ("K", K), ("V", V))):
        ref = xd @ Wqkv[i * C:(i + 1) * C].double().t().contiguous()
        if bias:
            ref += bqkv[i * C:(i + 1) * C].double()
        _check(f"qkv_proj {name}", got.t, ref.view(B, L, H, d).permute(0, 2, 1, 3))
        assert got.guards_intact(), f"write outside {name}"
    del xd, ref
    O = _randn(g, (B, H, L, d))
    Y = Guarded((B, L, C), dev)
    say(f"out_proj B={B} H={H} L={L} d={d} bias={bias}")
    dfa.dfa_out_proj(O, Wo, bo, Y.t)
    torch.cuda.synchronize()
    ref = O.double().permute(0, 2, 1, 3).reshape(B * L, C) @ Wo.double().t().contiguous()
    if bias:
        ref += bo.double()
    _check("out_proj Y", Y.t, ref.view(B, L, C))
    assert Y.guards_intact(), "write outside Y"
