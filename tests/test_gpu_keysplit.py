"""GPU parity of the launches that deal a workgroup's key tiles to several
wavefront groups (at most 512 workgroups of 64 queries and walks of at least 8
tiles; refreshes of at most 256 workgroups), at the edges of that rule, against
float64 attention on the same bf16 inputs, and of the one-pass and two-phase
refresh on both sides of the rule between them.  Bars: those of the attention
parity tests (max 1e-2, mean 1e-3 for unit-variance V; the fp32 residual R
carries the same probability rounding)."""
import pytest
import torch

from paper_2406_08552_amd import dfa
from tests.test_gpu_parity import MAX_ABS, MEAN_ABS, Guarded, say

pytestmark = pytest.mark.gpu


def _attn64(Q, K, V, w=None):
    S = torch.matmul(Q, K.transpose(-1, -2).contiguous()) / Q.shape[-1] ** 0.5
    if w is not None:
        i = torch.arange(Q.shape[-2], device=Q.device)
        S.masked_fill_((i[:, None] - i[None, :]).abs() > w, float("-inf"))
    return torch.matmul(torch.softmax(S, -1), V)


def _check(name, got, ref):
    err = (got.double() - ref).abs()
    assert torch.isfinite(got).all(), f"{name}: non-finite output"
    mx, mn = float(err.max()), float(err.mean())
    assert mx <= MAX_ABS and mn <= MEAN_ABS, f"{name}: max abs {mx:.3e}, mean abs {mn:.3e}"


# (B, H, L, d, w)
@pytest.mark.parametrize("B,H,L,d,w", [
    (1, 1, 449, 72, 200),       # 8 tiles, the last of one key
    (1, 2, 512, 64, 192),       # 8 whole tiles; a window of 8 tiles
    (2, 1, 515, 72, 16),        # refresh groups with a narrow band; the window in one group
    (1, 3, 1000, 64, 250),      # ragged last tile in the third of four groups
    (2, 8, 1024, 72, 256),      # 256 workgroups
    (1, 17, 1000, 72, 300),     # 272 workgroups: two groups
    (4, 16, 450, 64, 448),      # 512 workgroups, a band one key short of all
    (1, 2, 3000, 72, 200),      # windows of which some groups see nothing
    (1, 4, 70, 72, 20),         # a refresh of two tiles
    (3, 5, 65, 64, 16),         # the second tile of one key
    # more than 256 workgroups, one group: the refresh's one-pass form and its last length
    (2, 16, 577, 72, 72),
    (2, 7, 1280, 64, 160),
    (1, 14, 1280, 72, 700),
    (2, 7, 1281, 72, 160),      # two phases
    # 769 to 1024 workgroups at d = 72: one pass up to a band of 3/8 of the keys to each side
    (4, 16, 896, 72, 336),
    (4, 16, 896, 72, 337),
    (4, 16, 897, 72, 447),
    (5, 16, 600, 72, 300),
    (3, 16, 1100, 72, 137),     # one pass
    (3, 16, 1100, 72, 600),     # two phases, two query blocks per wavefront
    (3, 16, 1100, 64, 137),     # one pass
    # more workgroups: bands of 3/4 of the keys, and of half of them beyond 1024 tokens, in two phases
    (8, 16, 769, 72, 577),      # one query block per wavefront
    (8, 16, 769, 72, 576),      # one pass
    (4, 18, 1100, 72, 549),     # one pass
    (4, 18, 1100, 72, 550),
    (1, 277, 1100, 72, 137),    # 4986: one pass
    (1, 278, 1100, 72, 137),    # 5004: two phases
])
@pytest.mark.parametrize("spread", [1.0, 3.0])
def test_keysplit_vs_fp64(B, H, L, d, w, spread):
    dev = torch.device("cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(L + w)
    # spread: scores of standard deviation spread^2, so that the groups'
    # running maxima differ by many times the rescale margin
    Q, K = ((torch.randn((B, H, L, d), generator=g, device=dev) * spread).to(torch.bfloat16) for _ in range(2))
    V = torch.randn((B, H, L, d), generator=g, device=dev).to(torch.bfloat16)
    Qd, Kd, Vd = Q.double(), K.double(), V.double()
    full, win = _attn64(Qd, Kd, Vd), _attn64(Qd, Kd, Vd, w)
    O, R = Guarded((B, H, L, d), dev), Guarded((B, H, L, d), dev, torch.float32)
    say(f"keysplit B={B} H={H} L={L} d={d} w={w} spread={spread}")
    # near one-hot rows: outputs of size 1 to 4, whose bf16 rounding alone is 1.1e-3 on average and up to 2^-7
    bar = 4 if spread > 1 else 1
    dfa.dfa_attn_full(Q, K, V, O.t, 0)
    torch.cuda.synchronize()
    _check("full", O.t.float() / bar, full / bar)
    full_bits = O.t.clone()
    dfa.dfa_attn_full_and_residual(Q, K, V, O.t, R.t, w)
    torch.cuda.synchronize()
    _check("refresh O", O.t.float() / bar, full / bar)
    _check("refresh R", R.t / bar, (full - win) / bar)
    dfa.dfa_attn_window_plus_residual(Q, K, V, O.t, R.t, w)
    torch.cuda.synchronize()
    _check("window + R", O.t.float() / bar, full / bar)
    dfa.dfa_attn_window_plus_residual(Q, K, V, O.t, None, w)
    torch.cuda.synchronize()
    _check("window", O.t.float() / bar, win / bar)
    # a band that covers every key is full attention, bit for bit, and leaves no residual
    dfa.dfa_attn_window_plus_residual(Q, K, V, O.t, None, L - 1)
    dfa.dfa_attn_full_and_residual(Q, K, V, torch.empty_like(O.t), R.t, L - 1)
    torch.cuda.synchronize()
    assert torch.equal(O.t, full_bits)
    assert not R.t.any()
    assert O.guards_intact() and R.guards_intact()
