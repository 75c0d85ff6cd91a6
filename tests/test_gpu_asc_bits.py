"""The codes that compute the conditional half of the batch alone (ASC and the
two WA-RS + ASC codes) give the conditional half of the whole-batch code bit
for bit, also where the half launch has so few workgroups that it would be run
another way than the whole one."""
import pytest
import torch

from paper_2406_08552_amd import dfa
from tests.test_gpu_parity import say

pytestmark = pytest.mark.gpu

PAIRS = [(dfa.FULL, dfa.ASC_REUSE), (dfa.WARS_REFRESH, dfa.WARS_ASC_REFRESH), (dfa.WARS_REUSE, dfa.WARS_ASC_REUSE)]

# (B, H, L, d, w); workgroups of 64 and of 128 queries of the whole call
SHAPES = [
    (2, 16, 1024, 72, 256),     # 512, 256
    (2, 8, 1024, 64, 256),      # 256, 128
    (2, 30, 520, 72, 200),      # 540, 300
    (4, 13, 513, 64, 250),      # 468, 260: the whole call has 128-query workgroups
    (2, 12, 1300, 72, 400),     # 504, 264
    (2, 9, 1500, 64, 700),      # 432, 216: two-phase refresh of the whole call, half of it 216
    (4, 16, 256, 72, 32),       # 256, 128
    (4, 13, 1000, 72, 125),     # 832, 416
    (4, 13, 1000, 72, 500),     # a two-phase refresh, of which the half alone would be one-pass
    (2, 3, 65, 72, 20),         # 12, 12
    (6, 5, 16, 72, 2),          # short sequences
]


@pytest.mark.parametrize("B,H,L,d,w", SHAPES)
def test_conditional_half_is_bitwise(B, H, L, d, w):
    dev = torch.device("cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(3 * L + d)
    Q, K, V = (torch.randn((B, H, L, d), generator=g, device=dev).to(torch.bfloat16) for _ in range(3))
    say(f"ASC bits B={B} H={H} L={L} d={d} w={w}")
    R0 = torch.randn((B, H, L, d), generator=g, device=dev) * 0.1
    n = B // 2
    for whole, half in PAIRS:
        Ow, Oh, Rw, Rh = torch.empty_like(Q), torch.empty_like(Q), R0.clone(), R0.clone()
        dfa.dfa_plan_step(whole, Q, K, V, Ow, Rw, None, w)
        dfa.dfa_plan_step(half, Q, K, V, Oh, Rh, None, w)
        torch.cuda.synchronize()
        name = dfa.CODE_NAMES[half]
        assert torch.equal(Ow[:n], Oh[:n]) and torch.equal(Oh[n:], Oh[:n]), name
        assert torch.equal(Rw[:n], Rh[:n]) and torch.equal(Rh[n:], R0[n:]), name


def test_module_conditional_half_is_bitwise():
    dev = torch.device("cuda")
    B, H, L, d, w = 2, 16, 1024, 72, 256
    C = H * d
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    r = lambda shape, s=1.0: (torch.randn(shape, generator=g, device=dev) * s).to(torch.bfloat16)  # noqa: E731
    X, Wq, Wo = r((B, L, C)), r((3 * C, C), C ** -0.5), r((C, C), C ** -0.5)
    say("ASC bits of a module")
    for whole, half in PAIRS:
        Y = []
        for code in (whole, half):
            Q, K, V, O = (torch.empty((B, H, L, d), dtype=torch.bfloat16, device=dev) for _ in range(4))
            R = torch.full((B, H, L, d), 0.25, device=dev)
            Y.append(torch.empty_like(X))
            dfa.dfa_module_step(code, X, Wq, None, Wo, None, Q, K, V, O, R, Y[-1], None, w, H)
        torch.cuda.synchronize()
        assert torch.equal(Y[0][: B // 2], Y[1][: B // 2]), dfa.CODE_NAMES[half]
