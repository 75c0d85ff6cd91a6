"""The outputs, which leave as rows through LDS or straight from the registers:
every number of valid rows in a wavefront's last block, both head dims, one to
four destinations, against float64 attention.  Bars: those of the attention
parity tests (max 1e-2, mean 1e-3 for unit-variance V; W, O and R of a refresh
carry the same rounding)."""
import pytest
import torch

from paper_2406_08552_amd import dfa
from tests.test_gpu_keysplit import _attn64, _check
from tests.test_gpu_parity import Guarded, say

pytestmark = pytest.mark.gpu


# short kernel (one and two blocks, whole and ragged), 64-query workgroups with
# and without key groups, 128-query workgroups; the second block of a wavefront
# whole, of one row and empty; both sides of the sizes from which outputs leave
# through LDS (1 to 22 MiB of O, with and without a cache), and more than 80 MiB
# of O in short sequences (stored without allocation)
@pytest.mark.parametrize("B,H,L", [(6, 3, 1), (4, 5, 9), (2, 9, 16), (2, 3, 17), (4, 7, 32), (2, 3, 33), (2, 2, 79), (2, 16, 320),
                                   (20, 16, 273), (20, 16, 384), (20, 16, 391), (2, 80, 1400),
                                   (32, 16, 405), (40, 16, 32), (200, 16, 31), (20, 16, 79), (48, 16, 79),
                                   (24, 16, 31), (40, 16, 31), (200, 16, 20), (320, 16, 31), (1400, 16, 31), (14, 16, 79), (12, 16, 45)])
@pytest.mark.parametrize("d", [64, 72])
def test_output_rows(B, H, L, d):
    dev = torch.device("cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(17 * L + d)
    say(f"output rows B={B} H={H} L={L} d={d}")
    w = max(1, L // (2 if L > 1000 else 5))
    Q, K, V = (torch.randn((B, H, L, d), generator=g, device=dev).to(torch.bfloat16) for _ in range(3))
    full, win = _attn64(Q.double(), K.double(), V.double()), _attn64(Q.double(), K.double(), V.double(), w)
    O, C, R = Guarded((B, H, L, d), dev), Guarded((B, H, L, d), dev), Guarded((B, H, L, d), dev, torch.float32)
    for code, half, res in ((dfa.FULL, False, False), (dfa.WARS_REFRESH, False, True), (dfa.WARS_REUSE, False, False),
                            (dfa.ASC_REUSE, True, False), (dfa.WARS_ASC_REFRESH, True, True), (dfa.WARS_ASC_REUSE, True, False)):
        O.t.fill_(-7), C.t.fill_(-7)
        dfa.dfa_plan_step(code, Q, K, V, O.t, R.t, C.t, w)
        torch.cuda.synchronize()
        one = torch.full_like(O.t, -7)   # one destination (two under ASC), without a cache
        dfa.dfa_plan_step(code, Q, K, V, one, R.t, None, w)
        torch.cuda.synchronize()
        n = B // 2 if half else B
        name = dfa.CODE_NAMES[code]
        _check(f"{name} O", O.t[:n].float(), full[:n])
        if half:
            assert torch.equal(O.t[n:], O.t[:n]), name
        assert torch.equal(C.t, O.t), name   # every one of these codes writes the cache
        assert torch.equal(one, O.t), name
        if res:
            _check(f"{name} R", R.t[:n], (full - win)[:n])
    assert O.guards_intact() and C.guards_intact() and R.guards_intact()
