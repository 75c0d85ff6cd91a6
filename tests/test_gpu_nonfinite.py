"""Non-finite keys: a query that attends a NaN or infinite score gives what
float64 attention gives (NaN wherever that is NaN, finite elsewhere), whichever
form of the attention kernels a launch takes and however its keys are dealt to
wavefronts; a key outside the band stays out of the window attention."""
import pytest
import torch

from paper_2406_08552_amd import dfa
from tests.test_gpu_keysplit import _attn64
from tests.test_gpu_parity import say

pytestmark = pytest.mark.gpu


def _same_nans(name, got, ref):
    a, b = torch.isnan(got.double()), torch.isnan(ref)
    assert torch.equal(a, b), f"{name}: {int((a & ~b).sum())} NaN too many, {int((b & ~a).sum())} lost"


def _tiles(*ts):
    return [k for t in ts for k in range(64 * t, 64 * t + 64)]


# (B, H, L, d, w, keys): lengths of 64 k + 1, so that the last key is alone in
# its tile; `keys` is all that one group of wavefronts sees
KEY_GROUPS = [
    (1, 4, 65, 72, 20, [64]),                               # refresh, two groups
    (1, 4, 65, 64, 20, [64]),
    (1, 2, 449, 72, 70, _tiles(3) + [-1]),                  # full and refresh: the last of four and of two groups
    (1, 2, 513, 64, 200, _tiles(0, 4) + [512]),             # the first group of four
    (1, 1, 577, 72, 90, _tiles(1, 3, 5, 7)),                # the second of two, and two of four
    (1, 17, 961, 72, 200, _tiles(*range(1, 15, 2))),        # 272 workgroups: two groups
    (1, 2, 1025, 72, 161, [1024]),                          # the last window's fourth group
    (1, 2, 1025, 64, 161, [1024]),
]


@pytest.mark.parametrize("B,H,L,d,w,keys", KEY_GROUPS)
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_key_groups_keep_nonfinite_scores(B, H, L, d, w, keys, value):
    _check_all(B, H, L, d, w, keys, value)


# One-pass refreshes (more than 256 workgroups of 64 queries, and two key
# groups): the first and last query have one key outside their band
@pytest.mark.parametrize("B,H,L,d,w,keys", [
    (2, 16, 577, 72, 575, [576]),
    (2, 16, 577, 64, 575, [0]),
    (2, 7, 1280, 64, 1278, [1279]),
    (2, 2, 257, 72, 255, [256]),
    (1, 4, 65, 64, 63, [64]),
    (1, 2, 200, 72, 40, list(range(110, 200))),     # all keys outside the bands of the first queries' wavefronts and more
])
def test_refresh_keeps_nan_outside_the_band(B, H, L, d, w, keys):
    _check_all(B, H, L, d, w, keys, float("nan"))


# the other forms: short sequences, narrow bands, two phases
@pytest.mark.parametrize("B,H,L,d,w,keys", [
    (1, 2, 16, 72, 2, [15]),
    (1, 2, 31, 64, 20, [0]),
    (1, 2, 100, 72, 5, [99]),
    (2, 16, 1409, 64, 300, [1408]),
    (4, 16, 1300, 72, 1298, [0]),
])
def test_other_forms_keep_nan(B, H, L, d, w, keys):
    _check_all(B, H, L, d, w, keys, float("nan"))


def _check_all(B, H, L, d, w, keys, value):
    dev = torch.device("cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(L + d)
    Q, K, V = (torch.randn((B, H, L, d), generator=g, device=dev).to(torch.bfloat16) for _ in range(3))
    K[:, :, keys, 5] = value       # an infinite key scores +inf or -inf by the sign of the query's dim
    say(f"non-finite keys B={B} H={H} L={L} d={d} w={w} n={len(keys)} value={value}")
    full, win = _attn64(Q.double(), K.double(), V.double()), _attn64(Q.double(), K.double(), V.double(), w)
    O, R = torch.empty_like(Q), torch.empty((B, H, L, d), device=dev)
    dfa.dfa_attn_full(Q, K, V, O)
    torch.cuda.synchronize()
    _same_nans("full", O, full)
    dfa.dfa_attn_window_plus_residual(Q, K, V, O, None, w)
    torch.cuda.synchronize()
    _same_nans("window", O, win)
    dfa.dfa_attn_full_and_residual(Q, K, V, O, R, w)
    torch.cuda.synchronize()
    _same_nans("refresh O", O, full)
    _same_nans("refresh R", R, full - win)
