"""Prefill attention where the groups of a work group meet once or twice a turn, and where tiles of very few turns follow each other: every output
against the closed form in fp64, and the same bits again and again."""
import pytest
import torch

import dense_form as df
from paper_2507_19608_amd import binding as da

pytestmark = pytest.mark.gpu


# head_dim 64: all tiles resident at once (split ones, one barrier a turn); somewhat more, whole and split (two barriers in split tiles); twice as many; all
# whole.  head_dim 128: split and whole, and tiles of 2 to 5 turns one behind the other, whose next tile is told while the last one's readers may still be on their way
@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("B,Hq,Hkv,d,n,W", [
    (1, 16, 4, 64, 2047, 100), (1, 8, 8, 64, 1100, 65), (1, 16, 2, 64, 3000, 150), (3, 8, 8, 64, 2300, 300), (12, 16, 4, 64, 700, 35), (1, 10, 5, 128, 1500, 75),
    (40, 20, 5, 128, 230, 64), (64, 10, 5, 128, 201, 1), (48, 8, 4, 128, 330, 16)])
def test_every_output(window_mode, B, Hq, Hkv, d, n, W):
    g = torch.Generator(device="cuda").manual_seed(n)
    Q, K, V = (torch.cumsum(0.2 * torch.randn(B, h, n, d, generator=g, device="cuda"), 2).remainder(4.0).sub(2.0).bfloat16() for h in (Hq, Hkv, Hkv))
    mask, nnz, khat = da.delta_attn_delta_scan(K, 0.3, want_khat=True)
    first = None
    for _ in range(4):
        out = da.delta_attn_prefill(Q, K, V, 0.3, W, window_mode=window_mode)
        if first is None:
            first = out
        assert all(torch.equal(a, b) for a, b in zip(out, first))
    assert torch.equal(first[1], mask) and torch.equal(first[2], nnz)
    some = slice(0, 3)                                           # (rows of a few prompts: the rest would take a minute)
    worst = df.prefill_worst_error(Q[some], K[some], V[some], khat[some].double(), W, window_mode == da.DA_WINDOW_SLIDING, [first[0][some]])
    assert worst <= 2e-2
