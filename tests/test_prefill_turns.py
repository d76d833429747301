"""Prefill attention where the groups of a work group meet once or twice a turn, and where tiles of very few turns follow each other: every output
against the closed form in fp64, and the same bits again and again."""
import pytest
import torch

import attention_plans
import dense_form as df
from paper_2507_19608_amd import binding as da

pytestmark = pytest.mark.gpu


# head_dim 64: split tiles that are all resident (one barrier a turn); whole and split ones (two); somewhat more than are resident, most of them split (one barrier, and tickets),
# fewer of them or none (two); more still (two); twice as many and more, some split, or all whole (the kernel with one).  head_dim 128: split; whole and split, with a pause
# between tiles and without; tiles of 2 to 5 turns one behind the other, whose next tile is told while the last one's readers may still be on their way
@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("B,Hq,Hkv,d,n,W,tiles,split,stream", [
    (1, 16, 4, 64, 2047, 100, 256, 256, True), (1, 8, 8, 64, 1100, 65, 72, 72, True), (1, 16, 2, 64, 3000, 150, 376, 376, True), (3, 8, 8, 64, 2300, 300, 432, 432, True),
    (12, 16, 2, 64, 434, 21, 480, 288, False), (6, 16, 4, 64, 808, 40, 528, 432, True), (12, 16, 4, 64, 451, 22, 528, 336, False),
    (12, 16, 4, 64, 700, 35, 528, 0, False), (16, 12, 6, 64, 433, 21, 672, 672, False), (16, 32, 8, 64, 705, 35, 1664, 384, True), (16, 32, 8, 64, 501, 25, 1024, 0, True),
    (1, 10, 5, 128, 1500, 75, 120, 120, False), (16, 12, 6, 128, 460, 23, 480, 192, False), (16, 32, 8, 128, 450, 22, 1024, 128, True),
    (40, 20, 5, 128, 230, 64, 800, 0, True), (64, 10, 5, 128, 201, 1, 640, 0, True), (48, 8, 4, 128, 330, 16, 576, 0, False)])
def test_every_output(window_mode, B, Hq, Hkv, d, n, W, tiles, split, stream):
    plan = attention_plans.launch(B, Hq, Hkv, d, n, W, window_mode == da.DA_WINDOW_SLIDING)
    assert plan[:2] == (tiles, split) and plan.stream == stream
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
