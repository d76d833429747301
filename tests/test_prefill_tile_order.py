"""Launches of the matrix-core prefill whose tiles follow each other, without a pause (head_dim 128) or with one, and cuts into whole and split tiles: every
output element against the closed form, masks bit-exact; rows that hold NaN."""
import pytest

from paper_2507_19608_amd import binding as da
from util import rand_walk, to_dev

pytestmark = pytest.mark.gpu


def _check(B, Hq, Hkv, d, n, W, mode):
    import dense_form as df
    Q, K, V = (to_dev(rand_walk(s, B, H, n, d, "bf16", clip=3.5), "bf16") for s, H in ((7, Hq), (8, Hkv), (9, Hkv)))
    O, bits, nnz = da.delta_attn_prefill(Q, K, V, 0.2, W, window_mode=mode)
    khat, mask = df.reference_keys(K, 0.2)
    assert (df.unpack_bits(bits, d) == mask).all() and (nnz == mask.sum(dim=(2, 3))).all()
    assert df.prefill_worst_error(Q, K, V, khat, W, mode == da.DA_WINDOW_SLIDING, [O]) <= 2e-2


# whole tiles that outnumber the work groups by far (128: no pause, 64: pauses between tiles): of one turn (the first row tile, window a multiple of 64), two, three, four,
# five and more; ragged ones, waves and whole row tiles' ends past the last row, several head chunks per unit
@pytest.mark.parametrize("mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("B,Hq,Hkv,d,n,W", [
    (128, 20, 5, 128, 100, 64), (128, 20, 5, 128, 65, 10), (64, 20, 5, 128, 200, 128), (48, 20, 5, 128, 333, 16),
    (100, 8, 8, 128, 257, 64), (24, 16, 2, 128, 1030, 512),
    (100, 32, 8, 64, 128, 64), (100, 32, 8, 64, 97, 9), (50, 32, 8, 64, 300, 256), (70, 12, 6, 64, 1030, 51),
])
def test_tile_after_tile(B, Hq, Hkv, d, n, W, mode):
    _check(B, Hq, Hkv, d, n, W, mode)


# long tiles, few more than there are work groups; units that do not deal out evenly; cuts that leave some rows whole
@pytest.mark.parametrize("mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("B,Hq,Hkv,d,n,W", [
    (1, 20, 5, 128, 3500, 175), (3, 12, 3, 128, 2500, 100), (1, 32, 8, 64, 4650, 64), (7, 20, 5, 128, 598, 256), (4, 8, 8, 64, 1700, 85),
    (14, 20, 5, 128, 200, 10), (6, 20, 5, 128, 1000, 50), (14, 12, 6, 64, 300, 15), (2, 12, 6, 64, 2400, 120), (10, 24, 2, 128, 500, 25),
])
def test_cuts_and_long_tiles(B, Hq, Hkv, d, n, W, mode):
    _check(B, Hq, Hkv, d, n, W, mode)


@pytest.mark.parametrize("B,Hq,Hkv,d,n", [(1, 4, 1, 64, 300), (2, 8, 2, 128, 500), (64, 20, 5, 128, 260)])
def test_nan_stays_in_its_row(B, Hq, Hkv, d, n):
    """A NaN in a query row makes that row NaN and no other.  (The rows of a wave raise their running maxima together, so that
    others may round differently: a step of bf16 below 4 either way.)"""
    import torch
    Q, K, V = (to_dev(rand_walk(s, B, H, n, d, "bf16", clip=3.5), "bf16") for s, H in ((17, Hq), (18, Hkv), (19, Hkv)))
    clean, _, _ = da.delta_attn_prefill(Q, K, V, 0.2, 32)
    Q2 = Q.clone()
    hit = torch.zeros(B, Hq, n, dtype=torch.bool, device=Q.device)
    for i in (0, 1, 63, 64, n // 2, n - 1):
        hit[:, i % Hq, i] = True
    Q2[..., 3][hit] = float("nan")
    O, _, _ = da.delta_attn_prefill(Q2, K, V, 0.2, 32)
    assert torch.isnan(O[hit]).all()
    assert (O[~hit].float() - clean[~hit].float()).abs().max().item() <= 2e-2
