"""Launches of the matrix-core prefill whose tiles follow each other, without a pause (head_dim 128) or with one, and cuts into whole and split tiles: every
output element against the closed form, masks bit-exact; rows that hold NaN."""
import pytest

from paper_2507_19608_amd import binding as da
from util import rand_walk, to_dev

pytestmark = pytest.mark.gpu


def _check(B, Hq, Hkv, d, n, W, mode, pieces=None):
    """One call, or pieces of these sizes into an empty cache, which always take the tile-by-tile kernel."""
    import dense_form as df
    import torch
    Q, K, V = (to_dev(rand_walk(s, B, H, n, d, "bf16", clip=3.5), "bf16") for s, H in ((7, Hq), (8, Hkv), (9, Hkv)))
    if pieces is None:
        O, bits, nnz = da.delta_attn_prefill(Q, K, V, 0.2, W, window_mode=mode)
    else:
        cache = da.Cache(B, Hq, Hkv, d, n, max(W, 64), 0.2, torch.bfloat16)
        parts = [[t.contiguous() for t in part] for part in zip(*(t.split(pieces, dim=2) for t in (Q, K, V)))]
        done = [da.delta_attn_prefill_append(cache, *part, 0.2, W, window_mode=mode) for part in parts]
        O, bits, nnz = torch.cat([x[0] for x in done], 2), torch.cat([x[1] for x in done], 2), sum(x[2] for x in done)
        cache.close()
    khat, mask = df.reference_keys(K, 0.2)
    assert (df.unpack_bits(bits, d) == mask).all() and (nnz == mask.sum(dim=(2, 3))).all()
    assert df.prefill_worst_error(Q, K, V, khat, W, mode == da.DA_WINDOW_SLIDING, [O]) <= 2e-2


# whole tiles that outnumber the work groups by far (128: no pause, 64: pauses between tiles), of five turns and more and, at their prompts' beginning, fewer; ragged
# ones, waves and whole row tiles' ends past the last row, several head chunks per unit.  (Up to 200 rows of 128 and 416 of 64 a prompt in one call takes the
# short prompts' kernel: here many of them at once; as pieces, which do not, below.)
@pytest.mark.parametrize("mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("B,Hq,Hkv,d,n,W", [
    (128, 20, 5, 128, 100, 64), (128, 20, 5, 128, 65, 10), (64, 20, 5, 128, 200, 128), (48, 20, 5, 128, 333, 16),
    (100, 8, 8, 128, 257, 64), (24, 16, 2, 128, 1030, 512),
    (100, 32, 8, 64, 128, 64), (100, 32, 8, 64, 97, 9), (50, 32, 8, 64, 300, 256), (70, 12, 6, 64, 1030, 51),
])
def test_tile_after_tile(B, Hq, Hkv, d, n, W, mode):
    _check(B, Hq, Hkv, d, n, W, mode)


# the same by pieces, of tiles of one turn (window a multiple of 64), two, three and four, which a work group also begins with; with the hand-off to the cache in a launch
# of its own and (32 query heads a KV head) in the attention's; a second and a third piece
@pytest.mark.parametrize("mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("B,Hq,Hkv,d,pieces,W", [
    (128, 20, 5, 128, (100,), 64), (128, 20, 5, 128, (65,), 10), (64, 20, 5, 128, (200,), 128), (40, 32, 1, 128, (100,), 64), (40, 32, 1, 128, (70, 30, 45), 16),
    (100, 32, 8, 64, (128,), 64), (100, 32, 8, 64, (97,), 9), (50, 32, 8, 64, (300,), 256), (100, 32, 8, 64, (40, 57), 9), (80, 32, 1, 64, (100, 64), 64),
    (14, 20, 5, 128, (200,), 10), (14, 12, 6, 64, (300,), 15),
])
def test_short_pieces_tile_after_tile(B, Hq, Hkv, d, pieces, W, mode):
    _check(B, Hq, Hkv, d, sum(pieces), W, mode, list(pieces))


# long tiles, few more than there are work groups; units that do not deal out evenly; cuts that leave some rows whole.  (14 prompts of 200
# and 300 rows are the short prompts' kernel's in one call; as pieces above)
@pytest.mark.parametrize("mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("B,Hq,Hkv,d,n,W", [
    (1, 20, 5, 128, 3500, 175), (3, 12, 3, 128, 2500, 100), (1, 32, 8, 64, 4650, 64), (7, 20, 5, 128, 598, 256), (4, 8, 8, 64, 1700, 85),
    (14, 20, 5, 128, 200, 10), (6, 20, 5, 128, 1000, 50), (14, 12, 6, 64, 300, 15), (2, 12, 6, 64, 2400, 120), (10, 24, 2, 128, 500, 25),
])
def test_cuts_and_long_tiles(B, Hq, Hkv, d, n, W, mode):
    _check(B, Hq, Hkv, d, n, W, mode)


@pytest.mark.parametrize("B,Hq,Hkv,d,n", [(1, 4, 1, 64, 300), (2, 8, 2, 128, 500), (64, 20, 5, 128, 260), (2, 8, 2, 64, 600)])
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
