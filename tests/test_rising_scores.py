"""Scores that rise from block to block of keys by more than a softmax taken against an earlier maximum can hold: the running maximum is raised late, and
the probabilities of that block are taken again.  Against the fp64 oracle."""
import numpy as np
import pytest

from paper_2507_19608_amd import binding as da
from paper_2507_19608_amd import workloads as wl
from test_prefill_parity import run_case
from util import rand_walk

pytestmark = pytest.mark.gpu


# a maximum is held up to 2^8 too low, 5.5 in the exponent, and the largest float is 88: below, between, beyond, and down again; split tiles, whole ones, tile after tile
@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("d,B,Hq,Hkv,n", [(128, 1, 4, 1, 500), (64, 1, 4, 1, 500), (64, 64, 16, 4, 450), (128, 30, 16, 4, 330), (128, 20, 20, 5, 260)])
def test_rising_scores(window_mode, d, B, Hq, Hkv, n):
    rng = np.random.default_rng(n + d)
    Q = np.abs(rand_walk(1, B, Hq, n, d)) * 0 + 1.0 + 0.1 * rng.standard_normal((B, Hq, n, d))
    V = rand_walk(3, B, Hkv, n, d, clip=3.5)
    level = np.array([0.0, 35.0, 70.0, 150.0, 148.0, 320.0, 100.0, 330.0])[np.arange(n) // 64 % 8]     # of a block's scores
    K = (level / np.sqrt(d))[None, None, :, None] + 0.05 * rng.standard_normal((B, Hkv, n, d))
    Q, K = (wl.round_to_dtype(x, "bf16") for x in (Q, K))
    run_case(Q, K, V, 0.03, 40, "bf16", da.DA_SCORE_GATHER, window_mode=window_mode, q_heads=[0, Hq - 1])


@pytest.mark.parametrize("d,B,Hq,Hkv,n", [(128, 1, 4, 1, 500), (128, 30, 16, 4, 330), (128, 1, 4, 1, 2000), (64, 1, 4, 1, 500)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_not_a_number_stays_in_the_rows_that_see_it(value, d, B, Hq, Hkv, n):
    """A key with such an entry, in the middle of the prompt: rows before it stay finite and, within the rounding of the outputs, what they are without it;
    rows from it on, whose window it lies in, are NaN in every channel (it is in the reference keys of later rows too)."""
    import torch
    Q, K, V = (torch.from_numpy(np.ascontiguousarray(rand_walk(s, B, H, n, d, "bf16", clip=3.5))).to(torch.bfloat16).cuda() for s, H in ((17, Hq), (18, Hkv), (19, Hkv)))
    at, W = n // 2 + 3, 40
    Q[..., 3] = Q[..., 3].abs() + 0.25                           # positive: an infinite key scores infinity in every row
    clean, _, _ = da.delta_attn_prefill(Q, K, V, 0.2, W)
    K2 = K.clone()
    K2[:, :, at, 3] = value
    O, _, _ = da.delta_attn_prefill(Q, K2, V, 0.2, W)
    assert torch.isfinite(O[:, :, :at].float()).all()
    assert (O[:, :, :at].float() - clean[:, :, :at].float()).abs().max().item() <= 2e-2
    end = min(n, (at // W + 1) * W)                              # of the window the key lies in
    assert torch.isnan(O[:, :, at:end]).all()


@pytest.mark.parametrize("B,Hq,Hkv,n", [(1, 4, 1, 300), (30, 16, 4, 330), (64, 20, 5, 260)])
@pytest.mark.parametrize("sign", [1, -1])
def test_huge_scores_stay_in_their_row(sign, B, Hq, Hkv, n):
    """Queries whose scores are beyond 2^31, where a probability against the rounded maximum can be infinite: the rows 16 further on and 16 before, whose sums are
    taken in the same column of a matrix product, are within the rounding of the outputs what they are without them.  (head_dim 128: split tiles, whole ones,
    tile after tile.)"""
    import torch
    Q, K, V = (torch.from_numpy(np.ascontiguousarray(rand_walk(s, B, H, n, 128, "bf16", clip=3.5))).to(torch.bfloat16).cuda() for s, H in ((27, Hq), (28, Hkv), (29, Hkv)))
    K[..., 3] = sign * (K[..., 3].abs() + 0.25)
    clean, _, _ = da.delta_attn_prefill(Q, K, V, 0.2, 40)
    huge = torch.arange(n, device="cuda") % 64 < 16              # rows 0 .. 15 and, in other heads, 16 .. 31 of every 64
    hit = torch.stack([huge.roll(16 * (h % 2)) for h in range(Hq)])
    Q2 = Q.clone()
    Q2[..., 3] = torch.where(hit[None], torch.full_like(Q[..., 3], 3e11), Q[..., 3])
    O, _, _ = da.delta_attn_prefill(Q2, K, V, 0.2, 40)
    assert (O.float() - clean.float())[:, ~hit].abs().max().item() <= 2e-2
