"""Scores that rise from block to block of keys by more than a softmax taken against an earlier maximum can hold: the running maximum is raised late, and
the probabilities of that block are taken again.  Against the fp64 oracle."""
import numpy as np
import pytest

from paper_2507_19608_amd import binding as da
from paper_2507_19608_amd import workloads as wl
from test_prefill_parity import run_case
from util import rand_walk

pytestmark = pytest.mark.gpu


# 2^60 is 41 in the exponent, the largest float 88: below, between, beyond, and down again; split tiles, whole ones, tile after tile
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
