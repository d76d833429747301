"""Small fp32 prompts, whose work groups scan their keys themselves (head_dim 64 and 128, up to 32768 key elements, as many work groups as compute units), and
their neighbours outside that range: masks, counts and outputs against the oracle."""
import numpy as np
import pytest
import torch

from paper_2507_19608_amd import binding as da
from test_prefill_parity import run_case
from util import rand_walk, to_dev

pytestmark = pytest.mark.gpu


# one row; tiles of 16 rows and runs of 1 .. 32 rows with remainders; one row below, on and beyond 32768 elements; as many work groups as compute
# units and more; windows of one row, of all rows (nothing is scanned but for the mask), that straddle blocks of 32
@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("d,B,Hq,Hkv,n,W", [
    (64, 1, 1, 1, 1, 1), (64, 1, 2, 1, 15, 4), (64, 2, 4, 2, 17, 1), (64, 1, 1, 1, 65, 100), (64, 1, 8, 2, 177, 20), (64, 1, 1, 1, 511, 33), (64, 1, 1, 1, 512, 64),
    (64, 1, 1, 1, 513, 25), (64, 4, 4, 1, 240, 12), (64, 4, 4, 1, 241, 12), (128, 1, 1, 1, 2, 1), (128, 3, 2, 2, 47, 9), (128, 1, 4, 1, 255, 12), (128, 1, 1, 1, 256, 40),
    (128, 1, 1, 1, 257, 12)])
def test_small_fp32_prompts(window_mode, d, B, Hq, Hkv, n, W):
    Q, K, V = rand_walk(11, B, Hq, n, d), rand_walk(12, B, Hkv, n, d), rand_walk(13, B, Hkv, n, d)
    run_case(Q, K, V, 0.15, W, "f32", da.DA_SCORE_GATHER, window_mode=window_mode)


@pytest.mark.parametrize("d,n", [(64, n) for n in (7, 8, 9, 127, 128, 129, 383, 384, 385)] + [(128, n) for n in (8, 63, 64, 65, 191, 192, 193)])
def test_runs_of_whole_batches(d, n):
    """Runs of 8, 16, .. rows that end with the prompt, one row before and one behind: the same masks and counts as the scan's own entry point."""
    Kd = to_dev(rand_walk(n, 1, 1, n, d), "f32")
    mask, nnz, _ = da.delta_attn_delta_scan(Kd, 0.2)
    _, mask2, nnz2 = da.delta_attn_prefill(Kd, Kd, Kd, 0.2, 1)
    assert torch.equal(mask, mask2) and torch.equal(nnz, nnz2)


@pytest.mark.parametrize("kind", ["still", "drift", "jumps", "zeros", "nan"])
@pytest.mark.parametrize("d,n", [(64, 300), (128, 200)])
def test_the_same_mask_as_the_scan_alone(kind, d, n):
    """Keys whose runs settle late or never fire, signed zeros and NaN: bit for bit what the scan's own entry point says."""
    rng = np.random.default_rng(n)
    K = {"still": 0.01 * rng.standard_normal((1, 2, n, d)), "drift": 0.03 * np.arange(n)[None, None, :, None] + np.zeros((1, 2, n, d)),
         "jumps": rng.standard_normal((1, 2, n, d)) * (rng.random((1, 2, n, 1)) < 0.1), "zeros": np.where(rng.random((1, 2, n, d)) < 0.5, 0.0, -0.0),
         "nan": np.where(rng.random((1, 2, n, d)) < 0.01, np.nan, rng.standard_normal((1, 2, n, d)))}[kind]
    Kd, theta = to_dev(K, "f32"), 0.0 if kind == "zeros" else 0.1
    Q = torch.ones_like(Kd)
    mask, nnz, _ = da.delta_attn_delta_scan(Kd, theta)
    _, mask2, nnz2 = da.delta_attn_prefill(Q, Kd, Q, theta, 16)
    assert torch.equal(mask, mask2) and torch.equal(nnz, nnz2)
