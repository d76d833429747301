"""GPU parity of the prefill and scan kernels at the sizes where their tiling can go wrong: one row either side of a tile,
a block of keys, a segment, the smallest and largest of a dispatch's range.  Against the fp64 oracle; masks and nnz
bit-exact."""
import numpy as np
import pytest

from paper_2507_19608_amd import binding as da
from test_prefill_parity import run_case
from util import rand_walk

pytestmark = pytest.mark.gpu


def _walks(seed, B, Hq, Hkv, n, d, dtype):
    step = 0.05 if dtype == "f32" else 0.15
    return (rand_walk(seed, B, Hq, n, d, dtype), rand_walk(seed + 1, B, Hkv, n, d, dtype, step),
            rand_walk(seed + 2, B, Hkv, n, d, dtype, clip=3.5))


@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("dtype,d,n,W,B,Hq", [
    ("f32", 64, 15, 4, 1, 1), ("f32", 32, 17, 32, 1, 2), ("f32", 96, 33, 7, 2, 1), ("f32", 128, 255, 16, 1, 2),
    ("f32", 64, 257, 40, 1, 1), ("f32", 160, 70, 9, 1, 1), ("f32", 224, 65, 33, 1, 1), ("f32", 256, 289, 64, 1, 1),
    ("f32", 128, 1055, 52, 1, 8),      # 32-row tiles, ragged
    ("f32", 64, 513, 512, 4, 8),
    ("bf16", 32, 300, 15, 1, 2), ("bf16", 192, 97, 31, 1, 1), ("bf16", 96, 530, 26, 4, 8),
])
def test_binary32_products_kernel(window_mode, dtype, d, n, W, B, Hq):
    Q, K, V = _walks(301, B, Hq, 1, n, d, dtype)
    run_case(Q, K, V, 0.1 if dtype == "f32" else 0.2, W, dtype, da.DA_SCORE_GATHER, window_mode=window_mode)
