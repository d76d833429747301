"""Device memory of a decode cache: what its layout has to hold, and no more."""
import pytest
import torch

from paper_2507_19608_amd import binding as da
from util import TORCH_DTYPE

pytestmark = pytest.mark.gpu

CHUNK = 64


def _needed(units, heads, d, L, Wd, es, runs):
    chunks = -(-L // CHUNK)
    per_unit = L * (d // 32) * 4 + Wd * d * es + chunks * CHUNK * d * es + d * es + 8      # masks, ring, V, reference key, nnz
    per_unit += chunks * 4                                                                 # counts
    if runs:
        # survivors and carried-in values, 512 bytes of column masks and 256 of starts per 64 channels; one checkpoint
        per_unit += chunks * ((CHUNK + 1) * d * es + d // 64 * 768) + d * es + 4
        parts = min(32, -(-chunks // (4 if d == 64 else 1)))   # of the smallest work groups
    else:
        per_unit += chunks * CHUNK * d * es + (L // CHUNK + 1) * d * es + 4                # survivors; a checkpoint per chunk
        parts = chunks
    return units * per_unit + units * heads * parts * (d + 4) * 4


@pytest.mark.parametrize("dtype,d,Wd,heads,runs", [
    ("bf16", 32, 128, 1, False), ("bf16", 96, 128, 2, False), ("bf16", 160, 128, 1, False), ("bf16", 224, 128, 1, False),
    ("f32", 64, 128, 1, False), ("f32", 128, 64, 4, False), ("bf16", 64, 16, 1, False), ("bf16", 128, 4, 1, False),
    ("bf16", 64, 128, 1, True), ("bf16", 64, 64, 4, True), ("bf16", 128, 256, 1, True), ("bf16", 128, 128, 4, True),
])
def test_cache_takes_what_its_layout_needs(dtype, d, Wd, heads, runs):
    units, L = 32, 1 << 16
    da.Cache(1, 1, 1, 32, 64, 64, 0.1, torch.bfloat16).close()   # (the first one loads the library's device code)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    cache = da.Cache(units, heads, 1, d, L, Wd, 0.1, TORCH_DTYPE[dtype])
    taken = before - torch.cuda.mem_get_info()[0]
    cache.close()
    need = _needed(units, heads, d, L, Wd, 2 if dtype == "bf16" else 4, runs)
    page = 2 << 20                               # allocations are whole pages, except that those below one (nnz, reference
    assert need - 4 * page <= taken <= need + 10 * page, (taken, need)   # keys, counts of arrivals) may share one already held


@pytest.mark.parametrize("plan", [(0, 1 << 20), (-1, 0), (0, 64)])
@pytest.mark.parametrize("d,n", [(64, 700), (128, 513)])
def test_partial_rows_fit_whatever_the_plan(plan, d, n):
    """A plan that asks for more work groups per unit than the cache has rows for gets as many as fit: same results."""
    from test_decode_parity import run_decode
    from util import rand_walk
    steps = 2
    Q, K, V = (rand_walk(s, 2, H, n + steps, d, clip=3.5 if s == 7 else None) for s, H in ((5, 4), (6, 1), (7, 1)))
    run_decode(Q, K, V, n, steps, 0.2, 64, "bf16", plan=plan)
