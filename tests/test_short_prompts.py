"""Prompts that are scanned and attended in one launch, at the edges of its rows, items and work groups, on both sides of its lines; and the tile-by-tile
kernel at the sizes where its tiling can go wrong, which short prompts reach in pieces only.  Against the fp64 oracle; masks and counts exact."""
import pytest
import torch

import dense_form as df
from oracle import delta_oracle as orc
from paper_2507_19608_amd import binding as da
from test_prefill_parity import run_case
from test_scan_settle import _keys
from util import check_output, rand_walk, to_dev, unpack_mask

pytestmark = pytest.mark.gpu


def _walks(seed, B, Hq, Hkv, n, d):
    return rand_walk(seed, B, Hq, n, d), rand_walk(seed + 1, B, Hkv, n, d), rand_walk(seed + 2, B, Hkv, n, d, clip=3.5)


# rows: multiples of 8, 32 and 64 and one more or less, the longest prompt and one more; items of 8, 16 and 32 rows, heads in one or several
# groups; 4, 2 and 1 waves an item; several items a wave (many prompts), more work groups than compute units
@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("d,B,Hq,Hkv,n,W", [
    (64, 1, 4, 1, 1, 1), (64, 2, 2, 1, 7, 3), (128, 1, 4, 1, 9, 4), (64, 1, 1, 1, 32, 5), (128, 1, 1, 1, 33, 40), (64, 1, 8, 1, 65, 64), (128, 3, 6, 2, 64, 16),
    (64, 1, 32, 8, 127, 6), (64, 1, 3, 1, 193, 33), (128, 1, 16, 2, 199, 10), (128, 2, 4, 2, 200, 100), (128, 1, 4, 1, 201, 10),
    (64, 1, 4, 1, 257, 300), (64, 2, 12, 2, 415, 21), (64, 1, 4, 2, 416, 31), (64, 1, 4, 2, 417, 31),
    (64, 40, 8, 2, 150, 8), (128, 30, 4, 2, 97, 5), (64, 150, 2, 2, 40, 7), (128, 130, 4, 2, 35, 12),
])
def test_against_the_oracle(window_mode, d, B, Hq, Hkv, n, W):
    run_case(*_walks(n + d, B, Hq, Hkv, n, d), 0.2, W, "bf16", da.DA_SCORE_GATHER, window_mode=window_mode)


@pytest.mark.parametrize("kind,theta", [("quiet", 0.3), ("mixed", 0.3), ("drift", 0.3), ("mixed", 0.0)])
@pytest.mark.parametrize("units,n,d", [(1, 8, 64), (3, 63, 128), (2, 130, 64), (5, 200, 128), (300, 72, 64), (9, 416, 64), (257, 33, 128)])
def test_masks_and_counts(kind, theta, units, n, d):
    """Streams whose runs' guesses hold, mostly do not, or never do; entries that never compare greater, and both zeros."""
    K = _keys(kind, n + d, units, n, d, "bf16")
    if kind == "mixed":
        K[:, :, n // 2, 0], K[:, :, n // 3, 1], K[:, :, n // 4, 2] = float("inf"), float("-inf"), -0.0
    _, bits, nnz = da.delta_attn_prefill(K, K, K, theta, max(1, n // 20))
    _, mask = df.reference_keys(K, theta)
    assert (df.unpack_bits(bits, d) == mask).all() and (nnz == mask.sum(dim=(2, 3))).all()


@pytest.mark.parametrize("kind", ["quiet", "mixed", "drift"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [2, 55, 56, 57, 73, 80, 88, 89, 121, 194, 200])
def test_runs_of_unequal_length(kind, d, n):
    """The scan's first run, longer by the rows that the later ones warm up on: prompts of about as many rows, later runs of 8 and of 16, a last one of
    a few rows or none."""
    K = _keys(kind, n + d, 3, n, d, "bf16")
    _, bits, nnz = da.delta_attn_prefill(K, K, K, 0.3, 8)
    _, mask = df.reference_keys(K, 0.3)
    assert (df.unpack_bits(bits, d) == mask).all()
    assert (nnz == mask.sum(dim=(2, 3))).all()


@pytest.mark.parametrize("d,B,n", [(64, 1, 416), (64, 50, 100), (128, 1, 200), (128, 60, 70)])
def test_prompt_into_a_cache(d, B, n):
    """The reference keys that the cache is filled from: decode steps on what one launch has left against a prompt that came in pieces."""
    Hq, Hkv, W, theta = 4, 2, 16, 0.2
    x = [to_dev(t, "bf16") for t in _walks(n, B, Hq, Hkv, n + 3, d)]
    caches = [da.Cache(B, Hq, Hkv, d, n + 3, 64, theta, torch.bfloat16) for _ in range(2)]
    whole, cut = [t[:, :, :n].contiguous() for t in x], n // 2 + 3
    O, bits, nnz = da.delta_attn_prefill(*whole, theta, W, cache=caches[0])
    assert all(torch.equal(a, b) for a, b in zip((O, bits, nnz), da.delta_attn_prefill(*whole, theta, W)))
    for r in (slice(0, cut), slice(cut, n)):
        da.delta_attn_prefill_append(caches[1], *(t[:, :, r].contiguous() for t in x), theta, W)
    assert torch.equal(caches[0].mask_rows(), caches[1].mask_rows()) and torch.equal(caches[0].nnz(), nnz)
    for t in range(n, n + 3):
        a, b = (da.delta_attn_decode(c, *(s[:, :, t].contiguous() for s in x)) for c in caches)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    for c in caches:
        c.close()


def test_replays_from_a_captured_graph():
    for d, B, n in ((64, 1, 333), (128, 16, 200)):
        x = [to_dev(t, "bf16") for t in _walks(9, B, 4, 1, n, d)]
        want = da.delta_attn_prefill(*x, 0.2, 16)
        out = tuple(torch.empty_like(t) for t in want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            da.delta_attn_prefill_noalloc(*x, 0.2, 16, out)
        for _ in range(3):
            for t in out:
                t.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(s, t) for s, t in zip(out, want))


@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("d,n,W,B,Hq,Hkv", [
    (64, 31, 7, 1, 4, 1), (128, 32, 64, 1, 8, 2), (64, 33, 1, 1, 1, 1), (128, 63, 20, 2, 4, 1), (64, 65, 32, 1, 8, 1), (128, 129, 33, 1, 2, 1),
    (64, 255, 63, 1, 2, 2), (128, 200, 10, 16, 20, 5), (64, 416, 64, 2, 4, 1),
])
def test_tile_by_tile_kernel_on_short_prompts(window_mode, d, n, W, B, Hq, Hkv):
    """A whole prompt as the first piece: blocks left of some rows' windows and inside others', tiles that end in the middle, waves without
    rows, turns for which one of the two groups has no block."""
    Q, K, V = _walks(401, B, Hq, Hkv, n, d)
    cache = da.Cache(B, Hq, Hkv, d, n, 64, 0.2, torch.bfloat16)
    O, bits, nnz = da.delta_attn_prefill_append(cache, *(to_dev(t, "bf16") for t in (Q, K, V)), 0.2, W, window_mode=window_mode)
    cache.close()
    ref = orc.prefill(Q, K, V, 0.2, W, window_mode=window_mode)
    assert (unpack_mask(bits, d) == ref["mask"]).all() and (nnz.cpu().numpy() == ref["nnz"]).all()
    check_output(O, ref["O"], "bf16")


@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("d,n,W,B,Hq,Hkv", [(64, 447, 7, 1, 4, 1), (64, 449, 63, 1, 4, 2), (64, 513, 33, 1, 1, 1), (64, 575, 100, 1, 2, 2), (128, 255, 64, 1, 4, 1),
                                            (128, 257, 20, 1, 1, 1), (128, 289, 33, 2, 8, 2), (128, 321, 320, 1, 12, 6)])
def test_tile_by_tile_kernel_beyond_short_prompts(window_mode, d, n, W, B, Hq, Hkv):
    run_case(*_walks(402, B, Hq, Hkv, n, d), 0.2, W, "bf16", da.DA_SCORE_GATHER, window_mode=window_mode)


# (prompt's rows, pieces, stages with a call): one launch; two; the hand-off in the attention's; short prompts and fp32 into a cache
@pytest.mark.parametrize("dtype,n,pieces,stages", [
    ("bf16", 333, 0, {"attn"}), ("bf16", 500, 0, {"scan", "attn"}), ("f32", 200, 0, {"attn"}), ("f32", 600, 0, {"scan", "attn"}),
    ("bf16", 333, 1, {"attn", "cache_fill"}), ("bf16", 500, 1, {"scan", "attn"}), ("f32", 200, 1, {"scan", "attn", "cache_fill"}), ("bf16", 500, 2, {"scan", "attn"}),
])
def test_stages_that_are_timed(dtype, n, pieces, stages):
    """What the header says of launches that do the work of several stages."""
    Hq, Hkv, d = 4, 2, 64
    x = [to_dev(t, dtype) for t in _walks(21, 1, Hq, Hkv, n, d)]
    cache = da.Cache(1, Hq, Hkv, d, n, 64, 0.2, x[0].dtype) if pieces else None
    torch.cuda.synchronize()
    da.delta_attn_stage_timing_enable(True)
    da.delta_attn_stage_timing_read()
    if pieces < 2:
        da.delta_attn_prefill(*x, 0.2, 16, cache=cache)
    else:
        for r in (slice(0, n // 2), slice(n // 2, n)):
            da.delta_attn_prefill_append(cache, *(t[:, :, r].contiguous() for t in x), 0.2, 16)
    torch.cuda.synchronize()
    read = da.delta_attn_stage_timing_read()
    da.delta_attn_stage_timing_enable(False)
    if cache:
        cache.close()
    assert {name for name, (_, calls) in read.items() if calls} == stages
