"""Tensors that do not start on 16 bytes (slices of larger ones): the same kernels, so bit for bit the same results."""
import pytest
import torch

from paper_2507_19608_amd import binding as da
from util import rand_walk, to_dev

pytestmark = pytest.mark.gpu


def _moved(x, by):
    """The same values `by` elements further into an allocation."""
    y = torch.empty(x.numel() + by, dtype=x.dtype, device="cuda")[by:].view(x.shape)
    y.copy_(x)
    assert y.data_ptr() % 16 == by * x.element_size() % 16 and y.is_contiguous()
    return y


@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("by", [(1, 0, 0), (0, 1, 0), (0, 0, 1), (0, 3, 5), (7, 7, 4), (0, 8, 8)])
@pytest.mark.parametrize("B,Hq,Hkv,n,d,W", [(1, 1, 1, 1, 64, 1), (1, 2, 1, 2, 64, 2), (2, 4, 2, 257, 64, 16), (1, 4, 1, 1500, 128, 100),
                                            (3, 2, 2, 129, 128, 32)])
def test_prefill_of_moved_tensors(window_mode, by, B, Hq, Hkv, n, d, W):
    x = [to_dev(rand_walk(s, B, H, n, d, "bf16"), "bf16") for s, H in ((1, Hq), (2, Hkv), (3, Hkv))]
    y = [_moved(t, b) for t, b in zip(x, by)]
    L = n + 3
    caches = [da.Cache(B, Hq, Hkv, d, L, 64, 0.2, torch.bfloat16) for _ in range(2)]
    a, b = (da.delta_attn_prefill(*t, 0.2, W, window_mode=window_mode, cache=c) for t, c in zip((x, y), caches))
    assert all(torch.equal(s, t) for s, t in zip(a, b))
    out = tuple(torch.empty_like(t) for t in a)
    assert all(torch.equal(s, t) for s, t in zip(a, da.delta_attn_prefill_noalloc(*y, 0.2, W, out, window_mode=window_mode)))
    for i in range(3):                           # what the two calls left in their caches
        step = [to_dev(rand_walk(40 + i + s, B, H, 1, d, "bf16"), "bf16")[:, :, 0].contiguous() for s, H in ((0, Hq), (9, Hkv), (18, Hkv))]
        a, b = (da.delta_attn_decode(c, *step) for c in caches)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    for c in caches:
        c.close()


@pytest.mark.parametrize("by", [1, 5])
def test_moved_tensors_into_a_cache_of_many_chunks(by):
    """The hand-off to the cache in a launch of its own."""
    B, Hq, Hkv, n, d = 24, 8, 8, 450, 64
    x = [to_dev(rand_walk(s, B, H, n, d, "bf16"), "bf16") for s, H in ((1, Hq), (2, Hkv), (3, Hkv))]
    step = [to_dev(rand_walk(40 + s, B, H, 1, d, "bf16"), "bf16")[:, :, 0].contiguous() for s, H in ((0, Hq), (9, Hkv), (18, Hkv))]
    found = []
    for y in (x, [_moved(t, by) for t in x]):
        cache = da.Cache(B, Hq, Hkv, d, n + 1, 64, 0.2, torch.bfloat16)
        found.append(da.delta_attn_prefill(*y, 0.2, 20, cache=cache) + da.delta_attn_decode(cache, *step) + (cache.nnz().clone(),))
        cache.close()
    assert all(torch.equal(s, t) for s, t in zip(*found))


# short prompts in one launch, items of one wave and of several; split tiles, whole ones that end before the next begins, tile after tile without a pause: queries and
# outputs off 16 bytes
@pytest.mark.parametrize("by", [1, 4])
@pytest.mark.parametrize("B,Hq,Hkv,n,d", [(1, 4, 2, 333, 64), (70, 12, 6, 130, 64), (2, 4, 1, 300, 128), (16, 20, 5, 200, 128), (128, 20, 5, 65, 128),
                                          (1, 4, 2, 450, 64), (70, 12, 6, 430, 64), (16, 20, 5, 260, 128), (48, 20, 5, 333, 128)])
def test_queries_and_outputs_moved(by, B, Hq, Hkv, n, d):
    x = [to_dev(rand_walk(s, B, H, n, d, "bf16"), "bf16") for s, H in ((1, Hq), (2, Hkv), (3, Hkv))]
    want = da.delta_attn_prefill(*x, 0.2, 16)
    room = torch.full((want[0].numel() + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = (room[by:by + want[0].numel()].view(want[0].shape), torch.empty_like(want[1]), torch.empty_like(want[2]))
    da.delta_attn_prefill(_moved(x[0], by), x[1], x[2], 0.2, 16, out=out)
    assert all(torch.equal(s, t) for s, t in zip(out, want))
    assert (room[:by] == 7).all() and (room[by + want[0].numel():] == 7).all()


@pytest.mark.parametrize("d", [64, 128])
def test_chunked_prefill_and_scan_of_moved_tensors(d):
    B, Hq, Hkv, n, cut = 1, 4, 2, 300, 130
    x = [to_dev(rand_walk(s, B, H, n, d, "bf16"), "bf16") for s, H in ((1, Hq), (2, Hkv), (3, Hkv))]
    results = []
    for by in (0, 3):
        cache = da.Cache(B, Hq, Hkv, d, n, 64, 0.2, torch.bfloat16)
        for r in (slice(0, cut), slice(cut, n)):
            results.append(da.delta_attn_prefill_append(cache, *(_moved(t[:, :, r].contiguous(), by) for t in x), 0.2, 50))
        results.append(da.delta_attn_delta_scan(_moved(x[1], by), 0.2, want_khat=True))
        cache.close()
    for a, b in zip(results[:3], results[3:]):
        assert all(torch.equal(s, t) for s, t in zip(a, b))


def test_moved_tensors_in_a_captured_call():
    x = [to_dev(rand_walk(s, 1, H, 700, 64, "bf16"), "bf16") for s, H in ((1, 4), (2, 2), (3, 2))]
    want = da.delta_attn_prefill(*x, 0.2, 32)
    y = [_moved(t, 1) for t in x]
    out = tuple(torch.empty_like(t) for t in want)
    da.delta_attn_prefill_noalloc(*y, 0.2, 32, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        da.delta_attn_prefill_noalloc(*y, 0.2, 32, out)
    for _ in range(3):
        for t in out:
            t.zero_()
        for t in y:
            t.copy_(t.clone())
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(s, t) for s, t in zip(out, want))
