"""Calls on a stream that does not wait for the null stream: what a cache's first use needs has to be there."""
import pytest
import torch

from paper_2507_19608_amd import binding as da
from util import rand_walk, to_dev

pytestmark = pytest.mark.gpu

B, HQ, HKV, D, W, THETA = 32, 2, 1, 128, 32, 0.2
LONG = 1 << 17                                   # rows of room: 1 GiB an array, whose clearing takes the GPU 0.2 ms


def _rows(n):
    return [to_dev(rand_walk(s, B, H, n, D, clip=c), "bf16") for s, H, c in ((61, HQ, None), (62, HKV, None), (63, HKV, 3.5))]


def _fill_and_step(x, n, max_seq, wait):
    cache = da.Cache(B, HQ, HKV, D, max_seq, 64, THETA, torch.bfloat16)
    if wait:
        torch.cuda.synchronize()
    got = list(da.delta_attn_prefill(*(t[:, :, :n].contiguous() for t in x), THETA, W, cache=cache))
    for i in range(n, x[0].shape[2]):
        got += da.delta_attn_decode(cache, *(t[:, :, i].contiguous() for t in x))
    torch.cuda.current_stream().synchronize()
    cache.close()
    return got


def test_new_cache():
    """Used at once on another stream, a new cache gives what a small one gives that was waited for."""
    x = _rows(133)
    want = _fill_and_step(x, 130, 133, True)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        got = _fill_and_step(x, 130, LONG, False)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


def _two_pieces(x, cut, max_seq, wait):
    cache = da.Cache(B, HQ, HKV, D, max_seq, 64, THETA, torch.bfloat16)
    n = x[0].shape[2]
    got = []
    for r in (slice(0, cut), slice(cut, n)):
        got += da.delta_attn_prefill_append(cache, *(t[:, :, r].contiguous() for t in x), THETA, W)
        if wait:
            torch.cuda.synchronize()
    torch.cuda.current_stream().synchronize()
    cache.close()
    return got


def test_first_piece_of_a_chunked_prefill():
    """The first piece allocates and clears the cache's plain arrays and writes its rows there; the second one reads them."""
    x = _rows(200)
    want = _two_pieces(x, 90, 200, True)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        got = _two_pieces(x, 90, LONG, False)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_mask_and_counts_of_a_cache():
    """Copied out on another stream and read there at once, a cache's mask rows and counts are those of the calls that filled it."""
    n = 130
    x = _rows(n)
    cache = da.Cache(B, HQ, HKV, D, LONG, 64, THETA, torch.bfloat16)
    with torch.cuda.stream(torch.cuda.Stream()):
        _, bits, nnz = da.delta_attn_prefill(*x, THETA, W, cache=cache)
        got = cache.mask_rows().clone(), cache.nnz().clone()
        torch.cuda.current_stream().synchronize()
    assert torch.equal(got[0], bits) and torch.equal(got[1], nnz)
    cache.close()
