"""A prompt's rows on their way into a cache: in the attention launch, beside its tiles, where there are few, in a launch of their own where there are
many.  The same sequences as a small batch and inside a larger one, which lie on either side of that line: same masks, counts and, cut the
same way, decode steps to the bit; the small batch's decode steps against the closed form are other tests' work."""
import pytest
import torch

from paper_2507_19608_amd import binding as da
from util import rand_walk, to_dev

pytestmark = pytest.mark.gpu


# (head_dim, heads, small batch, large batch, pieces): last chunks of one row, whole, nearly whole; pieces that begin and end inside a chunk, that
# complete none, one and several; more chunks than work groups stay resident
@pytest.mark.parametrize("d,Hq,Hkv,small,large,pieces", [
    (64, 32, 8, 1, 24, (449,)), (64, 32, 8, 1, 24, (512,)), (64, 8, 4, 10, 48, (511,)), (64, 16, 2, 5, 24, (2049,)),
    (128, 20, 5, 1, 14, (640,)), (128, 8, 8, 1, 12, (513,)), (128, 4, 1, 2, 14, (4031,)), (128, 20, 5, 2, 6, (1700,)),
    (64, 32, 8, 1, 24, (300, 5, 15, 320)), (64, 4, 4, 3, 24, (63, 1, 1000, 64)), (128, 20, 5, 1, 14, (130, 62, 448)), (128, 4, 2, 2, 24, (1, 63, 700, 3)),
])
def test_either_launch_leaves_the_same_cache(d, Hq, Hkv, small, large, pieces):
    theta, steps, n = 0.2, 2, sum(pieces)
    x = [to_dev(rand_walk(s, large, H, n + steps, d, clip=c), "bf16") for s, H, c in ((5, Hq, None), (6, Hkv, None), (7, Hkv, 3.5))]
    found = []
    for B in (small, large):
        cache = da.Cache(B, Hq, Hkv, d, n + steps, 128, theta, torch.bfloat16)
        cache.set_launch_plan(1, 0)
        part = lambda i, j: [t[:B, :, i:j].contiguous() for t in x]
        at, outs = 0, []
        for m in pieces:
            if len(pieces) == 1:
                _, mask, nnz = da.delta_attn_prefill(*part(0, n), theta, 100, cache=cache)
            else:
                _, mask, nnz = da.delta_attn_prefill_append(cache, *part(at, at + m), theta, 100)
            outs += [mask[:small], nnz[:small]]
            at += m
        outs += [cache.nnz()[:small], cache.mask_rows()[:small]]
        for i in range(n, n + steps):
            outs += [t[:small] for t in da.delta_attn_decode(cache, *(t[:, :, 0] for t in part(i, i + 1)))]
        found.append([t.clone() for t in outs])
        cache.close()
    for a, b in zip(*found):
        assert torch.isfinite(a.float()).all()
        assert torch.equal(a.reshape(-1), b.reshape(-1))
