"""Decode steps at head_dim 128 with work groups of 4, 2 and 1 walkers: the plans that unit counts between and beyond the compute
units get, against the oracle on few units (wave slots given) and against one work group per unit on many."""
import pytest
import torch

from paper_2507_19608_amd import binding as da
from test_decode_parity import run_decode
from util import rand_walk, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("merge", [-1, 0])
@pytest.mark.parametrize("slots", [2, 4, 6, 8, 12, 20, 40, 100])
@pytest.mark.parametrize("n,steps,Hq,theta", [(62, 4, 4, 0.2), (127, 3, 1, 0.0), (640, 3, 32, 0.2), (1151, 2, 8, 5.0)])
def test_plans_against_the_oracle(merge, slots, n, steps, Hq, theta):
    """1, 2, 3 and 10 .. 19 chunks over 1 .. 50 walkers of 2 units; an empty window chunk becomes a history chunk on the way."""
    L = n + steps
    Q, K, V = rand_walk(81, 2, Hq, L, 128), rand_walk(82, 2, 1, L, 128), rand_walk(83, 2, 1, L, 128, clip=3.5)
    run_decode(Q, K, V, n, steps, theta, 64, "bf16", plan=(merge, slots))


@pytest.mark.parametrize("B,Hq,Hkv,n", [(12, 32, 8, 700), (28, 20, 5, 700), (32, 20, 5, 300), (24, 16, 8, 1200), (48, 8, 8, 450),
                                        (64, 16, 8, 200), (5, 20, 5, 3000)])
def test_plans_of_many_units_agree(B, Hq, Hkv, n):
    """The step's own choice, every work group the slots hold, and one work group per unit: the sums of a row are cut in
    different places, each rounded in binary32, its weights once to bf16 (2^-9) and the result to bf16 (2^-8 below 4)."""
    steps, d, theta = 3, 128, 0.2
    x = [to_dev(rand_walk(s, B, H, n + steps, d, clip=c), "bf16") for s, H, c in ((5, Hq, None), (6, Hkv, None), (7, Hkv, 3.5))]
    caches = [da.Cache(B, Hq, Hkv, d, n + steps, 64, theta, torch.bfloat16) for _ in range(3)]
    for cache, merge in zip(caches, (-1, 0, 1)):
        cache.set_launch_plan(merge, 0)
        da.delta_attn_prefill(*(t[:, :, :n].contiguous() for t in x), theta, 64, cache=cache)
    for i in range(n, n + steps):
        row = [t[:, :, i].contiguous() for t in x]
        (o, m), *others = [da.delta_attn_decode(cache, *row) for cache in caches]
        assert torch.isfinite(o).all()
        for o2, m2 in others:
            assert torch.equal(m, m2)
            assert (o.float() - o2.float()).abs().max().item() <= 4 * (2 ** -8 + 2 ** -9) / 2 + 2 ** -8
    for cache in caches:
        cache.close()


@pytest.mark.parametrize("B,Hq,Hkv,n", [(1, 8, 8, 255), (1, 32, 8, 256), (3, 8, 2, 511), (2, 32, 8, 575), (2, 4, 1, 4090), (2, 4, 1, 4095), (16, 5, 5, 640),
                                        (28, 8, 8, 1470), (28, 8, 8, 1534), (33, 8, 8, 200), (37, 20, 5, 500), (40, 16, 8, 700)])
def test_plans_of_four_walkers_agree(B, Hq, Hkv, n):
    """The same at head_dim 64, where work groups of 4 walkers take over: 4 and 5 chunks, 8 and 9, 64 and 65 (16 and 17 work groups
    a unit), nearly as many units as compute units, and more units than those."""
    steps, d, theta = 3, 64, 0.2
    x = [to_dev(rand_walk(s, B, H, n + steps, d, clip=c), "bf16") for s, H, c in ((5, Hq, None), (6, Hkv, None), (7, Hkv, 3.5))]
    caches = [da.Cache(B, Hq, Hkv, d, n + steps, 64, theta, torch.bfloat16) for _ in range(3)]
    for cache, merge in zip(caches, (-1, 0, 1)):
        cache.set_launch_plan(merge, 0)
        da.delta_attn_prefill(*(t[:, :, :n].contiguous() for t in x), theta, 64, cache=cache)
    for i in range(n, n + steps):
        row = [t[:, :, i].contiguous() for t in x]
        (o, m), *others = [da.delta_attn_decode(cache, *row) for cache in caches]
        assert torch.isfinite(o).all()
        for o2, m2 in others:
            assert torch.equal(m, m2)
            assert (o.float() - o2.float()).abs().max().item() <= 4 * (2 ** -8 + 2 ** -9) / 2 + 2 ** -8
    for cache in caches:
        cache.close()


@pytest.mark.parametrize("slots", [8, 64, 256])
@pytest.mark.parametrize("n,steps,Hq,theta", [(62, 4, 4, 0.2), (255, 3, 1, 0.0), (640, 3, 32, 0.2), (1151, 2, 8, 5.0)])
def test_plans_of_four_walkers_against_the_oracle(slots, n, steps, Hq, theta):
    """1 .. 19 chunks of 2 units; chunks that are window and history, and the newest row's, on the way."""
    L = n + steps
    Q, K, V = rand_walk(81, 2, Hq, L, 64), rand_walk(82, 2, 1, L, 64), rand_walk(83, 2, 1, L, 64, clip=3.5)
    run_decode(Q, K, V, n, steps, theta, 100, "bf16", plan=(-1, slots))


@pytest.mark.parametrize("d,Hq", [(64, 6), (64, 16), (128, 2), (128, 6), (128, 16)])
@pytest.mark.parametrize("parts", [2, 4, 5, 8, 9, 16, 17, 32])
def test_parts_of_a_unit_agree(d, Hq, parts):
    """Work groups of a unit, as many as a batch of the last one's reads takes, one more, and the most there are: each has one
    turn of its walkers, the last one a chunk of few rows."""
    Hkv, steps, theta, walkers = 2, 2, 0.2, 512 // d
    n = 64 * (walkers * (parts - 1) + 1) + 5
    x = [to_dev(rand_walk(s, 1, H, n + steps, d, clip=c), "bf16") for s, H, c in ((5, Hq, None), (6, Hkv, None), (7, Hkv, 3.5))]
    caches = [da.Cache(1, Hq, Hkv, d, n + steps, 64, theta, torch.bfloat16) for _ in range(2)]
    for cache, merge in zip(caches, (0, 1)):
        cache.set_launch_plan(merge, 8 * Hkv * parts)
        da.delta_attn_prefill(*(t[:, :, :n].contiguous() for t in x), theta, 64, cache=cache)
    for i in range(n, n + steps):
        row = [t[:, :, i].contiguous() for t in x]
        (o, m), (o1, m1) = [da.delta_attn_decode(cache, *row) for cache in caches]
        assert torch.isfinite(o).all() and torch.equal(m, m1)
        assert (o.float() - o1.float()).abs().max().item() <= 4 * (2 ** -8 + 2 ** -9) / 2 + 2 ** -8
    for cache in caches:
        cache.close()
