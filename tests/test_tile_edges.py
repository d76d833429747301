"""GPU parity of the prefill and scan kernels at the sizes where their tiling can go wrong: one row either side of a tile,
a block of keys, a segment, the smallest and largest of a dispatch's range.  Against the fp64 oracle; masks and nnz
bit-exact."""
import numpy as np
import pytest

from paper_2507_19608_amd import binding as da
from test_decode_parity import run_decode
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
    ("f32", 128, 1055, 52, 1, 8),      # many tiles, the last one ragged
    ("f32", 64, 513, 512, 4, 8),
    ("bf16", 32, 300, 15, 1, 2), ("bf16", 192, 97, 31, 1, 1), ("bf16", 96, 530, 26, 4, 8),
])
def test_binary32_products_kernel(window_mode, dtype, d, n, W, B, Hq):
    Q, K, V = _walks(301, B, Hq, 1, n, d, dtype)
    run_case(Q, K, V, 0.1 if dtype == "f32" else 0.2, W, dtype, da.DA_SCORE_GATHER, window_mode=window_mode)


@pytest.mark.parametrize("dtype,d,sizes", [
    ("bf16", 64, (1, 7, 8, 9, 1023, 1024, 1025, 1280)), ("bf16", 128, (5, 511, 512, 513, 640, 641)),
    ("bf16", 32, (2048, 2049)), ("bf16", 96, (682, 683, 897)), ("bf16", 256, (256, 257, 321)), ("f32", 32, (1024, 1025)),
    ("f32", 64, (512, 513, 769)), ("f32", 128, (255, 256, 257, 321)), ("f32", 160, (205, 300)), ("f32", 256, (128, 129, 193)),
    # several segments (of 128 rows): from more rows on than 64 KB hold in 8 channels
    ("bf16", 32, (4097, 4224)), ("bf16", 64, (4097, 4225)), ("bf16", 96, (4100,)), ("bf16", 128, (4223,)), ("bf16", 256, (4097,)),
    ("f32", 32, (2049, 2176)), ("f32", 64, (2049, 2177)), ("f32", 160, (2050,)), ("f32", 256, (2175,)),
])
def test_scan_segments(dtype, d, sizes):
    """One segment, few channels of every row in one launch, or several segments; ragged last ones, runs of a few rows or none:
    bursty and slow keys, so that some guesses of the time-parallel walk hold and some do not."""
    import torch
    import dense_form as df
    from paper_2507_19608_amd import workloads as wl
    from util import to_dev
    for n in sizes:
        rng = np.random.default_rng(n)
        K = rand_walk(n + d, 2, 2, n, d, dtype, 0.02)
        jump = rng.random((2, 2, n, 1)) < np.array([0.05, 0.002])[None, :, None, None]
        K = wl.round_to_dtype(np.where(jump, rng.standard_normal((2, 2, n, d)), K), dtype)
        Kd = to_dev(K, dtype)
        for theta in (0.0, 0.07, 5.0):
            bits, nnz, khat = da.delta_attn_delta_scan(Kd, theta, want_khat=True)
            ref_khat, ref_mask = df.reference_keys(Kd, theta)
            assert (df.unpack_bits(bits, d) == ref_mask).all(), (n, theta)
            assert (nnz == ref_mask.sum(dim=(2, 3))).all(), (n, theta)
            assert (khat.double() == ref_khat).all(), (n, theta)
        torch.cuda.synchronize()


@pytest.mark.parametrize("units,n", [(64, 1100), (1100, 1100), (65, 2100), (100, 2100), (300, 2049)])
def test_scan_of_many_short_rows(units, n):
    """One launch of 8 and of 16 channels a work group; 128-row segments, and the 256-row ones that only launches of many units take."""
    import dense_form as df
    from util import to_dev
    Kd = to_dev(rand_walk(17, units, 1, n, 64, "bf16", 0.03), "bf16")
    bits, nnz, khat = da.delta_attn_delta_scan(Kd, 0.1, want_khat=True)
    ref_khat, ref_mask = df.reference_keys(Kd, 0.1)
    assert (df.unpack_bits(bits, 64) == ref_mask).all() and (nnz == ref_mask.sum(dim=(2, 3))).all()
    assert (khat.double() == ref_khat).all()


@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("d,n,W,B,Hq,Hkv", [
    (64, 31, 7, 1, 4, 1), (128, 32, 64, 1, 8, 2), (64, 33, 1, 1, 1, 1), (128, 63, 20, 2, 4, 1), (64, 65, 32, 1, 8, 1),
    (128, 129, 33, 1, 2, 1), (64, 255, 100, 1, 2, 2), (128, 257, 64, 1, 1, 1), (64, 449, 63, 1, 4, 2), (128, 321, 320, 1, 12, 6),
    (64, 1000, 1000, 1, 4, 1),         # one window over everything
])
def test_matrix_core_tiles(window_mode, d, n, W, B, Hq, Hkv):
    """Blocks that lie left of some rows' windows and inside others', tiles that end in the middle, waves without rows,
    turns for which one of the two groups has no block.  (Up to 416 rows of 64 and 200 of 128 the short prompts' kernel; the tile-by-tile one on such
    sizes, by pieces: test_short_prompts.py.)"""
    Q, K, V = _walks(401, B, Hq, Hkv, n, d, "bf16")
    run_case(Q, K, V, 0.2, W, "bf16", da.DA_SCORE_GATHER, window_mode=window_mode)


@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("d,B,Hq,Hkv,n,W", [(64, 33, 32, 8, 300, 50), (128, 16, 20, 5, 900, 128), (64, 70, 8, 8, 520, 26),
                                            (128, 24, 16, 2, 777, 64)])
def test_whole_tiles_of_large_launches(window_mode, d, B, Hq, Hkv, n, W):
    """The 256-row tiles that only launches of many tiles take (300 rows of 64 are for the short prompts' kernel): every output against the closed form, masks too."""
    import torch
    import dense_form as df
    from util import to_dev
    Q, K, V = (to_dev(x, "bf16") for x in _walks(501, B, Hq, Hkv, n, d, "bf16"))
    O, bits, nnz = da.delta_attn_prefill(Q, K, V, 0.2, W, window_mode=window_mode)
    khat, mask = df.reference_keys(K, 0.2)
    assert (df.unpack_bits(bits, d) == mask).all() and (nnz == mask.sum(dim=(2, 3))).all()
    assert torch.isfinite(O).all()
    assert df.prefill_worst_error(Q, K, V, khat, W, window_mode == da.DA_WINDOW_SLIDING, [O]) <= 2e-2


@pytest.mark.parametrize("d,B,Hq,Hkv,n,W", [(128, 1, 20, 5, 4030, 256), (64, 2, 16, 2, 3001, 100), (64, 5, 12, 6, 700, 64),
                                            (128, 3, 8, 8, 1100, 55)])
def test_launches_that_hand_tiles_out(d, B, Hq, Hkv, n, W):
    """Whole and split tiles in one launch, more tiles than work groups, ragged last ones; and the same rows as chunked
    prefill, whose second piece starts inside a tile of the first."""
    import torch
    import dense_form as df
    from util import to_dev
    Q, K, V = (to_dev(x, "bf16") for x in _walks(701, B, Hq, Hkv, n, d, "bf16"))
    khat, mask = df.reference_keys(K, 0.2)
    cache = da.Cache(B, Hq, Hkv, d, n, max(W, 64), 0.2, torch.bfloat16)
    cut = n // 3 + 5
    pieces = [da.delta_attn_prefill_append(cache, *(x[:, :, r].contiguous() for x in (Q, K, V)), 0.2, W)[0]
              for r in (slice(0, cut), slice(cut, n))]
    for O in (da.delta_attn_prefill(Q, K, V, 0.2, W)[0], torch.cat(pieces, 2)):
        assert torch.isfinite(O).all()
        assert df.prefill_worst_error(Q, K, V, khat, W, False, [O]) <= 2e-2
    cache.close()


@pytest.mark.parametrize("window_mode", [da.DA_WINDOW_BLOCK, da.DA_WINDOW_SLIDING])
@pytest.mark.parametrize("dtype,d,n,W", [("bf16", 64, 700, 50), ("bf16", 128, 1200, 100), ("bf16", 96, 300, 20), ("f32", 64, 300, 20)])
def test_score_modes_give_the_same_bits(window_mode, dtype, d, n, W):
    """One computation stands behind both: in one call, and in two pieces where a cache can take them."""
    import torch
    from util import TORCH_DTYPE, to_dev
    x = [to_dev(t, dtype) for t in _walks(801, 2, 4, 2, n, d, dtype)]
    runs = []
    for mode in (da.DA_SCORE_GATHER, da.DA_SCORE_REBASE):
        runs.append(list(da.delta_attn_prefill(*x, 0.2, W, score_mode=mode, window_mode=window_mode)))
        if dtype == "bf16" and d in (64, 128):
            cache = da.Cache(2, 4, 2, d, n, 128, 0.2, TORCH_DTYPE[dtype])
            for r in (slice(0, n // 3), slice(n // 3, n)):
                runs[-1] += da.delta_attn_prefill_append(cache, *(t[:, :, r].contiguous() for t in x), 0.2, W, score_mode=mode,
                                                         window_mode=window_mode)
            cache.close()
    assert all(torch.equal(a, b) for a, b in zip(*runs))


def test_unaligned_keys_take_the_kernel_that_allows_them():
    """K and V one element off 16-byte alignment: same results within rounding (bit for bit, see test_unaligned_inputs.py)."""
    import torch
    from util import to_dev
    Q, K, V = (to_dev(x, "bf16") for x in _walks(601, 1, 4, 1, 200, 64, "bf16"))
    off = [torch.cat((x.new_zeros(1), x.flatten()))[1:].view(x.shape) for x in (K, V)]
    assert off[0].data_ptr() % 16 == 2
    a, b = da.delta_attn_prefill(Q, K, V, 0.2, 16), da.delta_attn_prefill(Q, off[0], off[1], 0.2, 16)
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    assert (a[0].float() - b[0].float()).abs().max().item() <= 2e-2


@pytest.mark.parametrize("n,steps,d,Hq,theta,plan", [
    (1535, 3, 64, 8, 0.2, (0, 16)),              # 24, then 25 chunks over the 8 walkers of one work group
    (1535, 3, 64, 8, 0.2, (0, 32)),              # over 16 of two: every other walker has one more
    (1535, 3, 64, 1, 0.0, (0, 64)), (900, 2, 64, 32, 5.0, (0, 64)),   # all and none of the entries survive
    (700, 2, 128, 32, 0.2, (0, 32)),             # 11 chunks over 4 walkers (of two waves) each of two work groups
    (831, 3, 128, 4, 0.0, (0, 64)), (1300, 2, 128, 8, 0.15, (0, 512)), (257, 2, 128, 2, 0.2, (1, 0)),
])
def test_decode_steps_of_several_work_groups(n, steps, d, Hq, theta, plan):
    """The work groups of a unit meet in memory, the last one merges: uneven walkers, walkers without a chunk, full and
    empty runs; consecutive steps on one cache find the count of arrivals back at zero."""
    L = n + steps
    Q, K, V = rand_walk(91, 2, Hq, L, d), rand_walk(92, 2, 1, L, d), rand_walk(93, 2, 1, L, d, clip=3.5)
    run_decode(Q, K, V, n, steps, theta, 64, "bf16", plan=plan)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [15, 16, 17, 63, 64, 65, 129, 143])
def test_hand_off_of_ragged_chunks(d, n):
    Q, K, V = rand_walk(94, 1, 2, n + 66, d), rand_walk(95, 1, 1, n + 66, d), rand_walk(96, 1, 1, n + 66, d, clip=3.5)
    run_decode(Q, K, V, n, 66, 0.2, 64, "bf16", check_every=5)
