"""The delta scan that holds all rows of a few channels in one work group, and its counts, which the launch after it adds up: masks, reference keys and counts
against the row-by-row recurrence, exactly, on both sides of every line of the rule that chooses it."""
import pytest
import torch

import dense_form as df
import scan_plans
from paper_2507_19608_amd import binding as da
from test_scan_settle import _keys
from util import TORCH_DTYPE

pytestmark = pytest.mark.gpu


# 8 channels a work group up to 512 work groups, 16 above, 32 above that and up to 512 rows; 64 KB of rows; 256 or 512 threads
@pytest.mark.parametrize("dtype,units,n,d", [
    ("bf16", 1, 63, 64), ("bf16", 1, 64, 64), ("bf16", 9, 65, 128), ("bf16", 1, 257, 32), ("bf16", 3, 600, 96), ("bf16", 8, 2048, 64),
    ("bf16", 1, 2049, 64), ("bf16", 2, 4096, 128), ("bf16", 65, 2049, 64), ("bf16", 1, 4097, 64),
    ("bf16", 65, 64, 64), ("bf16", 65, 513, 64), ("bf16", 33, 1030, 128), ("bf16", 65, 2048, 64), ("bf16", 129, 513, 64),
    ("bf16", 192, 513, 64), ("bf16", 129, 65, 64), ("bf16", 65, 512, 128), ("bf16", 129, 200, 96),
    ("f32", 1, 64, 64), ("f32", 5, 333, 32), ("f32", 1, 2048, 160), ("f32", 1, 2049, 64), ("f32", 65, 1024, 64), ("f32", 65, 1025, 64),
    ("f32", 17, 130, 256), ("f32", 129, 512, 64), ("f32", 129, 70, 64),
])
def test_masks_and_counts(dtype, units, n, d):
    W = max(1, n // 20)
    for kind, theta in (("quiet", 0.3), ("mixed", 0.3), ("drift", 0.3), ("mixed", 0.0)):
        K = _keys(kind, n + d, units, n, d, dtype)
        if kind == "mixed":                                      # what never compares greater, on either side of it, and both zeros
            K[:, :, n // 2, 0], K[:, :, n // 3, 1], K[:, :, n // 4, 2] = float("inf"), float("-inf"), -0.0
        Q = K.expand(units, 1, n, d).contiguous()
        _, bits, nnz = da.delta_attn_prefill(Q, K, K.contiguous(), theta, W)
        ref_khat, ref_mask = df.reference_keys(K, theta)
        assert (df.unpack_bits(bits, d) == ref_mask).all(), (kind, theta)
        assert (nnz == ref_mask.sum(dim=(2, 3))).all(), (kind, theta)
        bits, nnz, khat = da.delta_attn_delta_scan(K, theta, want_khat=True)
        assert (khat.double() == ref_khat).all() and (df.unpack_bits(bits, d) == ref_mask).all(), (kind, theta)
        assert (nnz == ref_mask.sum(dim=(2, 3))).all(), (kind, theta)


@pytest.mark.parametrize("d,cuts", [(64, (0, 64, 128, 193)), (128, (0, 70, 1200, 3300)), (64, (0, 4096, 4160, 8257))])
@pytest.mark.parametrize("kind", ["quiet", "mixed"])
def test_pieces(kind, d, cuts):
    """Pieces that continue from the cache's reference key, and their counts, of several units."""
    n, units = cuts[-1], 3
    K = _keys(kind, n + d, units, n, d, "bf16")
    cache = da.Cache(units, 1, 1, d, n, 64, 0.3, torch.bfloat16)
    bits, counts = zip(*(da.delta_attn_prefill_append(cache, *[K[:, :, a:b].contiguous()] * 3, 0.3, 32)[1:]
                         for a, b in zip(cuts, cuts[1:])))
    _, mask = df.reference_keys(K, 0.3)
    assert (df.unpack_bits(torch.cat(bits, 2), d) == mask).all()
    for (a, b), c in zip(zip(cuts, cuts[1:]), counts):
        assert (c == mask[:, :, a:b].sum(dim=(2, 3))).all()
    assert (cache.nnz() == mask.sum(dim=(2, 3))).all()
    cache.close()


@pytest.mark.parametrize("units,n,d", [(48, 6144, 64), (47, 6144, 64), (24, 6143, 128), (40, 6560, 96)])
def test_segments_of_384_rows(units, n, d):
    """The longest segments, at the line where they begin, with whole ones and a remainder at the end."""
    for kind in ("quiet", "mixed", "drift"):
        K = _keys(kind, n + d, units, n, d, "bf16")
        bits, nnz, khat = da.delta_attn_delta_scan(K, 0.3, want_khat=True)
        ref_khat, ref_mask = df.reference_keys(K, 0.3)
        assert (khat.double() == ref_khat).all() and (df.unpack_bits(bits, d) == ref_mask).all(), kind
        assert (nnz == ref_mask.sum(dim=(2, 3))).all(), kind


# (of the rules, more than 64 runs are 86 or more: 2049 rows of 8 channels)
@pytest.mark.parametrize("dtype,units,d,n,runs", [
    ("bf16", 3, 64, 65, 9), ("bf16", 3, 64, 512, 64), ("bf16", 3, 64, 1031, 43), ("bf16", 3, 64, 2043, 64), ("bf16", 3, 64, 2049, 86), ("bf16", 3, 64, 3067, 128),
    ("bf16", 3, 64, 3073, 97), ("bf16", 3, 64, 4096, 128), ("f32", 1, 32, 65, 9), ("f32", 1, 32, 2043, 64),
    ("bf16", 40, 128, 129, 17), ("bf16", 40, 128, 1019, 32), ("bf16", 40, 128, 1025, 43), ("bf16", 40, 128, 2043, 64),
])
def test_runs_in_order(dtype, units, d, n, runs):
    """Runs whose ends travel in order, 64 of them at a time: the fewest, as many as travel together, those and some more, and twice that; of 8 and of 32 rows; channels
    that never meet their guess, that meet it in most runs and that fire in every one; with and without a round in front."""
    plan = scan_plans.whole(dtype, units, n, d)
    assert plan.runs == runs and plan.rounds == (n > 2048 or units == 40)
    for kind, theta in (("quiet", 0.3), ("mixed", 0.3), ("drift", 0.3), ("drift", 0.02)):
        K = _keys(kind, n + d, units, n, d, dtype)
        ref_khat, ref_mask = df.reference_keys(K, theta)
        bits, nnz, khat = da.delta_attn_delta_scan(K, theta, want_khat=True)
        assert (khat.double() == ref_khat).all() and (df.unpack_bits(bits, d) == ref_mask).all(), (kind, theta)
        assert (nnz == ref_mask.sum(dim=(2, 3))).all(), (kind, theta)
        _, bits, nnz = da.delta_attn_prefill(K, K, K, theta, 32)       # (short prompts and small ones of fp32 scan in the attention's launch)
        assert (df.unpack_bits(bits, d) == ref_mask).all(), (kind, theta)
        assert (nnz == ref_mask.sum(dim=(2, 3))).all(), (kind, theta)
