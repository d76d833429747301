"""The delta scan where segments (or the runs of the one-launch form) cannot settle from their neighbours at once: channels that stay
quiet over whole segments, chains that meet late or never.  Bit-exact against the row-by-row recurrence, and in time linear in the rows."""
import numpy as np
import pytest
import torch

from paper_2507_19608_amd import binding as da
from util import TORCH_DTYPE

pytestmark = pytest.mark.gpu


def _keys(kind, seed, units, n, d, dtype):
    """Channel by channel: quiet (never fires), rare (fires about once in 700 rows), drifting (fires every few rows at a phase
    that a wrong guess does not find soon), lively (5 % whole-vector jumps)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    noise = torch.randn(units, 1, n, d, generator=gen, device="cuda")
    quiet = 0.01 * noise
    rare = quiet + (torch.rand(units, 1, n, d, generator=gen, device="cuda") < 1 / 700).cumsum(2).fmod(5)
    drift = (torch.arange(n, device="cuda").view(1, 1, n, 1) * 0.013).fmod(3.7) + 0.002 * noise
    lively = torch.where(torch.rand(units, 1, n, 1, generator=gen, device="cuda") < 0.05, noise, 0.1 * noise)
    kinds = {"quiet": [quiet], "rare": [rare], "drift": [drift], "mixed": [quiet, lively, rare, drift, lively]}[kind]
    channel = torch.arange(d, device="cuda") % len(kinds)
    K = kinds[0]
    for i, x in enumerate(kinds):
        K = torch.where(channel == i, x, K)
    return K.to(TORCH_DTYPE[dtype]).contiguous()


@pytest.mark.parametrize("kind", ["quiet", "rare", "drift", "mixed"])
@pytest.mark.parametrize("dtype,units,n,d", [
    ("bf16", 1, 1025, 64), ("bf16", 2, 2049, 64), ("bf16", 1, 128 * 17 + 1, 128), ("bf16", 1, 128 * 33 - 1, 64),
    ("bf16", 1, 128 * 65 + 40, 128), ("bf16", 1, 3000, 96), ("bf16", 1, 5000, 32), ("bf16", 200, 1400, 64),
    ("f32", 1, 128 * 18, 64), ("f32", 1, 4100, 160), ("f32", 2, 128 * 40 + 3, 32),
    # (of those above, up to 64 KB of rows in 8 channels are one launch)  17 and 33 segments; 9 of 256 rows; half a group of channels
    ("f32", 1, 2049, 64), ("bf16", 20, 4097, 128), ("bf16", 100, 2100, 64), ("bf16", 1, 4100, 96),
])
def test_segments_that_settle_late(kind, dtype, units, n, d):
    import dense_form as df
    K = _keys(kind, n + d, units, n, d, dtype)
    bits, nnz, khat = da.delta_attn_delta_scan(K, 0.3, want_khat=True)
    ref_khat, ref_mask = df.reference_keys(K, 0.3)
    assert (khat.double() == ref_khat).all()
    assert (df.unpack_bits(bits, d) == ref_mask).all() and (nnz == ref_mask.sum(dim=(2, 3))).all()
    if kind == "quiet":
        assert (nnz == d).all()


@pytest.mark.parametrize("kind", ["quiet", "rare", "drift", "mixed"])
@pytest.mark.parametrize("dtype,units,n,d", [("bf16", 1, 128 * 64 + 1, 32), ("bf16", 1, 128 * 129 + 2, 64), ("f32", 1, 128 * 65, 32), ("bf16", 24, 6144 + 1, 128),
                                             ("bf16", 24, 384 * 16 + 129, 128), ("bf16", 64, 4100, 64), ("bf16", 65, 4100, 64)])
def test_segments_in_order(kind, dtype, units, n, d):
    """64 segments whose ends travel together and one more, twice that; a last segment of one or two rows, whole, and of one row more than the two
    blocks that are looked at first; the most units that settle in order, and one more."""
    import dense_form as df
    K = _keys(kind, n + 7, units, n, d, dtype)
    bits, nnz, khat = da.delta_attn_delta_scan(K, 0.3, want_khat=True)
    ref_khat, ref_mask = df.reference_keys(K, 0.3)
    assert (khat.double() == ref_khat).all() and (df.unpack_bits(bits, d) == ref_mask).all()
    assert (nnz == ref_mask.sum(dim=(2, 3))).all()


@pytest.mark.parametrize("kind", ["quiet", "rare", "mixed"])
@pytest.mark.parametrize("d,cuts", [(64, (0, 1100, 4000)), (128, (0, 40, 2700)), (64, (0, 3001, 3002, 5200)), (128, (0, 300, 4500))])
def test_pieces_that_continue_a_cache(kind, d, cuts):
    """The rows of a piece start from the reference key the cache carries: in one launch, and over several segments (the last case)."""
    import dense_form as df
    n = cuts[-1]
    K = _keys(kind, n + d, 1, n, d, "bf16")
    cache = da.Cache(1, 1, 1, d, n, 64, 0.3, torch.bfloat16)
    bits, counts = zip(*(da.delta_attn_prefill_append(cache, *[K[:, :, a:b].contiguous()] * 3, 0.3, 32)[1:]
                         for a, b in zip(cuts, cuts[1:])))
    _, mask = df.reference_keys(K, 0.3)
    assert (df.unpack_bits(torch.cat(bits, 2), d) == mask).all() and sum(counts).item() == mask.sum().item()
    cache.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 128)])
def test_time_of_quiet_channels_grows_with_the_rows(dtype, d):
    """Four times the rows where nothing fires take four times as long (a fixed part makes it less; the 1.6 is for noise).
    An end value that travels one segment a round would make it sixteen times."""
    def best(n):
        K = _keys("quiet", 1, 1, n, d, dtype)
        times = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            _, nnz, khat = da.delta_attn_delta_scan(K, 0.3, want_khat=True)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        assert nnz.item() == d and (khat == K[:, :, :1]).all()
        return min(times)
    short, long = best(16384), best(65536)
    assert long <= 4 * 1.6 * short, (short, long)
