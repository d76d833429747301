"""The binding's compiled calls: the same results, refusals and objects as its Python code, which takes whatever is not in order."""
import gc
import struct
import sys
import threading
import time

import pytest
import torch

from paper_2507_19608_amd import binding as da


def test_leaves_what_is_not_in_order_to_python():
    from paper_2507_19608_amd import _marshal as m
    t = torch.zeros(1, 2, 64, 64)
    for args in ((), (t, t, t, 0.1, 8, 0.0, 0, 0, 0, None, None), (None,) * 11, (1, 2, 3, 0.1, 8, 0.0, 0, 0, 0, None, None)):
        assert m.prefill(*args) is None                        # (tensors of the CPU among them)
    for args in ((), (b"", t, t, t, None, None), (bytes(32), t, t, t, None, None), (None,) * 6):
        assert m.decode(*args) is None


def _qkv(B, Hq, Hkv, n, d, dt):
    g = torch.Generator(device="cuda").manual_seed(n)
    return tuple(torch.randn(B, h, n, d, generator=g, device="cuda").to(dt) for h in (Hq, Hkv, Hkv))


@pytest.fixture
def both_ways(monkeypatch):
    def call(f):
        assert da._torch() and da._marshal is not None
        fast = f()
        with monkeypatch.context() as m:
            m.setattr(da, "_marshal", None)
            slow = f()
        return fast, slow
    return call


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 1, 1, 256, 64, torch.float32), (1, 32, 8, 333, 64, torch.bfloat16), (2, 4, 2, 40, 96, torch.bfloat16)])
def test_prefill_both_ways(both_ways, shape):
    q, k, v = _qkv(*shape)
    fast, slow = both_ways(lambda: da.delta_attn_prefill(q, k, v, 0.3, 16))
    for a, b in zip(fast, slow):
        assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device and torch.equal(a, b)
    # theta as a whole number, and the caller's own buffers, which come back as they are
    out = tuple(torch.empty_like(t) for t in fast)
    ws = torch.empty(da.delta_attn_prefill_workspace_bytes(da.make_params(q, k, 16, 0.0)), dtype=torch.uint8, device="cuda")
    for got in both_ways(lambda: da.delta_attn_prefill(q, k, v, 0, 16, window_mode=da.DA_WINDOW_SLIDING, workspace=ws, out=out)):
        assert all(a is b for a, b in zip(got, out))


@pytest.mark.gpu
def test_strides_of_one_row(both_ways):
    q, k, v = _qkv(1, 2, 2, 1, 64, torch.bfloat16)
    odd = torch.empty_strided((1, 2, 1, 64), (7, 64, 13, 1), dtype=q.dtype, device="cuda").copy_(q)
    assert odd.is_contiguous()
    for a, b in zip(*both_ways(lambda: da.delta_attn_prefill(odd, k, v, 0.3, 16))):
        assert a.stride() == b.stride() and torch.equal(a, b)


@pytest.mark.gpu
def test_refusals_both_ways(monkeypatch):
    q, k, v = _qkv(1, 4, 2, 64, 64, torch.bfloat16)
    cache = da.Cache(1, 4, 2, 64, 4, 4, 0.1, torch.bfloat16)
    one = [t[:, :, 0].contiguous() for t in (q, k, v)]
    calls = [lambda: da.delta_attn_prefill(q, k, v.float(), 0.1, 8), lambda: da.delta_attn_prefill(q.transpose(1, 2), k, v, 0.1, 8),
             lambda: da.delta_attn_prefill(q.half(), k.half(), v.half(), 0.1, 8), lambda: da.delta_attn_prefill(q, k, v, -1.0, 8),
             lambda: da.delta_attn_prefill(q, k, v, 0.1, 0), lambda: da.delta_attn_prefill(q, k, v, 0.1, 8, score_mode=7),
             lambda: da.delta_attn_prefill(q, k, v, 0.1, 8, workspace=torch.empty(16, dtype=torch.uint8, device="cuda")),
             lambda: da.delta_attn_prefill(q, k, v, 0.1, 8, cache=cache), lambda: da.delta_attn_prefill(q.cpu(), k, v, 0.1, 8),
             lambda: da.delta_attn_prefill([q], k, v, 0.1, 8), lambda: da.delta_attn_prefill(q, k, v, "x", 8),
             lambda: da.delta_attn_decode(cache, one[0], one[1], one[2].float()), lambda: da.delta_attn_decode(cache, one[1], one[1], one[2])]

    def said():
        texts = []
        for f in calls:
            with pytest.raises(Exception) as e:
                f()
            texts.append((type(e.value), str(e.value)))
        return texts
    fast = said()
    monkeypatch.setattr(da, "_marshal", None)
    assert said() == fast


@pytest.mark.gpu
def test_decode_both_ways(monkeypatch):
    got = []
    for way in (da._marshal, None) if da._torch() else ():
        monkeypatch.setattr(da, "_marshal", way)
        cache = da.Cache(2, 8, 2, 64, 3, 3, 0.2, torch.bfloat16)
        rows = []
        for step in range(3):
            q, k, v = (t[:, :, 0].contiguous() for t in _qkv(2, 8, 2, 1 + step, 64, torch.bfloat16))
            out, row = torch.empty_like(q), torch.empty(2, 2, 2, dtype=torch.int32, device="cuda")
            if step == 1:
                o, m = da.delta_attn_decode(cache, q, k, v)
            else:
                o, m = da.delta_attn_decode(cache, q, k, v, out=out, mask_row=row)
                assert o is out and m is row
            rows += [o, m]
        with pytest.raises(da.DeltaAttnError) as e:                # full
            da.delta_attn_decode(cache, q, k, v)
        rows.append(str(e.value))
        cache.close()
        with pytest.raises(da.DeltaAttnError) as e:                # closed
            da.delta_attn_decode(cache, q, k, v)
        rows.append(str(e.value))
        got.append(rows)
    for a, b in zip(*got):
        assert a == b if isinstance(a, str) else torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("asks_for", ["a prefill's workspace", "a prefill's output", "a decode step's output"])
def test_other_threads_run_while_memory_is_asked_for(asks_for):
    """Memory that torch has to ask the driver for takes long, and waits for the device where others' is freed first: no other Python thread may stand
    still for it.  There is none left here: each call ends where it asks for it, with nothing launched.  Threads are only switched where one gives the
    interpreter up, so that the count moves only if the call does."""
    assert da._torch() and da._marshal is not None
    if asks_for == "a decode step's output":                       # (no cache: a step that came as far as the library would be refused)
        q, k, v = (torch.empty(4096, h, 128, dtype=torch.bfloat16, device="cuda") for h in (64, 1, 1))
        args = da._marshal.decode, struct.pack("P6i", 0, 4096, 64, 1, 128, da.DA_BF16, 0), q, k, v, None, None
    else:
        q, k, v = (torch.empty(1, h, 1 << 16, 64, dtype=torch.bfloat16, device="cuda") for h in (32, 1, 1))
        ws = None if asks_for == "a prefill's workspace" else torch.empty(16, dtype=torch.uint8, device="cuda")
        args = da._marshal.prefill, q, k, v, 0.1, 64, 0.0, 0, 0, 0, ws, None
    count, stop = [0], threading.Event()

    def others():
        while not stop.is_set():
            count[0] += 1
            time.sleep(1e-5)
    thread, moved, interval = threading.Thread(target=others), 0, sys.getswitchinterval()
    gc.collect()                                                   # (tensors that an earlier test's exceptions still hold)
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-6)
    thread.start()
    sys.setswitchinterval(1000)
    try:
        for _ in range(100):
            before = count[0]
            with pytest.raises(torch.OutOfMemoryError):
                args[0](*args[1:])
            moved += count[0] != before
    finally:
        sys.setswitchinterval(interval)
        stop.set()
        thread.join()
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert moved
