"""What the scan's kernels take for granted of the rules that cut it."""
import pytest

import scan_plans


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 160, 256])
def test_limits(dtype, d):
    lengths = [*range(1, 600), *(k * 64 + r for k in range(9, 66) for r in (-1, 0, 1)), 5003, 6143, 6144, 8192, 65536]
    for units in (1, 2, 3, 8, 16, 17, 31, 32, 33, 40, 64, 65, 100, 128, 129, 191, 192, 193, 256, 257, 300, 512, 2000):
        for n in lengths:
            w, s = scan_plans.whole(dtype, units, n, d), scan_plans.segments(dtype, units, n, d)
            case = (units, n, w, s)
            if w.L:
                assert w.L % 8 == 0 and w.L <= scan_plans.limit("run") <= 64, case          # a run's rows in the lanes of a wave
                assert w.runs * (w.channels // 2) <= w.threads <= 512 and w.warm % 8 == 0, case   # a thread for two channels of each
                assert w.lds <= scan_plans.limit("lds") and d % w.channels == 0, case
                assert w.channels < 32 or w.rounds >= w.runs, case                          # 32 channels: nothing else settles them
            assert s.nseg == 1 or s.S <= scan_plans.limit("segment"), case
            assert s.nseg == -(-n // s.S) and s.lds <= scan_plans.limit("lds"), case
