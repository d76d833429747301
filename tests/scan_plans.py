"""The rules that choose how a scan is cut, as the library's source has them, compiled for the CPU: a test that wants a certain number of runs takes it
from here, and a rule that changes cannot leave the test without them."""
import ctypes
import os
import re
import subprocess
import tempfile
from collections import namedtuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256                                                          # compute units of an MI355X

Whole = namedtuple("Whole", "channels threads L warm rounds lds runs")      # of scan_whole_kernel; L == 0: not for it
Segments = namedtuple("Segments", "S nseg warm channels waves lds")

_lib = None


def _rules():
    global _lib
    if _lib is None:
        text = open(os.path.join(ROOT, "paper_2507_19608_amd", "csrc", "delta_scan.hip")).read()

        def piece(start, end):
            found = re.findall(rf"^{start}.*?^{end}", text, re.S | re.M)
            assert len(found) == 1, (start, len(found))
            return found[0]
        code = "\n".join(["#include <cstddef>", "#include <cstdint>", "constexpr int kWave = 64;", f"static int device_cu_count() {{ return {CUS}; }}"]
                         + [re.search(rf"^constexpr int {name} = [^;]*;", text, re.M).group(0) for name in ("kScanLdsMax", "kSettleWaves", "kMostSegment")]
                         + [piece(r"struct ScanPlan \{", r"\};"), piece(r"static ScanPlan scan_plan\(", r"\}$"),
                            piece(r"struct WholePlan \{", r"\};"), piece(r"constexpr int kMostRun\b", r"\}$"),
                            """extern "C" int most_lds() { return kScanLdsMax; }
extern "C" int most_run() { return kMostRun; }
extern "C" int most_segment() { return kMostSegment; }
extern "C" void whole(int t, int u, int n, int d, int64_t *o) {
    const WholePlan p = whole_plan(t, u, n, d);
    const int64_t v[] = {p.dl, p.threads, p.L, p.warm, p.rounds, (int64_t)p.lds, p.L ? (n + p.L - 1) / p.L : 0};
    for (int k = 0; k < 7; ++k) o[k] = v[k];
}
extern "C" void segments(int t, int u, int n, int d, int64_t *o) {
    const ScanPlan p = scan_plan(t, u, n, d);
    const int64_t v[] = {p.S, p.nseg, p.warm, p.dl, p.waves, (int64_t)p.lds};
    for (int k = 0; k < 6; ++k) o[k] = v[k];
}
"""])
        with tempfile.TemporaryDirectory() as at:
            src, lib = os.path.join(at, "plans.cpp"), os.path.join(at, "plans.so")
            with open(src, "w") as f:
                f.write(code)
            subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", src, "-o", lib], check=True)
            _lib = ctypes.CDLL(lib)
    return _lib


def _ask(name, kind, dtype, units, n, d):
    out = (ctypes.c_int64 * len(kind._fields))()
    getattr(_rules(), name)({"f32": 0, "bf16": 1}[dtype], units, n, d, out)
    return kind(*out)


def whole(dtype, units, n, d):
    return _ask("whole", Whole, dtype, units, n, d)


def segments(dtype, units, n, d):
    return _ask("segments", Segments, dtype, units, n, d)


def limit(name):
    return getattr(_rules(), "most_" + name)()
