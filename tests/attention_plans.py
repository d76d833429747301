"""How the tile-by-tile attention cuts a prompt into tiles and which of its kernels takes them, by the rule as the library's source has it, compiled for the CPU: a
test that wants a certain form takes its shapes from here, and a rule that changes cannot leave the test without it."""
import ctypes
import os
import re
import subprocess
import tempfile
from collections import namedtuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256                                                          # compute units of an MI355X

# tiles of both kinds, the split ones of these, resident work groups; stream: the kernel with one barrier a turn on split tiles (head_dim 64), without a pause between
# whole ones (head_dim 128)
Launch = namedtuple("Launch", "tiles split resident stream")

_lib = None


def _rule():
    global _lib
    if _lib is None:
        text = {f: open(os.path.join(ROOT, "paper_2507_19608_amd", "csrc", f)).read() for f in ("kernels.hpp", "mfma.hpp", "prefill_mfma.hip")}

        def piece(source, start, end):
            found = re.findall(rf"^{start}.*?^{end}", text[source], re.S | re.M)
            assert len(found) == 1, (start, len(found))
            return found[0]
        code = "\n".join([
            "#include <atomic>\n#include <cmath>\n#include <cstddef>\n#include <cstdint>\n#include <utility>",
            "typedef unsigned short bf16_t; typedef void *hipStream_t; struct dim3 { int x; dim3(int x) : x(x) {} }; struct CacheFill { int items; };",
            f"static int device_cu_count() {{ return {CUS}; }}\nstatic void ensure_dynamic_lds(const void *, int, std::atomic<uint64_t> &) {{}}\nstatic int64_t got[4];",
            "#define hipLaunchKernelGGL(kernel, grid, block, lds, s, a, ...) (got[0] = (a).blocks, got[1] = (a).kinds[1].end, got[2] = slots, got[3] = stream)",
            piece("kernels.hpp", r"struct NnzSum \{", r"\};"), piece("kernels.hpp", r"struct PrefillArgs \{", r"\};"),
            piece("mfma.hpp", r"struct Divisor \{", r"\};"), piece("mfma.hpp", r"inline Divisor divisor\(", r"\}$"),
            piece("prefill_mfma.hip", r"constexpr int KB\b", r"constexpr int kQueueStride").rsplit("\n", 1)[0],
            piece("prefill_mfma.hip", r"struct MfmaArgs \{", r"\};"),
            "template <int D, int kForm, typename... Fill> static void prefill_mfma_kernel(MfmaArgs, Fill...) {}",
            piece("prefill_mfma.hip", r"int resident\(", r"\}$"), piece("prefill_mfma.hip", r"template <int D>\nvoid launch_d\(", r"\}$"),
            """extern "C" void plan(int B, int Hq, int Hkv, int d, int n, int nq, int W, int sliding, int64_t *o) {
    PrefillArgs p = {};
    p.dtype = 1, p.B = B, p.Hq = Hq, p.Hkv = Hkv, p.d = d, p.n = n, p.W = W, p.q_off = n - nq, p.nq = nq, p.sliding = sliding;
    d == 64 ? launch_d<64>(p, nullptr, nullptr) : launch_d<128>(p, nullptr, nullptr);
    for (int k = 0; k < 4; ++k) o[k] = got[k];
}
"""])
        with tempfile.TemporaryDirectory() as at:
            src, lib = os.path.join(at, "plans.cpp"), os.path.join(at, "plans.so")
            with open(src, "w") as f:
                f.write(code)
            subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", src, "-o", lib], check=True)
            _lib = ctypes.CDLL(lib)
    return _lib


def launch(B, Hq, Hkv, d, n, W, sliding=False, nq=None):
    out = (ctypes.c_int64 * 4)()
    _rule().plan(B, Hq, Hkv, d, n, n if nq is None else nq, W, int(sliding), out)
    return Launch(out[0], out[1], out[2], bool(out[3]))
