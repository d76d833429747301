"""Build libdelta_attn.so (HIP, gfx950) in-tree with hipcc, and, where there are torch and g++, the binding's compiled part.  No GPU is
needed to compile."""
import glob
import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_obj")
LIB = os.path.join(HERE, "libdelta_attn.so")
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))   # (another Python does not find it)

# packed fp32 instructions are switched off for every device compile (hipcc's host pass warns
# that it does not know the feature; harmless)
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-command-line-argument",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# Kernels whose loads are inline assembly.  A register that such a load has still to write and that is spilled meanwhile is stored
# with its old value, and an address that comes back from a spill may be used too early: where one of these spills there is no library.
NO_SPILLS = ("prefill_mfma.hip", "prefill_short.hip")


def compile_object(src: str, obj: str, no_spills: bool) -> None:
    cmd = ["hipcc"] + HIPCC_FLAGS + (["-Rpass-analysis=kernel-resource-usage"] if no_spills else []) + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    spills = [int(n) for n in re.findall(r"remark: .*[SV]GPRs Spill: (\d+)", r.stderr)]
    if r.returncode == 0 and no_spills and (not spills or any(spills)):
        os.remove(obj)
        raise RuntimeError(f"{src}: kernels that must not spill registers do: {spills}")
    # (what is left of a remark are the source lines that the compiler quotes under it)
    err = re.sub(r"[^\n]*remark: [^\n]*\n(?: *\d* \|[^\n]*\n)*", "", r.stderr + "\n") if no_spills else r.stderr
    err = "\n".join(l for l in err.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    deps = [src] + glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    if force or not os.path.exists(obj) or any(os.path.getmtime(obj) < os.path.getmtime(d) for d in deps):
        compile_object(src, obj, os.path.basename(src) in NO_SPILLS)
    return obj


def build_marshal(force: bool) -> None:
    """The binding's compiled part.  It calls the library through addresses that it is given, and links to torch alone: the one that it
    is built for, which it keeps the name of (the binding takes it for no other)."""
    try:
        import torch
    except ImportError as e:
        raise RuntimeError(f"there is no torch ({e})")
    src, built_for = os.path.join(CSRC, "marshal.cpp"), os.path.join(OBJ, "marshal.built_for")
    deps = [src] + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    if not force and os.path.exists(MARSHAL) and all(os.path.getmtime(MARSHAL) >= os.path.getmtime(d) for d in deps) \
            and os.path.exists(built_for) and open(built_for).read() == torch.__version__:
        return
    at = os.path.dirname(torch.__file__)
    include = [os.path.join(at, "include"), os.path.join(at, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include",
               sysconfig.get_paths()["include"]]
    r = subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-std=c++17", "-Wall", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                        f'-DBUILT_FOR="{torch.__version__}"']
                       + [a for d in include for a in ("-isystem", d)] + [src, "-o", MARSHAL, "-L" + os.path.join(at, "lib")]
                       + ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for {src}:\n{r.stderr}")
    sys.stderr.write(r.stderr)
    with open(built_for, "w") as f:
        f.write(torch.__version__)


def build(force: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        marshal = ex.submit(build_marshal, force)
        objs = list(ex.map(lambda s: _compile(s, force), srcs))
    if force or not os.path.exists(LIB) or any(os.path.getmtime(o) > os.path.getmtime(LIB) for o in objs):
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, check=True)
    try:
        marshal.result()
    except (RuntimeError, OSError) as e:                         # (no torch, no g++, no headers: whoever calls the library from C needs none)
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)                                   # (of other sources, or another torch)
        sys.stderr.write(f"{MARSHAL} is not built, the binding marshals in Python: {e}\n")
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
