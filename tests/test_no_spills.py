"""The attention kernel with a queue of tiles holds a ticket in a register while it is still on its way, so none of its variants may spill: a copy of that
register would hold the old value, and tiles would be handed out for ever.  What the compiler says of the objects that the library is linked from."""
import glob
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19608_amd", "csrc")
LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.parametrize("source", ["prefill_mfma.hip", "prefill_short.hip"])
def test_nothing_is_spilled(source, tmp_path):
    obj = os.path.join(CSRC, "_obj", source + ".o")
    if not os.path.exists(obj) or not os.path.exists(os.path.join(LLVM, "clang-offload-bundler")):
        pytest.skip("the library's objects or the compiler's tools are not here")
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, str(tmp_path / "copy.o")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={dev}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", dev], check=True, capture_output=True, text=True).stdout
    counts = re.findall(r"\.(?:s|v)gpr_spill_count:\s*(\d+)", notes)
    assert len(counts) >= 4 and not any(int(c) for c in counts), notes.count("spill_count")
