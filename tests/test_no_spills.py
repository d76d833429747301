"""The attention kernel with a queue of tiles holds a ticket in a register while it is still on its way, and queries likewise: none of its variants may spill or
copy such a register, or the copy would hold the old value (tiles would be handed out for ever).  What the compiler says of the objects that the library is
linked from, and what it has made of them."""
import os
import re
import subprocess

import pytest

from paper_2507_19608_amd import build

LLVM = "/opt/rocm/llvm/bin"


def _device_code(source, tmp_path):
    obj = os.path.join(build.OBJ, source + ".o")
    if not os.path.exists(obj) or not os.path.exists(os.path.join(LLVM, "clang-offload-bundler")):
        pytest.skip("the library's objects or the compiler's tools are not here")
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, str(tmp_path / "copy.o")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={dev}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    return dev


@pytest.mark.parametrize("source", ["prefill_mfma.hip", "prefill_short.hip"])
def test_nothing_is_spilled(source, tmp_path):
    dev = _device_code(source, tmp_path)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", dev], check=True, capture_output=True, text=True).stdout
    counts = re.findall(r"\.(?:s|v)gpr_spill_count:\s*(\d+)", notes)
    assert len(counts) >= 4 and not any(int(c) for c in counts), notes.count("spill_count")


def test_the_build_refuses_what_spills(tmp_path):
    src, obj = tmp_path / "spills.hip", str(tmp_path / "spills.o")
    src.write_text("""#include <hip/hip_runtime.h>
__global__ __attribute__((amdgpu_num_vgpr(24))) void spills(const float *x, float *y) {
    float v[64];
    for (int i = 0; i < 64; ++i) v[i] = x[i * 64 + threadIdx.x];
    __syncthreads();
    for (int i = 0; i < 64; ++i) y[i * 64 + threadIdx.x] = v[i] * v[63 - i];
}
""")
    build.compile_object(str(src), obj, False)
    assert os.path.exists(obj)
    with pytest.raises(RuntimeError, match="must not spill"):
        build.compile_object(str(src), obj, True)
    assert not os.path.exists(obj)


LINE = re.compile(r"\t(\S+)(.*?)\s*// ([0-9A-F]+): [0-9A-F ]+?(?: <(?:.*\+0x([0-9a-f]+)|[^+]*)>)?\s*$")


def _kernels(text):
    """Kernels of a disassembly, each a list of (address, operation, operands, target's offset from the kernel's first instruction)."""
    kernels, here = {}, None
    for line in text.splitlines():
        if m := re.match(r"[0-9a-f]+ <(.+)>:", line):
            here = kernels[m.group(1)] = []
        elif here is not None and (m := LINE.match(line)):
            here.append((int(m.group(3), 16), m.group(1), m.group(2).strip(), int(m.group(4) or "0", 16)))
    return kernels


def _registers(operands):
    out = set()
    for one, first, last in re.findall(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]", operands):
        out |= {int(one)} if one else set(range(int(first), int(last) + 1))
    return out


def _touched_in_flight(code):
    """(loads found, [(load, instruction)]): instructions that some path reaches from a load that inline assembly leaves in flight, with none of the waits that
    cover it in between, and that have a register of its answer as an operand.  Such a load stands behind an `s_nop 4` of its own."""
    index = {at: i for i, (at, _, _, _) in enumerate(code)}
    target = lambda i: index[code[0][0] + code[i][3]]
    loads, touched = 0, set()
    for i in range(1, len(code)):
        if code[i - 1][1:3] != ("s_nop", "4") or code[i][1] not in ("global_atomic_add", "global_load_dwordx4"):
            continue
        loads += 1
        answer, seen, todo = _registers(code[i][2].split(",")[0]), set(), [(i + 1, 0)]
        while todo:
            j, later = todo.pop()                                # later: requests since, of which a wait may leave as many
            while (j, later) not in seen:
                seen.add((j, later))
                _, op, operands, _ = code[j]
                wait = re.search(r"vmcnt\((\d+)\)", operands) if op == "s_waitcnt" else None
                if op == "s_endpgm" or (wait and int(wait.group(1)) <= later):
                    break
                if _registers(operands) & answer:
                    touched.add((" ".join(code[i][1:3]), f"{op} {operands}"))
                    break
                later = min(later + op.startswith(("global_", "buffer_load", "buffer_store", "scratch_", "flat_")), 63)
                if op.startswith("s_cbranch"):
                    todo.append((target(j), later))
                j = target(j) if op == "s_branch" else j + 1
    return loads, touched


def test_nothing_copies_what_is_in_flight(tmp_path):
    """Paths are taken regardless of what their branches test: some of them, which no wave takes, lead past a wait that only one group of waves makes, to where
    the answer is used or the same thing is asked for again.  Nothing else may stand there, least of all a move or a store."""
    dev = _device_code("prefill_mfma.hip", tmp_path)
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", dev], check=True, capture_output=True, text=True).stdout
    total = 0
    for name, code in _kernels(text).items():
        loads, touched = _touched_in_flight(code)
        total += loads
        for load, use in touched:
            again = use.split()[:2] == load.split()[:2]
            ticket = load.startswith("global_atomic_add") and use.startswith("v_lshlrev_b32")
            query = load.startswith("global_load_dwordx4") and use.startswith("v_mfma_f32_32x32x16_bf16")
            assert again or ticket or query, (name, load, use)
    assert total >= 20


@pytest.mark.parametrize("between,found", [("v_mov_b32_e32 v9, v5", 1), ("v_mov_b32_e32 v9, v6", 0), ("s_waitcnt vmcnt(1)", 1), ("s_waitcnt vmcnt(0)", 0)])
def test_the_search_finds_a_copy(between, found):
    lines = ["s_nop 4", "global_atomic_add v5, v1, v2, s[2:3] sc0", between, "v_mov_b32_e32 v8, v5" if "wait" in between else "s_waitcnt vmcnt(0)", "s_endpgm"]
    text = "0000000000000100 <kernel>:\n" + "".join(f"\t{l} // {256 + 8 * i:012X}: 00000000\n" for i, l in enumerate(lines))
    (code,) = _kernels(text).values()
    assert len(code) == 5 and _touched_in_flight(code)[0] == 1 and len(_touched_in_flight(code)[1]) == found


def _waited_for_at_once(code):
    """(tickets asked for, [instruction that waits for one with no product in between])"""
    index = {at: i for i, (at, _, _, _) in enumerate(code)}
    target = lambda i: index[code[0][0] + code[i][3]]
    tickets, waits = 0, set()
    for i in range(1, len(code)):
        if code[i - 1][1:3] != ("s_nop", "4") or code[i][1] != "global_atomic_add":
            continue
        tickets += 1
        seen, todo = set(), [(i + 1, 0)]
        while todo:
            j, later = todo.pop()
            while (j, later) not in seen:
                seen.add((j, later))
                _, op, operands, _ = code[j]
                if op == "s_endpgm" or op.startswith("v_mfma"):
                    break
                wait = re.search(r"vmcnt\((\d+)\)", operands) if op == "s_waitcnt" else None
                if wait and int(wait.group(1)) <= later:
                    waits.add((code[j][0], operands))
                    break
                later = min(later + op.startswith(("global_", "buffer_load", "buffer_store", "scratch_", "flat_")), 63)
                if op.startswith("s_cbranch"):
                    todo.append((target(j), later))
                j = target(j) if op == "s_branch" else j + 1
    return tickets, waits


def test_nobody_waits_for_a_ticket_at_once(tmp_path):
    """A ticket takes 2 us to come.  Wave 0 has a phase of products to do before it waits for it: a wait in front of the turn's barrier would hold all waves.  (The kernel
    that does not pause between tiles may ask in front of its first one, whose loads it has to wait for anyway.)"""
    dev = _device_code("prefill_mfma.hip", tmp_path)
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", dev], check=True, capture_output=True, text=True).stdout
    found = {name: _waited_for_at_once(code) for name, code in _kernels(text).items() if re.search("prefill_mfma_kernelILi(64ELi[012]|128ELi0)E", name)}
    assert len(found) == 8 and not any(waits for _, waits in found.values()), found
    assert all((tickets == 0) == ("ILi64ELi2E" in name) for name, (tickets, _) in found.items()), found


@pytest.mark.parametrize("between,found", [([], 1), (["v_mfma_f32_32x32x16_bf16 v[8:11], v[12:13], v[14:15], 0"], 0), (["s_waitcnt vmcnt(1)"], 1),
                                           (["global_load_lds_dwordx4 v[2:3], off", "s_waitcnt vmcnt(1)", "v_mfma_f32_32x32x16_bf16 v[8:11], v[12:13], v[14:15], 0"], 1)])
def test_the_search_finds_a_wait(between, found):
    lines = ["s_nop 4", "global_atomic_add v5, v1, v2, s[2:3] sc0", *between, "s_waitcnt vmcnt(0)", "s_endpgm"]
    text = "0000000000000100 <kernel>:\n" + "".join(f"\t{l} // {256 + 8 * i:012X}: 00000000\n" for i, l in enumerate(lines))
    (code,) = _kernels(text).values()
    assert _waited_for_at_once(code)[0] == 1 and len(_waited_for_at_once(code)[1]) == found
