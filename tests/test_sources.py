"""Properties of the kernel sources that no run can be relied on to show."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_19608_amd", "csrc")


def _asm_statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
            depth, i = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[i], 0)
                i += 1
            yield os.path.basename(path), text[m.end():i - 1]


def test_inline_assembly_leaves_m0_to_the_compiler():
    """m0 is the compiler's register: a statement that changed it behind its back could come between the compiler's own write
    and use.  Statements that need it take it as an operand."""
    seen = 0
    for path, body in _asm_statements():
        code = " ".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body.split(":")[0]))
        writes = re.findall(r"\bs_\w+\s+m0\b", code)
        assert not writes, (path, writes)
        if "load_lds" in code:
            seen += 1
            assert '"{m0}"' in body, (path, body)
    assert seen
