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


def test_inline_assembly_declares_m0():
    """A statement that changes m0 behind the compiler's back could come between the compiler's own write and use of it."""
    seen = 0
    for path, body in _asm_statements():
        code = " ".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body.split(":")[0]))
        if re.search(r"\bs_\w+\s+m0\b", code):
            seen += 1
            assert re.search(r':[^:]*"m0"\s*$', body.strip()), (path, body)
    assert seen
