"""What the compiler cannot check of the device sources."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_12491_amd", "csrc")


def _asm_statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "**", "*.h*"), recursive=True)):
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"\basm\s+volatile\s*\(", text):
            depth, end = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[end], 0)
                end += 1
            yield f"{os.path.basename(path)}:{text.count(chr(10), 0, m.start()) + 1}", text[m.end():end - 1]


def test_assembly_names_no_register_behind_the_compilers_back():
    """Registers reach an asm statement as operands ("v", "s", "{m0}") only: one that its text names itself is written or read
    without the compiler's knowledge (a clobber list does not help: m0 is reserved there)."""
    found = 0
    for where, stmt in _asm_statements():
        text = " ".join(re.findall(r'"((?:[^"\\]|\\.)*)"', stmt.split(":")[0])).replace("\\n", "\n").replace("\\t", " ")
        named = re.findall(r"\b(?:m0|vcc|exec|scc|[vsa]\d+|[vsa]\[\d+:\d+\])\b", text)
        assert not named, (where, named)
        found += "global_load_lds" in text and '"{m0}"' in stmt
    assert found >= 2                          # the transfers of the streaming score kernels
