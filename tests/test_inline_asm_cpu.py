"""Inline assembly tells the compiler about every register it writes by name."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def statements(src):
    """The operand text of every asm statement."""
    for m in re.finditer(r"\basm\s+volatile\s*\(", src):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = src[i]
            if c == '"' and src[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        yield src[m.end():i - 1]


def test_named_registers_are_clobbers():
    seen = 0
    for f in glob.glob(os.path.join(ROOT, "paper_2604_08542_amd", "csrc", "*")):
        for s in statements(open(f).read()):
            template = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', s.split(":", 1)[0]))
            for reg in re.findall(r"\bs_mov_b32 (m0|exec_lo|exec_hi|vcc_lo|vcc_hi|s\d+)\b", template):
                seen += 1
                assert re.search(rf':[^:]*"{reg}"[^:]*$', s), (os.path.basename(f), s)
    assert seen > 0
