"""What the kernels' sources have to keep to, seen without a GPU."""
import os
import re

from paper_2212_05231_amd import build as b

FILES = sorted(f for f in os.listdir(b.CSRC) if f.endswith((".hip", ".h")))


def test_asm_statements_hold_no_instruction():
    """The compiler puts the wait states that a matrix instruction needs in front of its own instructions only: one written in
    asm text may be given a register that the matrix instruction is still to write, among them those of a result that nobody
    reads.  So an asm statement is an empty barrier to the optimiser, in every kernel, whatever registers it is given."""
    found = 0
    for name in FILES:
        with open(os.path.join(b.CSRC, name)) as f:
            text = re.sub(r"//[^\n]*", "", f.read())
        for statement in re.finditer(r"\b(?:asm|__asm__)\s*(?:volatile\s*)?\(\s*(\"(?:[^\"\\]|\\.)*\")", text):
            found += 1
            line = text[:statement.start()].count("\n") + 1
            assert statement.group(1) == '""', f"{name}:{line}: asm text {statement.group(1)}"
        assert len(re.findall(r"\b(?:asm|__asm__)\b", text)) == len(re.findall(r"\b(?:asm|__asm__)\s*(?:volatile\s*)?\(\s*\"", text)), name
    assert found > 0
