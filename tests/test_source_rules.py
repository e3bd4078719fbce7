"""Rules of the HIP sources that no run can show: what an inline-assembler block has to declare."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_05607_amd", "csrc")


def asm_blocks():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = open(path).read()
        for m in re.finditer(r"\basm\s+volatile\s*\(", text):
            depth, i = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[i], 0)
                i += 1
            yield os.path.basename(path), text[m.end():i - 1]


def test_assembler_that_writes_m0_declares_it():
    # the compiler may keep a value of its own in m0 (indexed registers, its own loads into the LDS)
    found = [(path, body) for path, body in asm_blocks() if re.search(r"s_mov_b32\s+m0", body)]
    assert found
    for path, body in found:
        assert '"m0"' in body.rsplit(":", 1)[1], f"{path}: {body}"
