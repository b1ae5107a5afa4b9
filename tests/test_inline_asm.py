"""Inline assembly of the kernels: nothing but what its text says stands between two instructions of a block, so the wait states
of the instruction set have to be written out."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1812_07816_amd", "csrc")


def _blocks():
    """(file, instructions) of every asm statement: its string literals joined, split at line ends."""
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r'\basm\s+volatile\s*\(((?:\s*"(?:[^"\\]|\\.)*")+)', text):
            body = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', m.group(1)))
            yield os.path.basename(path), [i.strip() for i in re.split(r"\\n|;", body.replace("\\t", " ")) if i.strip()]


def test_a_load_to_lds_waits_for_m0():
    """One wait state between a scalar write of M0 and a load that takes its LDS address from it."""
    writes = 0
    for name, ins in _blocks():
        for i, a in enumerate(ins):
            if not re.match(r"s_mov_b32 m0\b", a):
                continue
            writes += 1
            assert i + 1 < len(ins) and ins[i + 1].startswith("s_nop"), (name, ins)
    assert writes == 2, writes      # load_lds_asm and dma16: the expression above still finds them
