"""Inline asm of the kernels: the compiler adds no wait states inside an asm block, so the one that the hardware needs between
a scalar write of m0 and a copy to LDS (which takes its LDS address from m0) has to be written out."""
import glob
import os
import re

from paper_2605_12471_amd import build


def _asm_blocks():
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*.h")) + glob.glob(os.path.join(build.CSRC, "*.hip"))):
        for m in re.finditer(r'asm volatile\(((?:\s*"(?:[^"\\]|\\.)*")+)', open(path).read()):
            text = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', m.group(1)))
            yield os.path.basename(path), [i.strip() for i in re.split(r"\\n|\\t", text) if i.strip()]


def test_wait_state_between_m0_and_copy_to_lds():
    copies = 0
    for name, instructions in _asm_blocks():
        for i, ins in enumerate(instructions):
            if re.match(r"(global|buffer|scratch)_load_lds_|buffer_load_\w+ .*\blds\b", ins):
                copies += 1
                writes = [j for j in range(i) if re.match(r"s_\w+ m0\b", instructions[j])]
                assert writes, f"{name}: {ins}: m0 is not set in the block"
                assert i - writes[-1] >= 2, f"{name}: no wait state between '{instructions[writes[-1]]}' and '{ins}'"
    assert copies
