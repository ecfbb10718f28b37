"""Inline asm of the kernels: the compiler adds no wait states inside an asm block, so the one that the hardware needs between
a scalar write of m0 and a copy to LDS (which takes its LDS address from m0) has to be written out; and it does not know of the copies
that are in flight, so a wait written by hand may count only what is written by hand."""
import glob
import os
import re
import subprocess

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


def test_no_wait_counts_loads_that_the_compiler_makes(tmp_path):
    """The fp32 kernel for small steps copies keys to LDS in asm and leaves the loads of the values to the compiler, which may make fewer or
    more of them: in its machine code no wait from the source leaves a
    number of loads in flight."""
    asm = str(tmp_path / "few_f32.s")
    flags = [f for f in build.HIPCC_FLAGS if not f.startswith("-Rpass")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "attn_few_f32.hip"), "-o", asm],
                   check=True, capture_output=True)
    text = open(asm).read()
    kernels = re.findall(r"^(_ZN\w*attn_few_f32_kernel\w*):.*?s_endpgm", text, re.S | re.M)
    assert len(kernels) == 4
    written = re.findall(r"#ASMSTART\s*\n\s*s_waitcnt vmcnt\((\d+)\)", text)
    assert written and set(written) == {"0"}
