"""How many workgroups of a kernel a CU holds at once, from the registers and the LDS that the compiler gives it: launch rules
(csrc/plan.cpp) count on these."""
import os
import re
import subprocess

import pytest

from paper_2604_16734_amd import build as B

LDS_OF_A_CU = 160 * 1024


def _registers_and_waves(source, tmp_path):
    """{mangled kernel name: (vector registers, waves per SIMD, bytes of scratch memory)} as the compiler reports them."""
    cmd = [B._hipcc()] + B.FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(B.CSRC, source),
                                    "-o", str(tmp_path / "device.o")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    found = {}
    for part in r.stderr.split("Function Name: ")[1:]:
        number = lambda what: int(re.search(what + r".*?: (\d+)", part).group(1))
        found[part.split()[0]] = number("VGPRs"), number("Occupancy"), number("ScratchSize")
    return found


def test_split_key_workgroups_at_d_64(tmp_path):
    """Without scores two workgroups of eight waves on the four SIMDs of a CU, with either number of row tiles."""
    try:
        B._hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    kernels = _registers_and_waves("attention_split.hip", tmp_path)
    for row_tiles in (1, 2):
        name, = [k for k in kernels if "attention_split_kernelILi64ELi%dELi0EE" % row_tiles in k]
        registers, waves, scratch = kernels[name]
        assert waves >= 4 and scratch == 0, (name, registers, waves, scratch)
        rows, strips = 32 * row_tiles, 2 * 8 * 32 * 64 * 2
        assert 2 * (strips + 2 * 8 * 32 * 4 + rows * 64 * 2 + rows * 4) <= LDS_OF_A_CU
