"""Division by a number that the host knows (csrc/divide.h), as the kernels do it, against the integer division."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_quotient_is_the_integer_division(tmp_path):
    exe = str(tmp_path / "divide")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-I", os.path.join(os.path.dirname(HERE), "paper_2604_16734_amd", "csrc"),
                    os.path.join(HERE, "host_asan", "divide.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr
