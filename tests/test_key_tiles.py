"""The key tiles that attention.hip brings in through moving descriptors (csrc/key_tiles.h), against following them tile by tile."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_fed_tiles_lie_in_the_cache_or_in_the_block(tmp_path):
    exe = str(tmp_path / "key_tiles")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-I", os.path.join(os.path.dirname(HERE), "paper_2604_16734_amd", "csrc"),
                    os.path.join(HERE, "host_asan", "key_tiles.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr
