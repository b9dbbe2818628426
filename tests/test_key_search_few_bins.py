"""The search of test_key_search.py with the histogram of 512 bins that the selection takes for few candidates."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_key_search_with_fewer_bins(tmp_path):
    exe = str(tmp_path / "key_search")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-DKEY_SEARCH_BITS=kvp::kSelectFewBinBits",
                    "-I", os.path.join(os.path.dirname(HERE), "paper_2604_16734_amd", "csrc"),
                    os.path.join(HERE, "host_asan", "key_search.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr
