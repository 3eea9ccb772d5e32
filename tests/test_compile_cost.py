"""Looking for the forms that a launch may take stays cheap beside packing a program (CPU only)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2608_00358_amd", "csrc")

# Packed with the search / without: 1.85-2.1, with every core busy as well; 3.0-3.9 where the search
# sorted all pairs twice.
LIMIT = 2.5


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_packing_a_wide_exchange(tmp_path):
    exe = str(tmp_path / "compile_cost")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, os.path.join(HERE, "native", "compile_cost.cpp"),
                    os.path.join(CSRC, "compiler.cpp"), "-o", exe], check=True)
    for turn in range(3):  # (three tries: a busy host may slow one side of a measurement)
        out = subprocess.run([exe, str(LIMIT)], capture_output=True, text=True, timeout=120)
        print(out.stdout)
        if out.returncode != 1:
            break
    assert out.returncode == 0, out.stdout
