"""The uniform form of a phase (sent in the launch packet, without a program image) says the same as
the phase's steps, over schedules, fold orders, types, chunkings, groups and odd counts. The native
driver expands both forms element by element (CPU only)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2608_00358_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_uniform_form_equals_the_steps(tmp_path):
    exe = str(tmp_path / "uniform_phases")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, os.path.join(HERE, "native", "uniform_phases.cpp"),
                    os.path.join(CSRC, "compiler.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(out.stdout[-2000:])
    assert out.returncode == 0 and "bad 0" in out.stdout, out.stdout[-2000:]
