"""A record of measured traffic goes stale with any source that decides what a launch runs (CPU only)."""
import os
import shutil

import bench

CSRC = os.path.join(bench.ROOT, "paper_2608_00358_amd", "csrc")


def test_digest_covers_kernels_and_the_code_that_chooses_them(tmp_path):
    copy = tmp_path / "csrc"
    shutil.copytree(CSRC, copy)
    whole = bench.library_digest(str(copy))
    assert whole == bench.library_digest()
    for name in ("executor_uniform.hip", "executor_runs.h", "compiler.cpp", "program.h", "api.cpp"):
        with open(copy / name, "a") as f:
            f.write("// changed\n")
        changed = bench.library_digest(str(copy))
        assert changed != whole, name
        whole = changed
