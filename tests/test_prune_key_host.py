"""csrc/prune_key.h, the key of a block, compiled for the host: ordinary blocks against plain sums,
and a block of 2^32 elements, whose count does not fit in 32 bits (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_block_key_counts_every_element(tmp_path):
    exe = str(tmp_path / "prune_key_count")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wno-unknown-pragmas",
                        "-I", os.path.join(ROOT, "paper_2106_08846_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "prune_key_count.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
