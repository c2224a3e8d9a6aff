"""The LDS convolution's slice arithmetic on the host: tests/nn_tile_check.cpp is
compiled against paper_1806_10247_amd/csrc/nn_tile.hpp and run."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_slices_decode_to_tap_and_channel_within_the_tile(tmp_path):
    exe = str(tmp_path / "nn_tile_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1806_10247_amd", "csrc"),
                    os.path.join(ROOT, "tests", "nn_tile_check.cpp"), "-o", exe], check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "0 failures" in r.stdout, r.stdout
