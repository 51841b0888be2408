"""The tiles of the long-row stages, by the launch rule itself on the host."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_tiles_of_all_batches(tmp_path):
    from paper_2511_11608_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    exe = str(tmp_path / "tiles")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-w", os.path.join(HERE, "long_row_tiles.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
