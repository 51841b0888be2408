"""The row kernel's reads of LDS stay inside its allocation for every block layout: the kernel's own index functions, on the host."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_block_ordered_values_are_read_inside_lds(tmp_path):
    from paper_2511_11608_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    exe = str(tmp_path / "reach")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-w", os.path.join(HERE, "row_kernel_reach.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
