"""Rules that the kernels and their launchers take from integers alone (waits, splits, block
orders), checked over their whole ranges on the CPU: each program under tests/host includes the
library's own headers, is compiled for the host only and runs without a GPU."""
import os
import subprocess

import pytest

from paper_2607_17644_amd import build as B

HOST = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.mark.parametrize("name", ["dkdv_split_waits", "gemm_ranges", "block_order", "ring_tiles", "out_proj_splits"])
def test_rule(name, tmp_path):
    exe = str(tmp_path / name)
    r = subprocess.run([B.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I",
                        os.path.join(B.ROOT, "include"), "-I", B.CSRC, os.path.join(HOST, name + ".cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
