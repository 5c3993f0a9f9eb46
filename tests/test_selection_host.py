"""The smooth-data shortcut of the tangential selections against the exact
weights, on the host: compiled from the kernels' own header (host pass of hipcc,
no device code)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2309_10534_amd", "csrc")


def test_smooth_shortcut_implies_the_large_stencil(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = tmp_path / "selection_host"
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I", CSRC, "-x", "hip",
                    os.path.join(HERE, "selection_host.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
    applied = int(r.stdout.split("applied ")[1].split()[0])
    assert applied > 100000
