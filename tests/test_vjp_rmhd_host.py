"""CPU test of the RMHD adjoint's hand-written sweeps: tests/vjp_rmhd_host_check.cpp compiles
the device headers for the host and compares the pair-flux and node sweeps and the WENO
gradient with dual-number derivatives."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rmhd_backward_sweeps_match_dual_numbers(tmp_path):
    hipcc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))
                  if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not available")
    exe = tmp_path / "vjp_rmhd_host_check"
    res = subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950",
                          "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2107_12027_amd", "csrc"),
                          "-o", str(exe), os.path.join(ROOT, "tests", "vjp_rmhd_host_check.cpp")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0, run.stdout
