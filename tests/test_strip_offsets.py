"""The strip tiles' 32-bit load offsets at the largest sizes that their steps
accept, on the CPU: tests/strip_offsets_check.hip runs the kernels' own offset
functions over the first, middle and last blocks of (mu, nu)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_offsets_fit_32_bits(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    from paper_2012_15662_amd import build as b
    flags = [f for f in b.HIPFLAGS if f not in ("-shared", "-O3")] + ["-O1", "--offload-host-only"]
    exe = str(tmp_path / "strip_offsets_check")
    r = subprocess.run([hipcc, *flags, "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(b.HERE, "csrc"),
                        os.path.join(ROOT, "tests", "strip_offsets_check.hip"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert " 0 failures" in r.stdout
