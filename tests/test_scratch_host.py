"""Scratch memory asked for and calls that run with less, on the CPU: the library's
objects linked against tests/scratch_host_check.hip, which answers the HIP runtime's
calls (allocations up to a size it sets, launches that do nothing)."""
import os
import shutil
import subprocess

import pytest

from tests.test_abi_host_sanitized import CSRC, ROOT, _objects


def test_scratch_sizes_and_fallbacks(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    from paper_2012_15662_amd import build as b
    objs = _objects() + [os.path.join(b.HERE, "_build", "rif_api.hip.o")]
    flags = [f for f in b.HIPFLAGS if f not in ("-shared", "-O3")] + ["-O1"]
    obj, exe = str(tmp_path / "check.o"), str(tmp_path / "check")
    r = subprocess.run([hipcc, *flags, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-c",
                        os.path.join(ROOT, "tests", "scratch_host_check.hip"), "-o", obj], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([hipcc, "--offload-arch=gfx950", obj, *objs, "-o", exe, "-L/opt/rocm/lib", "-lrocsolver", "-lrocblas",
                        "-Wl,-rpath,/opt/rocm/lib"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert " 0 failures" in r.stdout
