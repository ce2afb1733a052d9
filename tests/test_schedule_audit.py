"""Shapes and orders of the stage launches on the host (CPU only): the runtime's
own column rules over a range of extents (tests/sanitize/schedule_audit.cpp),
under the host sanitizers."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_schedule_audit(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "schedule_audit")
    san = []
    for f in ("-fsanitize=address,undefined", "-fno-sanitize-recover=all"):
        san += ["-Xarch_host", f]
    r = subprocess.run([hipcc, "--offload-host-only", "-x", "hip", "-std=c++17", "-O1", "-g", *san,
                        "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2107_03747_amd", "csrc"),
                        "-Wno-unused-command-line-argument",
                        os.path.join(ROOT, "tests", "sanitize", "schedule_audit.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 violations" in r.stdout, (r.stdout + r.stderr)[-3000:]
