"""Host-side check of the candidate bytes' geometry (tests/candidate_bytes_check.cpp,
built with the kernels' own index header).  CPU only: it runs no kernel."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_candidate_bytes(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = tmp_path / "candidate_bytes_check"
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1",
                    "-I", os.path.join(ROOT, "paper_1502_07303_amd", "csrc"),
                    os.path.join(ROOT, "tests", "candidate_bytes_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
