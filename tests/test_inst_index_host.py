"""The institution index's host build and slot lookup (the header the kernel
includes, compiled for the host) against a plain interval search."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_inst_index_host_lookup_vs_interval_search(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", "-I",
                        os.path.join(ROOT, "paper_2106_12863_amd", "csrc"),
                        os.path.join(ROOT, "tests", "inst_index_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "bad 0" in r.stdout
