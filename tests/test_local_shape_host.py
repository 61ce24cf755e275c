"""The local reduce's shape rule (the header the library includes, compiled for
the host): its window keeps the time jitter that the dispatch counts on."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_local_window_keeps_the_promised_span(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", "-I",
                        os.path.join(ROOT, "paper_2106_12863_amd", "csrc"),
                        os.path.join(ROOT, "tests", "local_shape_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "bad 0" in r.stdout
