"""Host-only checks of rules on the shape of a round, compiled from the library's own
headers (no GPU needed)."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_round_rules():
    src = os.path.join(ROOT, "tests", "native", "round_rules.cpp")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "round_rules")
        b = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                            "-I", os.path.join(ROOT, "include"),
                            "-I", os.path.join(ROOT, "paper_2504_03667_amd", "csrc"), src, "-o", exe],
                           capture_output=True, text=True)
        assert b.returncode == 0, b.stderr[-3000:]
        r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        assert "round rules ok" in r.stdout
