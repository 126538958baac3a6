"""Host-only checks of the one-shot batched call, compiled from the library's own
source with stand-ins for the runtime (no GPU needed)."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_one_shot_batches():
    src = os.path.join(ROOT, "tests", "native", "batch_host.cpp")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "batch_host")
        b = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                            "-I", os.path.join(ROOT, "include"),
                            "-I", os.path.join(ROOT, "paper_2504_03667_amd", "csrc"), src, "-o", exe],
                           capture_output=True, text=True)
        assert b.returncode == 0, b.stderr[-3000:]
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        assert "batch host ok" in r.stdout
