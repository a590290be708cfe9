"""AF_CHECK's status words, read back every 16 steps: every step of a call failing its checks,
and every step not launched after one that did (tests/check_words.cpp, CPU only)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_12915_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc missing")
def test_status_of_every_step(tmp_path):
    exe = str(tmp_path / "check_words")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-O1", "-g", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}",
                    os.path.join(CSRC, "af_api.hip"), "-x", "hip", os.path.join(ROOT, "tests", "check_words.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=900)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr[-2000:]
