"""The step kernels' tiles walked on the host under the sanitizers, every shape that is launched
(tests/step_bounds.cpp; CPU only)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_12915_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc missing")
def test_step_tiles_walk(tmp_path):
    exe = str(tmp_path / "step_bounds")
    subprocess.run([HIPCC, "-std=c++17", "-O0", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host",
                    "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=all", f"-I{CSRC}",
                    f"-I{os.path.join(ROOT, 'include')}", os.path.join(ROOT, "tests", "step_bounds.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=900)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=900, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
