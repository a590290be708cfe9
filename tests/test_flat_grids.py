"""Grids of four rows or columns: their tiles are mostly empty, so a step of few cells has many
work-items, and HIP takes fewer than 2^32 along an axis of a launch."""
import os
import subprocess

import pytest

from paper_2605_12915_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_12915_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc missing")
def test_tile_runs(tmp_path):
    exe = str(tmp_path / "tile_runs")
    subprocess.run([HIPCC, "-std=c++17", "-O1", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}",
                    os.path.join(ROOT, "tests", "tile_runs.cpp"), "-o", exe], check=True, capture_output=True, timeout=900)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr


@pytest.mark.gpu
def test_flat_step():
    """1.3e8 x 4 cells (FP64; 4.4e9 work-items, 133 GB with the second state): a 260 x 4 flow
    repeated 5e5 times steps as the 260 x 4 grid does."""
    import torch

    from paper_2605_12915_amd.stepper import Stepper
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    reps = 500_000
    P = I.random_smooth(260, 4, seed=5, amp=0.1, vel=(0.35, -0.25))
    s0, dt = torch.from_numpy(P.state()).to(dev), P.dt_for_cfl(0.4)
    if torch.cuda.mem_get_info(dev)[0] < 160e9:
        pytest.skip("needs 160 GB of device memory")
    x = torch.empty((16, 4, reps * 260), dtype=torch.float64, device=dev)
    for k in range(16):
        x[k].view(4, reps, 260).copy_(s0[k][:, None, :].expand(4, reps, 260))
    print("flat grid", reps * 260, "x 4", flush=True)
    st = Stepper(reps * 260, 4, P.h, P.gamma, check_errors=False, device=dev)
    st.step(x, dt, 2)
    assert st.read_status() == 0
    small = Stepper(260, 4, P.h, P.gamma, check_errors=True, device=dev)
    small.step(s0, dt, 2)
    for k in range(16):
        err = (x[k].view(4, reps, 260) - s0[k][:, None, :]).abs_().max()
        assert float(err) <= 1e-12 * float(s0[k].abs().max()), k
    del x, st
    torch.cuda.empty_cache()
