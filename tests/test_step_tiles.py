"""The tile variants of the fused step: which grid takes which is a rule on its size, so
sizes on both sides of the rule, whole tiles and remainders, long and flat grids, both point
updates, against the oracle; and the packed tile's indexing walked on the host."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_12915_amd import inputs as I

from tests.f32bound import f32_tolerance

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_12915_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

# 4x4 tiles: up to 256; 8x8 tiles: up to 256 in FP64, up to 640 in FP32; in FP32 1024 threads up to 256 tiles of 31x10
SIZES = [(64, 64), (65, 64), (4, 4), (5, 203), (128, 128), (129, 128), (150, 150), (151, 149), (16, 1030), (2061, 13), (165, 100), (200, 205), (208, 200),
         (248, 320), (249, 320), (125, 511)]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc missing")
def test_packed_tile_walk(tmp_path):
    exe = str(tmp_path / "packed_tile")
    subprocess.run([HIPCC, "-std=c++17", "-O0", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host",
                    "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=all", f"-I{CSRC}",
                    f"-I{os.path.join(ROOT, 'include')}", os.path.join(ROOT, "tests", "packed_tile.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=900)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]


@pytest.mark.gpu
@pytest.mark.parametrize("scheme", ["tai", "rb"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_step_vs_oracle(orc, nx, ny, scheme):
    import torch

    from paper_2605_12915_amd.stepper import Stepper, from_perturbation, to_perturbation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    P = I.random_smooth(nx, ny, seed=nx + 7 * ny, amp=0.1, vel=(0.35, -0.25))
    s0, n = P.state(), 2
    dt = P.dt_for_cfl(0.19 if scheme == "rb" else 0.4)
    print("tiles", nx, ny, scheme, flush=True)
    want = orc.run(s0, P.h, P.gamma, dt, n, scheme=1 if scheme == "rb" else 0)
    st = Stepper(nx, ny, P.h, P.gamma, scheme=scheme, device=dev, check_errors=True)
    x = torch.from_numpy(s0).to(dev)
    st.step(x, dt, n)
    err = np.abs(x.cpu().numpy() - want).max(axis=(1, 2)) / np.abs(want).max(axis=(1, 2))
    assert err.max() <= 1e-12, (st.dominant_kernel(), err)
    st = Stepper(nx, ny, P.h, P.gamma, precision="f32", scheme=scheme, bg=P.bg, device=dev, check_errors=True)
    x = torch.from_numpy(to_perturbation(s0, P.bg, P.gamma)).to(dev)
    st.step(x, dt, n)
    err = np.abs(from_perturbation(x.cpu().numpy(), P.bg, P.gamma) - want).max(axis=(1, 2))
    tol = f32_tolerance(want, s0, P.bg, P.gamma, n)
    assert np.all(err <= tol), (st.dominant_kernel(), err / tol)


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(24, 17), (77, 65), (208, 200), (300, 301)])   # one of each FP32 kernel
def test_f32_new_trajectory(nx, ny):
    """A call on another buffer reads nothing of the compensation that an earlier trajectory
    left: bit for bit the result of a new context, checked steps too."""
    import torch

    from paper_2605_12915_amd.stepper import Stepper, to_perturbation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    P = I.random_smooth(nx, ny, seed=nx, amp=0.1, vel=(0.35, -0.25))
    s0, dt = to_perturbation(P.state(), P.bg, P.gamma), P.dt_for_cfl(0.4)
    got = []
    for used, check in ((False, False), (True, False), (True, True)):
        st = Stepper(nx, ny, P.h, P.gamma, precision="f32", bg=P.bg, device=dev, check_errors=check)
        if used:
            y = torch.from_numpy(s0).to(dev)
            st.step(y, dt, 3)
        x, z = torch.from_numpy(s0).to(dev), torch.empty(16, ny, nx, dtype=torch.float32, device=dev)
        st.step(x, dt, 3)
        st.step_out(x, dt, z)
        got.append((x.cpu(), z.cpu()))
    for x, z in got[1:]:
        assert torch.equal(x, got[0][0]) and torch.equal(z, got[0][1])
