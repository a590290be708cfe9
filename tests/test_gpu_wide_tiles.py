"""FP64 grids that take 31x10 tiles: those whose 15x10 tiles just exceed what runs at once (the
second round of a few tiles made them up to 12% slower than wide tiles), and long ones of 31
columns.  The sizes on both sides of the rule, whole tiles and remainders, both point updates,
against the oracle."""
import numpy as np
import pytest

from paper_2605_12915_amd import inputs as I

pytestmark = pytest.mark.gpu


# 513 narrow tiles or more and 256 wide ones or fewer; 31 columns, more than 384 wide tiles
@pytest.mark.parametrize("scheme", ["tai", "rb"])
@pytest.mark.parametrize("nx,ny,wide", [(31, 1700, False), (31, 1701, True), (31, 2560, True), (31, 2561, False), (31, 3840, False),
                                        (31, 3841, True), (32, 3841, False), (61, 1093, True), (248, 320, True), (249, 320, False),
                                        (307, 249, True), (310, 240, False)])
def test_step_vs_oracle(orc, nx, ny, wide, scheme):
    import torch

    from paper_2605_12915_amd.stepper import Stepper
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    P = I.random_smooth(nx, ny, seed=nx + 7 * ny, amp=0.1, vel=(0.35, -0.25))
    s0, n = P.state(), 2
    dt = P.dt_for_cfl(0.19 if scheme == "rb" else 0.4)
    print("wide tiles", nx, ny, scheme, flush=True)
    st = Stepper(nx, ny, P.h, P.gamma, scheme=scheme, device=dev, check_errors=True)
    assert ("31, 10, 512" in st.dominant_kernel()) == wide, st.dominant_kernel()
    x = torch.from_numpy(s0).to(dev)
    st.step(x, dt, n)
    want = orc.run(s0, P.h, P.gamma, dt, n, scheme=1 if scheme == "rb" else 0)
    err = np.abs(x.cpu().numpy() - want).max(axis=(1, 2)) / np.abs(want).max(axis=(1, 2))
    assert err.max() <= 1e-12, (st.dominant_kernel(), err)
