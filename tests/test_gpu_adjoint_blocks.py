"""The adjoint's increment kernel completes blocks of 16 x 8 node-cells by itself: grids smaller
than a block's window (its node-cells wrap onto themselves), whole blocks, and one node-cell
more or less in each direction, both point updates, by the dot-product identity
<lambda, J v> = <J^T lambda, v> with J v from the oracle's complex step."""
import numpy as np
import pytest

from paper_2605_12915_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["tai", "rb"])
@pytest.mark.parametrize("nx,ny", [(4, 4), (5, 9), (16, 8), (17, 7), (15, 9), (32, 24), (33, 25), (48, 4), (4, 48)])
def test_transpose(orc, nx, ny, scheme):
    import torch

    from paper_2605_12915_amd.stepper import Stepper
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    P = I.random_smooth(nx, ny, seed=3 * nx + ny, amp=0.08, vel=(0.3, -0.2), kmax=1)
    s0, dt = P.state(), P.dt_for_cfl(0.19 if scheme == "rb" else 0.35)
    rng = np.random.default_rng(nx * 100 + ny)
    v, lam = rng.normal(size=s0.shape), rng.normal(size=s0.shape)
    _, Jv = orc.step_jvp(s0, v, P.h, P.gamma, dt, scheme=1 if scheme == "rb" else 0)
    print("adjoint block", nx, ny, scheme, flush=True)
    st = Stepper(nx, ny, P.h, P.gamma, scheme=scheme, device=dev)
    x, c = torch.from_numpy(s0).to(dev), torch.from_numpy(lam).to(dev)
    g = st.adjoint(x, c, dt)
    # every output is written whatever was in the buffer, and the input cotangent is left alone
    h = st.adjoint(x, c, dt, out=torch.full_like(x, 7.0))
    assert float((g - h).abs().max()) <= 1e-12 * float(g.abs().max())
    assert np.array_equal(c.cpu().numpy(), lam)
    gap = abs(float((g.cpu().numpy() * v).sum()) - float((lam * Jv).sum()))
    assert gap <= 1e-11 * np.linalg.norm(lam) * np.linalg.norm(Jv)
