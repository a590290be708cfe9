"""The diagnostics' totals on large grids: a thread's chain of additions grows with the grid,
the rounding errors of the totals do not."""
import math

import pytest

pytestmark = pytest.mark.gpu


def _uniform(torch, dev, n, W, gamma=1.4):
    r, u, v, p = W
    vals = [r, r * u, r * v, p / (gamma - 1) + 0.5 * r * (u * u + v * v)] + list(W) * 3
    x = torch.empty((16, n, n), dtype=torch.float64, device=dev)
    for k in range(16):
        x[k].fill_(vals[k])
    return x, vals


def test_totals_of_a_uniform_state():
    """8192^2 cells of h = 1/8192 (a power of two): every total is the value itself.  Bound: a
    thread's own sum to one rounding, then 20 additions up to the total (6 + 3 in a block, 2 + 6
    + 3 over the blocks) of one rounding each."""
    import torch

    from paper_2605_12915_amd.stepper import Stepper
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev, n = torch.device("cuda:0"), 8192
    st = Stepper(n, n, 1.0 / n, 1.4, device=dev)
    for W in ((1.1, 0.7 / 1.1, -0.37 / 1.1, 0.9), (0.1, 7.0, 3.0, 0.04)):
        x, vals = _uniform(torch, dev, n, W)
        d = st.diagnostics(x)
        for name, want in zip(("mass", "momx", "momy", "energy"), vals):
            err = abs(d[name] - want) / abs(want)
            print(name, want, "relative error", err, flush=True)
            assert err <= 22 * 2.0 ** -53
        del x


def test_totals_not_finite():
    """A total with an infinite summand is infinite, one with a NaN is NaN, the others stay."""
    import torch

    from paper_2605_12915_amd.stepper import Stepper
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev, n = torch.device("cuda:0"), 600
    st = Stepper(n, n, 1.0 / n, 1.4, device=dev)
    x, vals = _uniform(torch, dev, n, (1.1, 0.5, -0.3, 0.9))
    x[0, 3, 5] = math.inf
    x[1, 599, 599] = -math.inf
    x[2, 0, 0] = math.nan
    d = st.diagnostics(x)
    assert d["mass"] == math.inf and d["momx"] == -math.inf and math.isnan(d["momy"])
    assert abs(d["energy"] - vals[3]) <= 1e-14 * vals[3]
