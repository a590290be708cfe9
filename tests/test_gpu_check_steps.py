"""AF_CHECK over more steps than are read back together: the status is that of the first
step that failed, the state returns to the call's input, and nothing of the failed call
is left for the next one."""
import math

import numpy as np
import pytest

from tests.test_gpu_parity import _converging, _oracle_statuses

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("r0,low,high", [(0.494, 1, 15), (0.46, 16, 40)])
def test_first_failing_step(orc, precision, r0, low, high):
    import torch

    from paper_2605_12915_amd._lib import AF_ERR_ACOUSTIC_CFL, AfError
    from paper_2605_12915_amd.stepper import Stepper, to_perturbation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    P = _converging()
    s0, dt = P.state(), r0 * P.h / math.sqrt(1.4)
    sts = _oracle_statuses(orc, P, s0, dt, 45)
    first = next(k for k, s in enumerate(sts) if s)
    print("first failing step", first, sts, flush=True)
    assert low <= first <= high and sts[first] == 1
    st = Stepper(P.nx, P.ny, P.h, P.gamma, precision=precision, bg=P.bg, device=dev, check_errors=True)
    h0 = s0 if precision == "f64" else to_perturbation(s0, P.bg, P.gamma)
    for n in (first + 1, first + 2, 45):
        x = torch.from_numpy(h0).to(dev)
        with pytest.raises(AfError) as e:
            st.step(x, dt, n)
        assert e.value.code == AF_ERR_ACOUSTIC_CFL, n
        assert np.array_equal(x.cpu().numpy(), h0), n
        st.step(x, dt, first)                       # the good steps pass on the same context
        plain = Stepper(P.nx, P.ny, P.h, P.gamma, precision=precision, bg=P.bg, device=dev)
        y = torch.from_numpy(h0).to(dev)
        plain.step(y, dt, first)
        assert torch.equal(x, y)
