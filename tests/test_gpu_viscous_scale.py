"""Steps whose Helmholtz shift Re / (c dt) is too large for a double: no
viscosity at all (Re = infinity, the wall values kept by the last row), and
Reynolds numbers, implicitness and step sizes whose quotient overflows.

The viscous terms are below the last place of 1/dt times the state, so a step
equals that with a shift of 1e100 or more that does not overflow.  Tolerance:
both solve the same systems up to the rounding of the shift, 1e-13 as the
other FP64 step checks.
"""
import numpy as np
import pytest

from gpu_support import make_solver
from inputs import make_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extreme,plain", [(dict(Re=float("inf")), dict(Re=1e100)), (dict(Re=1e306), dict(Re=1e100)),
                                           (dict(Re=1e300, dt=1e-9), dict(Re=1e100, dt=1e-9)),
                                           (dict(Re=2e3, c=1e-306), dict(Re=2e3, c=1e-100))])
@pytest.mark.parametrize("precision", [0, 1])
def test_step_without_viscosity(extreme, plain, precision):
    import torch
    print("step", extreme, plain, precision, flush=True)
    states = []
    for kw in (extreme, plain):
        s = make_solver(**dict(dict(N=21, M=6, K=6, mp=1, alpha=1.1, dt=0.01, precision=precision), **kw))
        u = make_state(21, 6, 6, 1, 1.1, s.nodes(), 1e-2, 4.0, 4.0, 7)
        s.set_state(torch.from_numpy(u))
        s.step(2)
        states.append(s.get_state().cpu().numpy())
    got, ref = states
    assert np.isfinite(got).all()
    assert np.max(np.abs(got - ref)) <= 1e-13 * np.max(np.abs(ref))
    assert np.max(np.abs(got - u)) > 1e-13  # (it did step)
