"""Theta stage on grids that take the 16-point kernel: every azimuthal length
it is built for, an axial length that 16 does not divide (the last tile is
ragged), the fewest workgroups it is chosen for and one fewer, with and
without the Coriolis force.

Tolerance: as the other FP64 transform checks, 1e-13 (rounding of two FFTs and
a product); in mixed precision the FP32 transforms' 2e-6 of the largest
coefficient (24-bit mantissa, two transforms of up to 192 x 96 points).
"""
import numpy as np
import pytest

from gpu_support import make_solver
from inputs import make_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,M,K,rot", [(64, M, 18, 0.0) for M in (2, 3, 4, 6, 8, 12, 16, 18, 24, 32, 36, 48, 64)] +
                         [(64, 12, 18, 0.3), (64, 16, 18, 0.3), (52, 6, 24, 0.0), (51, 6, 24, 0.0), (37, 12, 32, 0.0)] +
                         # the fewest workgroups in FP64 (144) and on lines of 72 in FP32 (192), and fewer
                         [(48, 6, 16, 0.0), (47, 6, 16, 0.0), (64, 24, 16, 0.0), (63, 24, 16, 0.0)])
def test_nonlinear_wide(N, M, K, rot, precision):
    import torch

    from oracle import Oracle, Params
    kw = dict(N=N, M=M, K=K, mp=1, alpha=1.1, Re=2000.0, dt=0.01)
    print("nonlinear", kw, precision, flush=True)
    s = make_solver(precision=precision, **kw)
    if rot:
        s.set_rotation(0.2, -0.1, rot)
    o = Oracle(Params(rotation=(0.2, -0.1, rot) if rot else (0.0, 0.0, 0.0), **kw))
    u = make_state(N, M, K, 1, 1.1, s.nodes(), 5e-2, 4.0, 4.0, 11)
    got = s.nonlinear(torch.from_numpy(u)).cpu().numpy()
    ref = o.nonlinear(u)
    assert np.max(np.abs(got - ref)) <= (2e-6 if precision else 1e-13) * np.max(np.abs(ref))
