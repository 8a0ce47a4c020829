"""The diagnostics' per-mode sums, their reduction and the corrector
difference at the edges of their forms: fewest modes, more than 64 axial
modes per m (a second round of lanes), more than 16 m (a second round of
waves), 64 rows, and fewer entries per m than the corrector difference has
threads.

Tolerances: E, D and the flux are sums of positive terms or short dot
products in FP64 over at most 64 x 127 x 64 entries, 1e-12 relative; g and the
divergence as elsewhere 1e-12 of the largest entry; the corrector difference
1e-6 relative (its predictor and corrector agree to several digits).
"""
import numpy as np
import pytest

from gpu_support import make_solver
from inputs import make_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,K", [(13, 2, 2), (24, 18, 36), (64, 3, 64), (33, 32, 4)])
def test_diagnostics_and_corrector_difference(N, M, K):
    import torch

    from oracle import Oracle, Params
    from oracle.timestep import pc_difference
    kw = dict(N=N, M=M, K=K, mp=1, alpha=1.1, Re=1800.0, dt=0.004)
    print("diagnostics", kw, flush=True)
    s, o = make_solver(**kw), Oracle(Params(**kw))
    u = make_state(N, M, K, 1, 1.1, s.nodes(), 1e-2, 4.0, 4.0, 17)
    u[2, M - 1, 1] += 0.01  # a wall value in a far mode, seen by g and by the energies
    s.set_state(torch.from_numpy(u))
    d, ref = s.diagnostics(check=False), o.diagnostics(u)
    for k in ("E", "D", "flux", "tau_w"):  # (I takes the last step's beta: none yet)
        assert abs(d[k] - ref[k]) <= 1e-12 * abs(ref[k]), k
    g, dm = o.boundary_and_divergence(u)
    scale = np.max(np.abs(u))
    assert abs(d["g_norm"] - g) <= 1e-12 * scale * max(1.0, g / scale)
    assert abs(d["div_max"] - dm) <= 1e-12 * scale * max(1.0, dm / scale)
    s.step(1)
    u1, up = o.step_pc(u)
    ref = pc_difference(o, u1, up)
    assert abs(s.pc_difference() - ref) <= 1e-6 * ref
