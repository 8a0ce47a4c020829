"""Substep solve at the edges of its row tiles: each number of tiles with the
least and the most padding, one wave layout and the other (up to 32 rows both
modes of a wave lie side by side), and workgroups whose last waves have no m.

Tolerance: both sides solve the same systems to rounding; the pressure
operator's condition (~1/h^2 at the wall) sets 1e-11, as in test_gpu_parity.
"""
import numpy as np
import pytest

from gpu_support import make_solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,K,mp", [(N, 3, 4, 1 + N % 3) for N in
                                      (12, 16, 17, 24, 25, 31, 32, 33, 40, 41, 49, 56, 57, 63, 64)] +
                         [(20, 18, 16, 1), (36, 18, 16, 1), (36, 9 * 2, 16, 2)])
def test_substep_at_tile_edges(N, M, K, mp):
    import torch

    import paper_1705_03838_amd as opf
    from oracle import Oracle, Params
    from oracle.spectral import to_pm
    kw = dict(N=N, M=M, K=K, mp=mp, alpha=1.2, Re=2000.0, dt=0.01)
    print("substep", kw, flush=True)
    s = make_solver(**kw)
    o = Oracle(Params(**kw))
    rng = np.random.default_rng(N)
    R = rng.standard_normal((3, M, 2 * K - 1, N)) + 1j * rng.standard_normal((3, M, 2 * K - 1, N))
    R[:, 0, :K - 1] = np.conj(R[:, 0, :K - 1:-1])  # a real right-hand side field
    R[:, 0, K - 1] = R[:, 0, K - 1].real
    u, p = s.radial_solve(opf.OPF_SOLVE_RAW, torch.from_numpy(R), want_pressure=True)
    uref, pref = o.solve(to_pm(R), want_pressure=True)
    pref[0, K - 1] = 0  # (0,0) has no pressure
    assert np.max(np.abs(u.cpu().numpy() - uref)) <= 1e-11 * np.max(np.abs(uref))
    assert np.max(np.abs(p.cpu().numpy() - pref)) <= 1e-11 * np.max(np.abs(pref))
