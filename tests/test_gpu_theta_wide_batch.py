"""Grids on both sides of the rule for the 16-point theta kernel.

Its batched form gives members bitwise equal to single runs (one path for both:
the rule looks at one member's grid), in both precisions.  The tuner times no
tz where the kernel does not use it, which also shows the path that a grid
takes: by its axial points, a ragged last tile counted as the part that is
used, and on lines of 144 not where a second or a third workgroup per compute
unit has only begun.

Tolerance of the nonlinear term: as the other transform checks, 1e-13 in FP64
and 2e-6 in mixed precision.
"""
import numpy as np
import pytest

from gpu_support import make_ensemble, make_solver, oracle_nodes
from inputs import make_state

pytestmark = pytest.mark.gpu

# (N, M, K, precision), tiles of 16 axial points in brackets.  Wide: FP64 on lines
# of 18 (129, near the fewest) and 36 (192), on axial lines of 54; mixed, lines of
# 72 (199, near the fewest) and 18 (288).  Not: 126 tiles, 156 workgroups that
# are 117 tiles, lines of 144 at 144, 288 and 576, mixed at 192 and 258, and a
# small grid.
GRIDS = [(43, 6, 16, 0), (32, 12, 32, 0), (60, 8, 18, 0), (59, 24, 18, 1), (48, 6, 32, 1),
         (42, 6, 16, 0), (52, 18, 12, 0), (24, 48, 32, 0), (48, 48, 32, 0), (64, 48, 48, 0), (64, 24, 16, 1), (43, 6, 32, 1),
         (21, 6, 4, 0)]
MEM = [dict(N=N, M=M, K=K, precision=p) for N, M, K, p in GRIDS]
WIDE = [True] * 5 + [False] * 8


def members():
    return [dict(m, mp=1, alpha=1.1 + 0.1 * i + 0.03 * j, Re=1900.0 + 50 * j, dt=0.002) for i, m in enumerate(MEM) for j in range(2)]


def test_members_equal_single_runs():
    import torch
    mem = members()
    e = make_ensemble(mem)
    states = []
    for i, kw in enumerate(mem):
        st = make_state(kw["N"], kw["M"], kw["K"], 1, kw["alpha"], oracle_nodes(kw["N"]), 1e-2, 4.0, 4.0, 60 + i)
        states.append(st)
        e.members[i].set_state(torch.from_numpy(st))
    e.step(3)
    for i, kw in enumerate(mem):
        print("member", kw, flush=True)
        s = make_solver(**kw)
        s.set_state(torch.from_numpy(states[i]))
        s.step(3)
        assert np.array_equal(e.members[i].get_state().cpu().numpy(), s.get_state().cpu().numpy()), kw
    e.close()


def test_tuner_times_no_tile_that_is_not_used():
    e = make_ensemble(members())
    rep = e.tune(2)
    assert len(rep["classes"]) == len(MEM)
    for c, wide in zip(rep["classes"], WIDE):
        tz = {x["tz"] for x in c["candidates"]}
        assert len(tz) == 1 if wide else len(tz) > 1, c
    e.close()


@pytest.mark.parametrize("N,M,K,precision", [(43, 6, 16, 0), (42, 6, 16, 0), (56, 48, 32, 0), (52, 48, 32, 0), (59, 24, 18, 1),
                                             (58, 24, 18, 1)] + [(52, M, 36, 1) for M in (2, 3, 4, 6, 8, 12, 16, 18)])
def test_nonlinear_term(N, M, K, precision):
    import torch

    from oracle import Oracle, Params
    kw = dict(N=N, M=M, K=K, mp=1, alpha=1.1, Re=2000.0, dt=0.01)
    print("nonlinear", kw, precision, flush=True)
    s = make_solver(precision=precision, **kw)
    u = make_state(N, M, K, 1, 1.1, s.nodes(), 5e-2, 4.0, 4.0, 12)
    got = s.nonlinear(torch.from_numpy(u)).cpu().numpy()
    ref = Oracle(Params(**kw)).nonlinear(u)
    assert np.max(np.abs(got - ref)) <= (2e-6 if precision else 1e-13) * np.max(np.abs(ref))
