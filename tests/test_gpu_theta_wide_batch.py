"""Classes of an ensemble whose theta stage takes the 16-point kernel.

The batched form of that kernel gives members bitwise equal to single runs (one
path for both: the rule that chooses it looks at one member's grid), in both
precisions, at the fewest workgroups it is chosen for and at an axial length
that 16 does not divide, beside a class below the rule.  The tuner times no tz
where the kernel does not use it.
"""
import numpy as np
import pytest

from gpu_support import make_ensemble, make_solver, oracle_nodes
from inputs import make_state

pytestmark = pytest.mark.gpu

# FP64: 144 workgroups (the fewest), 192, and 240 on axial lines of 54; mixed:
# 192 on azimuthal lines of 72 (the fewest), 288 on lines of 18.  The last below both.
MEM = [dict(N=48, M=6, K=16, precision=0), dict(N=32, M=12, K=32, precision=0), dict(N=60, M=8, K=18, precision=0),
       dict(N=64, M=24, K=16, precision=1), dict(N=48, M=6, K=32, precision=1), dict(N=21, M=6, K=4, precision=0)]
WIDE = [True] * 5 + [False]


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
