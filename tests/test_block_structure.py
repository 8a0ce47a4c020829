"""Block form of the radial operators (Section 2.2: banded systems per Fourier
mode), on the oracle's own dense operators, for every N the library takes.

The substep solve cuts the rows into tiles of four aligned to the wall, with
the last eight rows as one block, and assumes that every operator is block
tridiagonal in that partition, that the couplings between blocks depend on
neither m nor k (only, close to the axis, on the parity), and that block
elimination without pivoting between blocks is accurate.
"""
import numpy as np
import pytest

from oracle import Oracle, Params


def edges(N):
    """First rows of the blocks (a shorter first tile stands for the padded one), then N."""
    pad = -N % 4
    return [max(4 * i - pad, 0) for i in range((N + pad - 8) // 4 + 1)] + [N]


def block_solve(A, b, e):
    nb = len(e) - 1
    blk = [slice(e[i], e[i + 1]) for i in range(nb)]
    inv, v = [], []
    for i in range(nb):
        D, r = A[blk[i], blk[i]], b[blk[i]]
        if i:
            D = D - A[blk[i], blk[i - 1]] @ inv[-1] @ A[blk[i - 1], blk[i]]
            r = r - A[blk[i], blk[i - 1]] @ v[-1]
        inv.append(np.linalg.inv(D))
        v.append(inv[-1] @ r)
    x = b.copy()
    x[blk[-1]] = v[-1]
    for i in range(nb - 2, -1, -1):
        x[blk[i]] = v[i] - inv[i] @ (A[blk[i], blk[i + 1]] @ x[blk[i + 1]])
    return x


@pytest.mark.parametrize("N", range(12, 65))
def test_operators_in_blocks(N):
    o = Oracle(Params(N=N, M=6, K=4, mp=1, alpha=1.3, Re=2500.0, dt=0.004))
    e = edges(N)
    block = np.searchsorted(e, np.arange(N), side="right") - 1
    off = np.abs(block[:, None] - block[None, :])
    couplings = {}
    rng = np.random.default_rng(N)
    for mu in (0, 1, 2, 5):
        for kap in (0.0, 3.9):
            L = o.lap(mu, [kap])[0]
            L[-1] = 0.0
            L[-1, -1] = 1.0
            assert not L[off > 1].any()
            # the couplings of one parity are the same for every m and k, and of
            # both parities but for entries with row + column <= 3
            c = np.where(off == 1, L, 0.0)
            assert np.array_equal(couplings.setdefault(mu % 2, c), c)
            for A in ([] if mu == 0 and kap == 0.0 else [L]) + [-2.0 * 2500.0 * o.helm(mu, [kap])[0]]:
                A = A.copy()
                A[-1] = 0.0
                A[-1, -1] = 1.0
                b = rng.standard_normal(N)
                x = np.linalg.solve(A, b)
                assert np.max(np.abs(block_solve(A, b, e) - x)) <= 1e-11 * np.max(np.abs(x))
    n = np.arange(N)
    far = n[:, None] + n[None, :] > 3
    assert np.array_equal(couplings[0][far], couplings[1][far])
