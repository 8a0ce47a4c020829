"""Inverse diagonal blocks of the radial operators as the library stores them
(its images), against the same block elimination in extended precision.

Every operator of a small context is compared, Helmholtz and pressure, at
radial sizes with the least and the most padding rows.  The images are found
in the solver's workspace by the first one's entries.

Tolerance, relative to the largest entry of a block: storage in double gives
1.1e-16; entries of the operators that are rounded once or twice (a fused or
a separate multiply and add in d2 + d1 / r) change a block by up to 1.2e-15,
from the elimination below on both; the scale of the Helmholtz systems is
within four units in the last place of Re / c, 0.9e-15.  2.2e-15 in all.  The
elimination in plain double precision is 2.7e-15 or more off (asserted, so
that the bound is known to see it).
"""
import numpy as np
import pytest

from gpu_support import make_solver, oracle_nodes

LD = np.longdouble
BOUND = 2.2e-15


def tiles(N):
    return ((N - 5) // 4 + 1) // 2 * 2


def operator(N, tab, mu, kap):
    """Rows of d2/dr2 + (1/r) d/dr - (mu^2/r^2 + kap^2), the wall row that of the identity, in double."""
    _, _, d1, d2, s0 = tab
    r = oracle_nodes(N)
    A = np.zeros((N, N))
    for n in range(N - 1):
        A[n, s0[n]:s0[n] + 9] = d2[mu % 2, n] + 1.0 / r[n] * d1[mu % 2, n]
        ri = 1.0 / r[n]
        A[n, n] -= mu * mu * ri * ri + kap * kap
    A[-1, -1] = 1.0
    return A


def inverse(D, T):
    n = len(D)
    m, v = D.copy(), np.eye(n, dtype=T)
    for q in range(n):
        p = m[q, q]
        m[q], v[q] = m[q] / p, v[q] / p
        for r in range(n):
            if r != q:
                f = m[r, q]
                m[r], v[r] = m[r] - f * m[q], v[r] - f * v[q]
    return v


def blocks(A, shift, T):
    """The inverse diagonal blocks of the elimination in precision T: tiles of four rows, then the last eight."""
    N = len(A)
    nt = tiles(N)
    pad = 4 * nt + 8 - N
    B = np.eye(N + pad, dtype=T)
    B[pad:, pad:] = A.astype(T)
    i = np.arange(pad, pad + N - 1)
    B[i, i] -= T(shift)
    out = []
    for t in range(nt + 1):
        a, b = slice(4 * t - 4, 4 * t), slice(4 * t, 4 * t + (4 if t < nt else 8))
        D = B[b, b].copy()
        if t:
            D = D - B[b, a] @ (out[-1] @ B[a, b])
        out.append(inverse(D, T))
    return out


def stored(img, nt):
    """Blocks of one image: element [i][k] of tiles 2p, 2p+1 at 32 p + 2 (4 k + i) + 0, 1."""
    t = [img[32 * (q // 2) + q % 2:][:32:2].reshape(4, 4).T for q in range(nt + 4)]
    return t[:nt] + [np.block([[t[nt], t[nt + 1]], [t[nt + 2], t[nt + 3]]])]


def distance(got, ref):
    return max(float(np.max(np.abs(g - r)) / np.max(np.abs(r))) for g, r in zip(got, ref))


def images(s, first, count, nt):
    """The library's images: `count` in a row, found by the blocks of the first."""
    off = s._ws_ptr - s.ws.data_ptr()
    w = s.ws[off:off + s.ws_bytes // 8 * 8].cpu().numpy().view(np.float64)
    size = 16 * (nt + 4)
    want = float(first[0][0, 0])
    with np.errstate(invalid="ignore"):
        at = np.nonzero(np.abs(w - want) <= 1e-9 * abs(want))[0]
    for i in at:
        if i + count * size <= len(w):
            got = stored(w[i:i + size], nt)
            if np.isfinite(w[i:i + size]).all() and distance(got, first) < 1e-9:
                return w[i:i + count * size].reshape(count, size)
    raise AssertionError("no image in the workspace")


@pytest.mark.gpu
@pytest.mark.parametrize("N,mp,Re,dt", [(64, 1, 5300.0, 0.002), (57, 2, 2400.0, 0.01), (41, 3, 2400.0, 0.005),
                                        (24, 1, 2400.0, 0.01), (12, 1, 1500.0, 0.02)])
def test_images_are_right_to_a_unit_in_the_last_place(N, mp, Re, dt):
    import paper_1705_03838_amd as opf
    M, K, alpha, c = 8, 8, 1.25, 0.5
    print("images", N, mp, Re, dt, flush=True)
    s = make_solver(N=N, M=M, K=K, mp=mp, alpha=alpha, Re=Re, dt=dt, c=c)
    tab = opf.host_tables(N=N, M=M, K=K)
    assert np.array_equal(tab[0], oracle_nodes(N))
    nt, MU, shift = tiles(N), mp * (M - 1) + 2, Re / c / dt
    ops = [(mu, k, shift) for k in range(K) for mu in range(MU)] + [(mp * m, k, 0.0) for k in range(K) for m in range(M)]
    first = blocks(operator(N, tab, 0, 0.0), shift, LD)
    img = images(s, first, len(ops), nt)
    worst, plain = 0.0, 0.0
    for (mu, k, sh), g in zip(ops, img):
        if mu == 0 and k == 0 and sh == 0.0:
            assert not g.any()  # (0,0) has no pressure
            continue
        A = operator(N, tab, mu, alpha * k)
        ref = blocks(A, sh, LD)
        worst = max(worst, distance(stored(g, nt), ref))
        plain = max(plain, distance(blocks(A, sh, np.float64), ref))
    print("worst %.2e, plain double %.2e" % (worst, plain), flush=True)
    assert plain > BOUND
    assert worst <= BOUND


@pytest.mark.gpu
def test_scale_is_not_moved_without_need():
    """1/dt a power of two: Re / c times 1/dt is exact, so the shift is that of
    Re / c itself.  At Re = 1e30 the blocks are those of -shift to 1e-20, and
    their diagonal shows it to a rounding (half a unit in the last place of the
    reciprocal, 1.1e-16)."""
    Re, dt, c = 1e30, 2.0 ** -7, 0.5
    s = make_solver(N=24, M=4, K=4, mp=1, alpha=1.25, Re=Re, dt=dt, c=c)
    nt, shift = tiles(24), Re / c / dt
    first = [-np.eye(4) / shift] * nt + [np.diag([-1.0 / shift] * 7 + [1.0])]
    img = images(s, first, 1, nt)[0]
    for got, ref in zip(stored(img, nt), first):
        assert np.max(np.abs(np.diag(got) / np.diag(ref) - 1.0)) <= 1.2e-16 * 2
