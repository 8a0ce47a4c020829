"""The residual layers as chains of one workgroup per 32 rows, the merged
gradient launches and the tiled Adam step, at the edges of their forms: one
wave to sixteen (widths 32 to 512), widths that end inside a 256-wide (224)
or 128-wide (288, 480) chunk, one layer and the most (8), a single row, ragged
row tiles, a row count whose weight gradients are split over K (1100) and one
whose products take the 128 x 128 tiles (512 x 512 x 4096).

Tolerance: 1e-2 relative (norm-wise) against the bfloat16 oracle.  One
bfloat16 flip (2^-8) in a few percent of the entries per layer is below 3e-3
for three layers; eight layers add up to sqrt(8 / 3) of that, 5e-3.  The FP32
accumulation over at most 4096 products adds 4096 2^-24 = 2.4e-4.
"""
import numpy as np
import pytest

from test_gpu_mlp import check_grads, make_net, nrel, rows, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width, layers, n", [
    (32, 1, 1), (64, 8, 33), (224, 2, 64), (256, 4, 150), (256, 1, 1100), (288, 2, 40), (480, 1, 32), (512, 8, 65),
    (512, 1, 4096)])
def test_gradients_and_step_match_bf16_oracle(torch_cuda, width, layers, n):  # noqa: F811
    from oracle.mlp import adam, backward, forward, loss, unflatten
    s, net, p = make_net(torch_cuda, width=width, layers=layers, max_rows=n, lr=1e-2)
    rng = np.random.default_rng(width + layers + n)
    x, t = rows(rng, n, net.din), rows(rng, n, net.dout)
    xd, td = torch_cuda.from_numpy(x), torch_cuda.from_numpy(t)
    x64, t64 = x.astype(np.float64), t.astype(np.float64)
    say("mlp chain", width, layers, n)
    y, cache = forward(p, x64, layers, bf16=True)
    assert nrel(net.forward(xd).cpu().numpy().astype(np.float64), y) <= 1e-2
    lg, g = net.gradient(xd, td)
    assert abs(lg - loss(y, t64)) <= 1e-3 * loss(y, t64)
    check_grads(g, backward(p, cache, y, t64, layers, bf16=True), layers)
    # a step, and the bfloat16 weight copies that follow it
    p0 = net.get_params().astype(np.float64)
    net.train(xd, td, batch=n, epochs=1)
    p1 = net.get_params().astype(np.float64)
    ref, _, _ = adam(p0, g.astype(np.float64), np.zeros_like(p0), np.zeros_like(p0), 1, lr=1e-2)
    assert np.max(np.abs(p1 - ref)) <= 1e-6
    q = unflatten(p1, net.din, width, layers, net.dout)
    y, cache = forward(q, x64, layers, bf16=True)
    assert nrel(net.forward(xd).cpu().numpy().astype(np.float64), y) <= 1e-2
    _, g = net.gradient(xd, td)
    check_grads(g, backward(q, cache, y, t64, layers, bf16=True), layers)


@pytest.mark.parametrize("N, M, K, rank, batch", [
    (24, 2, 2, 1, 1),     # fewest rows; output columns end half way through a 64-wide tile
    (24, 12, 6, 3, 9),    # 132 rows: a second chunk of column sums; two pairs per wave, a last pass of one pair
    (48, 3, 4, 16, 13),   # the benchmark's profile length and rank: four passes, the last of one pair
    (64, 2, 3, 16, 5),    # the most gradient entries per thread
    (64, 2, 3, 13, 6)])   # the same with a rank that does not divide 256
def test_pair_gradient_edges(torch_cuda, N, M, K, rank, batch):  # noqa: F811
    """The loss head and the one reading of dL/dY that follows it.  Loss: 1e-5
    against the oracle's head on the device's own rows (FP32 sums over 3 N
    entries, 192 2^-24); gradients as above."""
    import paper_1705_03838_amd as opf
    from gpu_support import make_solver
    from oracle.mlp import backprop, feature_rows, flatten, forward, head, init_params, unflatten
    s = make_solver(N=N, M=M, K=K, mp=1, alpha=0.9, Re=1500.0, dt=0.005)
    net = opf.Mlp(s, width=64, layers=2, rank=rank)
    flat = flatten(init_params(net.din, 64, 2, net.dout, seed=N + rank), 2).astype(np.float32)
    net.set_params(flat)
    p = unflatten(flat.astype(np.float64), net.din, 64, 2, net.dout)
    rng = np.random.default_rng(rank + batch)
    pairs = rng.standard_normal((4, 2) + s.shape) + 1j * rng.standard_normal((4, 2) + s.shape)
    idx = rng.integers(0, 4, batch).astype(np.int32)
    say("pair gradient", N, M, K, rank, batch)
    lg, g = net.pair_gradient(torch_cuda.from_numpy(pairs), idx)
    X = feature_rows(M, K, 1, 0.9)
    rows_dev = net.forward(torch_cuda.from_numpy(X.astype(np.float32))).cpu().numpy().astype(np.float64)
    ldev, _ = head(rows_dev, pairs[idx], rank)
    assert abs(lg - ldev) <= 1e-5 * ldev
    F, cache = forward(p, X, 2, bf16=True)
    _, dF = head(F.astype(np.float32).astype(np.float64), pairs[idx], rank)
    check_grads(g, backprop(p, cache, dF, 2, bf16=True), 2)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_set_params_refuses_non_finite_values(torch_cuda, bad):  # noqa: F811
    """Wherever the value stands in the blocks of the test, and without a
    change to the parameters that are there; the largest finite value passes."""
    import paper_1705_03838_amd as opf
    s, net, _ = make_net(torch_cuda)
    p0 = net.get_params()
    for i in (0, 4095, 4096, net.n_params - 1):
        q = p0.copy()
        q[i] = bad
        with pytest.raises(opf.OpfError):
            net.set_params(q)
    assert np.array_equal(net.get_params(), p0)
    q = p0.copy()
    q[4096] = np.finfo(np.float32).max
    net.set_params(q)
    assert np.array_equal(net.get_params(), q)
