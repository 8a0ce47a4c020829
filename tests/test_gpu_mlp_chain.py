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
