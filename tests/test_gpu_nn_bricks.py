"""Network kernels at the edges of their bricks, against the FP64 oracle.

Operands are BF16 values, so that a result differs from the oracle only by FP32
accumulation: 1e-4 of the output's rms (27 cin products of unit-scale terms, 27 cin
2^-24 < 2e-4 in the worst order, its square root in practice); with SiLU on load the
activation is rounded to BF16 on both sides and may differ by one unit: 1e-2.
"""
import numpy as np
import pytest
import torch

from oracle import nn_oracle as nn
from paper_2501_13046_amd import grtnn as gn
from test_gpu_nn import bf, cf, cl, silu_bf, to_dev
from test_gpu_nn import test_network_gradients as network_gradients

pytestmark = pytest.mark.gpu


# sides below, at and past bricks of 2 x 4 x 8, 2 x 2 x 16, 4 x 8 x 8 and 4 x 4 x 16 cells
# (from 256 bricks and channel tiles on the larger ones), slices of 8, 16 and 32
# channels, one and several of them, output channels that end inside a tile or a quad
@pytest.mark.parametrize("n,cin,cout,act", [(1, 8, 5, False), (2, 32, 16, True), (9, 64, 7, False), (12, 16, 4, False),
                                            (20, 24, 17, False), (16, 96, 20, False), (34, 16, 24, False),
                                            (36, 64, 48, False), (44, 8, 20, True), (40, 32, 18, False),
                                            (48, 32, 16, True), (48, 24, 3, False)])
def test_convolution_on_any_side(n, cin, cout, act):
    rng = np.random.default_rng(100 * n + cin + cout)
    x = bf(rng.standard_normal((cin, n, n, n)))
    W = bf(rng.standard_normal((cout, cin, 3, 3, 3)) * np.sqrt(2.0 / (27 * cin)))
    b = rng.uniform(-0.1, 0.1, cout).astype(np.float32).astype(np.float64)
    y = gn.conv3_forward(to_dev(cl(x), torch.bfloat16), to_dev(W.reshape(-1), torch.float32),
                         to_dev(b, torch.float32), n, cin, cout, act)
    ref = nn.conv3(torch.tensor(silu_bf(x) if act else x), torch.tensor(W), torch.tensor(b)).numpy()
    err = np.abs(cf(y.cpu().numpy(), n) - ref).max() / np.sqrt(np.mean(ref ** 2))
    print(f"n={n} {cin}->{cout} act={act}: max err / rms = {err:.2e}", flush=True)
    assert err < (1e-2 if act else 1e-4)


# cells past the grid in one or more directions, one and several bricks per block (from 257
# bricks and tile pairs on), tiles of one octet, output channels that end inside a tile
@pytest.mark.parametrize("n,cin,cout,act", [(1, 8, 5, False), (2, 16, 16, False), (7, 24, 8, True), (9, 16, 20, False),
                                            (20, 40, 12, False), (16, 24, 33, False), (34, 16, 4, False),
                                            (48, 8, 16, False), (40, 16, 24, True)])
def test_weight_gradient_on_any_side(n, cin, cout, act):
    rng = np.random.default_rng(10 * n + cin + cout)
    x = bf(rng.standard_normal((cin, n, n, n)))
    dy = np.zeros(((cout + 7) // 8 * 8, n, n, n))
    dy[:cout] = bf(rng.standard_normal((cout, n, n, n)))
    dW, db = gn.conv3_backward_weight(to_dev(cl(x), torch.bfloat16), to_dev(cl(dy), torch.bfloat16), n, cin,
                                      cout, act)
    _, rW, rb = nn.conv3_vjp(silu_bf(x) if act else x, np.zeros((cout, cin, 3, 3, 3)), np.zeros(cout), dy[:cout])
    eW = np.abs(dW.cpu().numpy().reshape(rW.shape) - rW).max() / np.sqrt(np.mean(rW ** 2))
    eb = np.abs(db.cpu().numpy() - rb).max() / np.sqrt(np.mean(rb ** 2))
    print(f"n={n} {cin}->{cout} act={act}: dW {eW:.2e} db {eb:.2e}", flush=True)
    assert eW < (1e-2 if act else 1e-4) and eb < 1e-4


# an odd coarse side: the upsampling's adjoint takes coarse cells in pairs along z
def test_network_gradients_on_an_odd_coarse_side():
    network_gradients(6, 2, (16, 32))


# bricks that overhang the grid read wrapped cells for the cells past it: an infinite
# activation there must not turn a gradient into NaN (0 * infinity)
@pytest.mark.parametrize("n", [7, 9, 12, 18, 20, 34])
def test_weight_gradient_of_infinite_activations(n):
    cin, cout = 8, 16
    rng = np.random.default_rng(n)
    x = bf(rng.standard_normal((cin, n, n, n)))
    dy = bf(rng.standard_normal((cout, n, n, n)))
    cells = {1: (0, 0, 0), 2: (n - 1, n - 1, n - 1), 3: (0, n // 2, n - 1)}
    for ci, w in cells.items():
        x[(ci,) + w] = np.inf
    dW, db = gn.conv3_backward_weight(to_dev(cl(x), torch.bfloat16), to_dev(cl(dy), torch.bfloat16), n, cin, cout,
                                      False)
    dW = dW.cpu().numpy().reshape(cout, cin, 3, 3, 3)
    for ci, w in cells.items():
        for t in np.ndindex(3, 3, 3):  # dW[t] = sum_v dy[v] x[v + t - 1]
            v = tuple((w[a] - t[a] + 1) % n for a in range(3))
            np.testing.assert_array_equal(dW[(slice(None), ci) + t], np.sign(dy[(slice(None),) + v]) * np.inf)
    finite = [ci for ci in range(cin) if ci not in cells]
    assert np.isfinite(dW[:, finite]).all() and np.isfinite(db.cpu().numpy()).all()
