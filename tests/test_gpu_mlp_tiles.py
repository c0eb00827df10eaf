"""The minibatch gradient at the edges of its tiles (128 rows, four waves of 32, halves of
16) and of its grid (256 workgroups, one tile each before they loop), against the oracle's
formulas evaluated in FP64 with the operands that the kernels round to BF16 (the first
layer's activations, W2 and dZ2) rounded the same way: without that, one unit of one row
whose pre-activation lies within BF16's rounding of zero decides the comparison (it did at
17 rows: |z2| = 3e-4).

What is left is FP32 arithmetic: sums of n terms (2^-24 each, taken as they come: 1e-5 of
the norm at these sizes) and the values that FP32 rounding moves across a BF16 boundary
(a share 2^-24 / 2^-9 of them, by 2^-9 each: 2^-9 sqrt(2^-15) = 1e-5 of the norm); the
bound is ten times their sum.
"""
import numpy as np
import pytest
import torch

from gpu_common import announce, have_gpu, require_lib
from oracle import mlp
from paper_2102_06248_amd import inputs

pytestmark = pytest.mark.gpu


def _bf16(a):
    return torch.as_tensor(a, dtype=torch.float32).bfloat16().double().numpy()


def _reference(p, X, t):
    W1, b1, W2, b2, W3, b3 = (p[k] for k in ("W1", "b1", "W2", "b2", "W3", "b3"))
    z1 = X @ W1.T + b1
    h1, w2 = _bf16(np.maximum(z1, 0.0)), _bf16(W2)
    z2 = h1 @ w2.T + b2
    h2 = np.maximum(z2, 0.0)
    err = h2 @ W3[0] + b3[0] - t
    dy = 2.0 * err / len(t)
    dz2 = dy[:, None] * W3[0] * (z2 > 0)
    dz1 = (_bf16(dz2) @ w2) * (z1 > 0)
    return np.mean(err ** 2), {"W1": dz1.T @ X, "b1": dz1.sum(0), "W2": _bf16(dz2).T @ h1, "b2": dz2.sum(0),
                               "W3": (dy @ h2)[None], "b3": np.array([dy.sum()])}


@pytest.mark.parametrize("n", [1, 15, 17, 127, 129, 32768, 32769, 65536 + 31])
def test_gradient_at_tile_and_grid_edges(n):
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    F = require_lib()
    announce(f"mlp gradient, {n} rows")
    rng = np.random.default_rng(n)
    p = mlp.init_params(n)
    for k, shape in (("b1", 64), ("b2", 64), ("b3", 1)):
        p[k] = rng.normal(size=shape) * 0.2
    p["W3"] = rng.normal(size=(1, 64)) * 0.3
    X = rng.normal(size=(n, 4)).astype(np.float32)
    t = rng.normal(size=n).astype(np.float32)
    xyz, tets = inputs.kuhn_cube(2)
    with F.Simulation(xyz, tets, device=0) as s:
        F.fepic_ws_set_weights(s.ctx, mlp.flatten(p).astype(np.float32))
        p = mlp.unflatten(F.fepic_ws_get_weights(s.ctx).astype(np.float64))
        loss, g = F.fepic_mlp_grad(s.ctx, X, t)
    ref_loss, ref = _reference(p, X.astype(np.float64), t.astype(np.float64))
    assert abs(loss - ref_loss) <= 2e-4 * ref_loss
    g = mlp.unflatten(g.astype(np.float64))
    for name, _ in mlp.SHAPES:
        # b3's terms cancel over the rows: held to the sum of their magnitudes, |dy| <= 2 rms / n each
        scale = max(np.linalg.norm(ref[name]), 2.0 * np.sqrt(ref_loss) if name == "b3" else 0.0)
        assert np.linalg.norm(g[name] - ref[name]) <= 2e-4 * scale, name
