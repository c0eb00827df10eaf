"""fepic_mlp_grad and fepic_mlp_grad_noalloc give the same bits, gradient and loss: one block of
rows, several, one per workgroup of the grid, and several per workgroup.
"""
import numpy as np
import pytest

from gpu_common import announce, have_gpu, require_lib
from oracle import mlp
from paper_2102_06248_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 777, 20_000, 32_768, 65_536])
def test_same_bits(n):
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    F = require_lib()
    import torch

    announce(f"mlp gradient, both entry points, {n} rows")
    rng = np.random.default_rng(n)
    X, t = rng.normal(size=(n, 4)).astype(np.float32), rng.normal(size=n).astype(np.float32)
    xyz, tets = inputs.kuhn_cube(2)
    with F.Simulation(xyz, tets, device=0) as s:
        F.fepic_ws_set_weights(s.ctx, mlp.flatten(mlp.init_params(n)).astype(np.float32))
        loss, grad = F.fepic_mlp_grad(s.ctx, X, t)
        dX, dt, dg, dl = (torch.from_numpy(a).to("cuda") for a in (X, t, np.zeros(F.FEPIC_MLP_N_PARAMS, np.float32),
                                                                  np.zeros(1)))
        torch.cuda.synchronize()
        F.fepic_mlp_grad_noalloc(s.ctx, n, dX.data_ptr(), dt.data_ptr(), dg.data_ptr(), dl.data_ptr())
        torch.cuda.synchronize()
    assert np.array_equal(dg.cpu().numpy().view(np.uint32), grad.view(np.uint32))
    assert dl.cpu().item() == loss
