"""Whatever call a context's pinned block is first needed by (fields set, a read-out, a species, a
step), the results are the same; a context that has computed network gradients before takes it
up as well.
"""
import numpy as np
import pytest

from gpu_common import announce, have_gpu, jittered_kuhn, require_lib
from oracle import mlp
from oracle.constants import M_E, Q_E
from paper_2102_06248_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", ["fields", "read_out", "species", "step", "push", "rho", "gradient"])
def test_first_use(first):
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    F = require_lib()
    announce(f"first call: {first}")
    xyz, tets = jittered_kuhn(5, seed=1)[:2]
    x, u = inputs.beam_particles(500, 0.2, 0.2, 0.8, 2000.0, 5.0, M_E, 11)
    x[:, :2] += 0.5

    def run(warm):
        with F.Simulation(xyz, tets, device=0, preconditioner=F.FEPIC_PC_JACOBI, deterministic=1, diagnostics=1) as L:
            if warm == "fields":
                F.fepic_set_fields(L.ctx, e=np.zeros(L.sizes["n_edges"]))
            elif warm == "read_out":
                assert all(not np.any(a) for a in F.fepic_get_fields(L.ctx))
            elif warm == "rho":
                assert not np.any(F.fepic_get_rho(L.ctx, L.n_nodes))
            elif warm == "step":
                F.fepic_step(L.ctx, 1e-11)
            elif warm == "push":
                F.fepic_push_particles(L.ctx, 1e-11)
            elif warm == "gradient":
                F.fepic_ws_set_weights(L.ctx, mlp.flatten(mlp.init_params(1)).astype(np.float32))
                rng = np.random.default_rng(1)
                F.fepic_mlp_grad(L.ctx, rng.normal(size=(64, 4)).astype(np.float32), rng.normal(size=64).astype(np.float32))
            s = F.fepic_add_species(L.ctx, -Q_E, M_E, 1e6)
            F.fepic_upload_particles(L.ctx, s, x, u, ids=np.arange(len(x)))
            F.fepic_set_uniform_B(L.ctx, [0.0, 0.004, 0.02])
            st = [F.fepic_step(L.ctx, 1e-11) for _ in range(3)]
            p = F.fepic_get_particles(L.ctx, s)
            o = np.argsort(p["id"])
            return ([(a.n_crossings, a.n_particles) for a in st], *F.fepic_get_fields(L.ctx), *F.fepic_get_current(L.ctx),
                    p["x"][o], p["u"][o])

    a, b = run("species"), run(first)
    assert a[0] == b[0] and a[0][0][1] > 0
    for p, q in zip(a[1:], b[1:]):
        assert np.array_equal(p, q)
