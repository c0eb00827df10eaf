"""Solves in one launch (every row block a resident workgroup) where they can go wrong: one
partial block, a few, the most that one workgroup per CU holds and the first mesh past it
(Jacobi: iterations launched one by one; auxiliary space: two row blocks per workgroup, then
one by one), nodes of more edges than one chunk of incidences, far levels, several solves
through the same exchange words, the iteration budget, and two contexts solving at once.

Held to the solver's stopping rule recomputed in numpy, like the row blocks' test.
"""
import threading

import numpy as np
import pytest
import scipy.sparse as sp

from gpu_common import announce, have_gpu, jittered_kuhn, require_lib
from paper_2102_06248_amd import inputs
from test_gpu_row_blocks import fan

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.fixture(scope="module")
def F():
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    return require_lib()


def operators(F, L):
    n = L.sizes["n_edges"]
    M, S = (sp.csr_matrix((v, (r, c)), shape=(n, n)) for r, c, v in (F.fepic_get_matrix(L.ctx, w) for w in (0, 1)))
    d = M.diagonal() > 0
    return M, S, d, 6.0 / np.sqrt(np.median(S.diagonal()[d] / M.diagonal()[d]))


def check_step(F, L, M, S, dt):
    """One vacuum step; ||b - A e|| <= TOL ||b|| up to the products' round-off."""
    e0, e1, _ = F.fepic_get_fields(L.ctx)
    st = F.fepic_step(L.ctx, dt)
    x, prev, _ = F.fepic_get_fields(L.ctx)
    assert np.array_equal(prev, e0)
    A = M + 0.25 * dt * dt * S
    b = M @ (2 * e0 - e1) - dt * dt * (S @ (0.5 * e0 + 0.25 * e1))
    nb = np.linalg.norm(b)
    width = int(np.diff(M.indptr).max())
    round_off = width * 2.0 ** -53 * np.linalg.norm(abs(A) @ abs(x)) / nb
    assert np.linalg.norm(b - A @ x) / nb <= TOL + 2 * round_off
    return st.cg_iters


def start(F, L, d):
    n = L.sizes["n_edges"]
    F.fepic_set_fields(L.ctx, *(np.where(d, inputs.random_field_dofs(n, 1.0, s), 0.0) for s in (3, 4)))


# n = 26: 129,194 rows, 253 blocks of 512; n = 27: 144,423 rows, 283 blocks for 256 CUs
@pytest.mark.parametrize("n,deterministic", [(2, 0), (7, 0), (7, 1), (26, 0), (27, 0)])
def test_stopping_rule(F, n, deterministic):
    announce(f"one launch: n={n}, deterministic={deterministic}")
    xyz, tets = jittered_kuhn(n, seed=1)[:2]
    with F.Simulation(xyz, tets, device=0, cg_tol=TOL, preconditioner=F.FEPIC_PC_JACOBI, cg_max_iters=20000,
                      deterministic=deterministic) as L:
        M, S, d, dt = operators(F, L)
        start(F, L, d)
        for _ in range(3):
            assert check_step(F, L, M, S, dt) > 0


# n = 33: 261,459 rows, 511 blocks, two for each of 256 workgroups; n = 34: 558 blocks; the
# fan's axis nodes have more than 80 edges
@pytest.mark.parametrize("mesh,far", [(2, -1), (7, -1), (12, 0), (12, 1), (12, 2), (26, -1), (27, -1), (33, -1), (34, -1),
                                      ("fan", 0)])
@pytest.mark.parametrize("solve", ["fp64", "mixed"])
def test_stopping_rule_auxiliary_space(F, mesh, far, solve):
    announce(f"one launch, auxiliary space: {mesh}, far levels {far}, {solve}")
    xyz, tets = fan(40) if mesh == "fan" else jittered_kuhn(mesh, seed=1)[:2]
    precision = F.FEPIC_SOLVE_MIXED if solve == "mixed" else F.FEPIC_SOLVE_FP64
    with F.Simulation(xyz, tets, device=0, cg_tol=TOL, preconditioner=F.FEPIC_PC_AUX, cg_max_iters=5000,
                      solve_precision=precision, aux_far_levels=far) as L:
        M, S, d, dt = operators(F, L)
        start(F, L, d)
        for _ in range(2):
            assert check_step(F, L, M, S, dt) > 0


def test_iteration_budget(F):
    announce("one launch: iteration budget")
    xyz, tets = jittered_kuhn(7, seed=1)[:2]
    with F.Simulation(xyz, tets, device=0, cg_tol=TOL, preconditioner=F.FEPIC_PC_JACOBI, cg_max_iters=3) as L:
        _, _, d, dt = operators(F, L)
        start(F, L, d)
        with pytest.raises(F.FepicError):
            F.fepic_step(L.ctx, dt)


def test_two_contexts_at_once(F):
    announce("one launch: two contexts at once")
    xyz, tets = jittered_kuhn(23, seed=1)[:2]   # 176 workgroups each: not resident side by side
    out, ref, errors = {}, None, []

    def run(k):
        try:
            with F.Simulation(xyz, tets, device=0, cg_tol=TOL, preconditioner=F.FEPIC_PC_JACOBI, cg_max_iters=20000,
                              deterministic=1) as L:
                _, _, d, dt = operators(F, L)
                start(F, L, d)
                for _ in range(4):
                    F.fepic_step(L.ctx, dt)
                out[k] = F.fepic_get_fields(L.ctx)[0]
        except Exception as e:   # reported by the main thread
            errors.append(e)

    run(0)
    ref = out.pop(0)
    threads = [threading.Thread(target=run, args=(k,)) for k in (1, 2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    assert np.array_equal(out[1], ref) and np.array_equal(out[2], ref)
