"""The edge matrices' products by row blocks (16-bit columns, halo staged in LDS) at the
sizes where they can go wrong: one partial block, a few blocks with a ragged last one, and
a fan of tets around a chain of axis edges, whose rows of thousands of entries overflow the
halo list so that their blocks gather from memory, and exceed the slots held in registers.

One vacuum step from random fields; the solution is held to the solver's stopping rule
||b - A e|| <= tol ||b|| recomputed in numpy from the library's exported M and S (those are
pinned against the oracle's quadrature elsewhere).  The rule is the library's own on FP64
products, so only round-off separates the two: slots per row * 2^-53 * || |A| |e| || / ||b||,
added to the bound.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from gpu_common import announce, have_gpu, jittered_kuhn, require_lib
from paper_2102_06248_amd import inputs

pytestmark = pytest.mark.gpu
TOL = 1e-10
DT_CELLS = 6.0


@pytest.fixture(scope="module")
def F():
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    return require_lib()


def fan(n):
    """n tets around each of two axis edges a0-a1-a2, closed by apexes above and below and an
    outer ring, so that the axis, spoke and ring edges are interior."""
    th = 2 * np.pi * np.arange(n) / n
    ring = np.stack([np.cos(th), np.sin(th)], 1)
    axis = np.array([[0, 0, z] for z in (-1.0, 0.0, 1.0)])
    ends = np.array([[0, 0, -2.0], [0, 0, 2.0]])
    inner = np.column_stack([ring, np.zeros(n)])
    outer = np.column_stack([2.5 * ring, np.zeros(n)])
    xyz = np.concatenate([axis, ends, inner, outer])
    i = np.arange(n)
    r0, r1 = 5 + i, 5 + (i + 1) % n
    o0, o1 = r0 + n, r1 + n
    full = np.full(n, 1)
    tets = []
    for a, b in ((3, 0), (0, 1), (1, 2), (2, 4)):
        tets.append(np.stack([a * full, b * full, r0, r1], 1))
    # between the rings, above and below: the quad (r0, r1, o0, o1) joined to each end node,
    # its diagonal from the lower to the higher ring position
    for e in (3, 4):
        tets.append(np.stack([e * full, r0, r1, o1], 1))
        tets.append(np.stack([e * full, r0, o0, o1], 1))
    return xyz, np.concatenate(tets).astype(np.int32)


MESHES = {"one_partial_block": lambda: jittered_kuhn(2, seed=1)[:2], "ragged_blocks": lambda: jittered_kuhn(7, seed=2)[:2],
          # 37,043 rows: more blocks than the deterministic mode's 64 workgroups
          "looped_blocks": lambda: jittered_kuhn(17, seed=3)[:2], "fan": lambda: fan(1600)}


@pytest.mark.parametrize("mesh,solve", [("one_partial_block", "fp64"), ("one_partial_block", "mixed"),
                                        ("one_partial_block", "jacobi"), ("one_partial_block", "deterministic"),
                                        ("ragged_blocks", "fp64"), ("ragged_blocks", "mixed"),
                                        ("ragged_blocks", "jacobi"), ("ragged_blocks", "deterministic"),
                                        ("looped_blocks", "deterministic"), ("fan", "fp64"), ("fan", "mixed"),
                                        ("fan", "jacobi")])
def test_solution_meets_stopping_rule(F, mesh, solve):
    announce(f"row blocks: {mesh}, {solve}")
    xyz, tets = MESHES[mesh]()
    opts = {"fp64": dict(), "mixed": dict(solve_precision=F.FEPIC_SOLVE_MIXED),
            "jacobi": dict(preconditioner=F.FEPIC_PC_JACOBI),
            "deterministic": dict(preconditioner=F.FEPIC_PC_JACOBI, deterministic=1)}[solve]
    with F.Simulation(xyz, tets, device=0, cg_tol=TOL, aux_far_levels=0, **opts) as L:
        n = L.sizes["n_edges"]
        M, S = (sp.csr_matrix((v, (r, c)), shape=(n, n)) for r, c, v in (F.fepic_get_matrix(L.ctx, w) for w in (0, 1)))
        width = int(np.diff(M.indptr).max())
        if mesh == "fan":
            assert width > 4096 + 512   # more columns than a block's list and own rows hold
        # a step of DT_CELLS cells by the operators' own scale
        d = M.diagonal() > 0
        dt = DT_CELLS / np.sqrt(np.median(S.diagonal()[d] / M.diagonal()[d]))
        e0, e1 = (np.where(d, inputs.random_field_dofs(n, 1.0, s), 0.0) for s in (3, 4))
        F.fepic_set_fields(L.ctx, e0, e1)
        F.fepic_step(L.ctx, dt)
        x, prev, _ = F.fepic_get_fields(L.ctx)
    assert np.array_equal(prev, e0)
    A = M + 0.25 * dt * dt * S
    b = M @ (2 * e0 - e1) - dt * dt * (S @ (0.5 * e0 + 0.25 * e1))
    nb = np.linalg.norm(b)
    round_off = width * 2.0 ** -53 * np.linalg.norm(abs(A) @ abs(x)) / nb
    assert np.linalg.norm(b - A @ x) / nb <= TOL + 2 * round_off
