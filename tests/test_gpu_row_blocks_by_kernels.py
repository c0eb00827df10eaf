"""The row-block products by a launch per kernel and iteration on meshes whose solves are one
launch otherwise (switched off here), and the deterministic mode's loop over several blocks per
workgroup, which only meshes past the one-launch solve reach: held to the stopping rule, and
the deterministic ones to repeat bit for bit.
"""
import numpy as np
import pytest

from gpu_common import announce, have_gpu, jittered_kuhn, require_lib
from test_gpu_give_up import options
from test_gpu_one_launch import TOL, check_step, operators, start
from test_gpu_row_blocks import MESHES, fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    return require_lib()


@pytest.mark.parametrize("mesh", ["one_partial_block", "ragged_blocks", "looped_blocks"])
@pytest.mark.parametrize("solve", ["jacobi", "deterministic", "fp64", "mixed"])
def test_by_kernels(F, mesh, solve):
    announce(f"row blocks by kernels: {mesh}, {solve}")
    xyz, tets = MESHES[mesh]()
    with F.Simulation(xyz, tets, device=0, cg_tol=TOL, **options(F, solve)) as L:
        M, S, d, dt = operators(F, L)
        start(F, L, d)
        F.fepic_set_solve_polls(L.ctx, -1)
        for _ in range(2):
            assert check_step(F, L, M, S, dt) > 0
            assert F.fepic_get_solve_form(L.ctx) == (F.FEPIC_SOLVE_FORM_KERNELS, 0)


# 144,423 rows: 283 blocks, five for some of 64 workgroups; the fan's axis rows are gathered
@pytest.mark.parametrize("mesh", ["cube", "fan"])
def test_deterministic_past_one_launch(F, mesh):
    announce(f"row blocks, deterministic past the one-launch solve: {mesh}")
    xyz, tets = jittered_kuhn(27, seed=1)[:2] if mesh == "cube" else fan(1600)
    out = []
    for _ in range(2):
        with F.Simulation(xyz, tets, device=0, cg_tol=TOL, **options(F, "deterministic")) as L:
            M, S, d, dt = operators(F, L)
            start(F, L, d)
            iters = [check_step(F, L, M, S, dt) for _ in range(2)]
            assert F.fepic_get_solve_form(L.ctx) == (F.FEPIC_SOLVE_FORM_KERNELS, 0)
            out.append((iters, F.fepic_get_fields(L.ctx)[0]))
    assert out[0][0] == out[1][0] and out[0][0][0] > 0
    assert np.array_equal(out[0][1].view(np.uint64), out[1][1].view(np.uint64))
