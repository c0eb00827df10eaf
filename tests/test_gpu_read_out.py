"""Read-outs through the pinned buffer, exact round trips at the sizes where the pieces meet:
all arrays in one fill, arrays split over several fills of 65,536 words, four-byte and
widened pieces of odd length.
"""
import numpy as np
import pytest

from gpu_common import announce, have_gpu, jittered_kuhn, require_lib
from paper_2102_06248_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    return require_lib()


# 19, 604 and 102,024 edges; 18, 864 and 169,344 faces
@pytest.mark.parametrize("n", [1, 4, 24])
def test_fields(F, n):
    announce(f"read-out: fields, n={n}")
    xyz, tets = jittered_kuhn(n, seed=1)[:2]
    with F.Simulation(xyz, tets, device=0) as L:
        ne, nf = L.sizes["n_edges"], L.sizes["n_faces"]
        free = np.zeros(ne, bool)
        free[F.fepic_get_matrix(L.ctx, 0)[0]] = True   # wall edges have no row and are held at zero
        for k in range(2):       # again with other values through the same buffer
            e, ep = (np.where(free, inputs.random_field_dofs(ne, 1.0, 10 * k + s), 0.0) for s in (3, 4))
            b = inputs.random_field_dofs(nf, 1.0, 10 * k + 5)
            F.fepic_set_fields(L.ctx, e, ep, b)
            got = F.fepic_get_fields(L.ctx)
            assert np.array_equal(got[0], e) and np.array_equal(got[1], ep) and np.array_equal(got[2], b)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("count", [1, 70_001])
def test_particles(F, count, precision):
    announce(f"read-out: {count} particles, {precision}")
    xyz, tets = jittered_kuhn(4, seed=1)[:2]
    rng = np.random.default_rng(0)
    lo, hi = xyz.min(0), xyz.max(0)
    x = lo + (hi - lo) * (0.1 + 0.8 * rng.random((count, 3)))
    u = rng.normal(size=(count, 3)) * 1e6
    with F.Simulation(xyz, tets, device=0, precision=F.FEPIC_ALL_FP64 if precision == "fp64" else F.FEPIC_FP32_PUSH_FP64_ACC) as L:
        F.fepic_add_species(L.ctx, -1.6e-19, 9.1e-31, 1.0)
        F.fepic_inject_particles(L.ctx, 0, x, u)
        p = F.fepic_get_particles(L.ctx, 0, ("id", "x", "u"))
    order = np.argsort(p["id"])
    assert np.array_equal(p["id"][order], np.arange(count))
    assert np.array_equal(p["u"][order], u if precision == "fp64" else u.astype(np.float32))
    # positions come back from barycentric coordinates of the storage precision, each rounded
    # once and multiplied by coordinates of magnitude up to the box
    eps = 2.0 ** -50 if precision == "fp64" else 2.0 ** -22
    assert np.abs(p["x"][order] - x).max() <= 4 * eps * np.abs(xyz).max() + eps * np.ptp(xyz)
