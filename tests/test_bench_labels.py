"""What bench.py's roofline line says of the PCG iteration follows from how the library made
the solve, not from the mesh's size."""
import pytest

import bench


@pytest.mark.parametrize("pc,solve,one_launch,kernel", [
    ("jacobi", "fp64", False, "k_cg_iter"), ("jacobi", "fp64", True, "k_cg_solve"),
    ("aux", "fp64", True, "k_pcg_solve"), ("aux", "mixed", True, "k_pcg_solve"),
    ("aux", "fp64", False, "k_pcg_q"), ("aux", "mixed", False, "k_pcg_q<float>")])
def test_iteration_roofline(pc, solve, one_launch, kernel):
    r = bench.iteration_roofline(pc, solve, one_launch, 4000.0, 123)
    assert r["kernel"].startswith(kernel)
    if one_launch:   # the matrix does not leave the registers: no share of HBM is claimed
        assert r["achieved"] is None and r["frac"] is None and r["traffic"] is None
    else:
        assert r["bound"] == "hbm" and r["achieved"] == 4000.0 and r["traffic"] == 123
        assert r["frac"] == round(4000.0 / bench.HBM_PEAK_GBS, 4)
