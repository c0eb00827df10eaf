"""Failed device allocations leave no error behind: a call that does without the memory (the
exchange words of a one-launch solve) goes on, instead of failing at its next check.
"""
import ctypes

import numpy as np
import pytest

from gpu_common import announce, have_gpu, jittered_kuhn, require_lib
from paper_2102_06248_amd import inputs

pytestmark = pytest.mark.gpu
TOO_MUCH = 1 << 60   # bytes


@pytest.fixture(scope="module")
def F():
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    return require_lib()


def test_failed_allocation_leaves_no_error(F):
    announce("failed allocation")
    lib = ctypes.CDLL(F.LIB_PATH)
    dmalloc = getattr(lib, "_ZN5fepic7dmallocEP9fepic_ctxm")   # fepic::dmalloc(fepic_ctx*, size_t)
    dmalloc.restype, dmalloc.argtypes = ctypes.c_void_p, [ctypes.c_void_p, ctypes.c_size_t]
    ctx = F.fepic_create(device=-1)
    try:
        lib.hipGetLastError()
        assert dmalloc(ctx, TOO_MUCH) is None
        assert lib.hipGetLastError() == 0
    finally:
        F.fepic_destroy(ctx)


@pytest.mark.parametrize("pc", ["jacobi", "aux"])
def test_step_without_memory_for_the_exchange_words(F, pc):
    announce(f"one-launch solve without memory for its words: {pc}")
    lib = ctypes.CDLL(F.LIB_PATH)
    lib.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
    lib.hipFree.argtypes = [ctypes.c_void_p]
    state = {"full": False, "refused": 0}

    def alloc(n):   # once "full", as hipMalloc answers when there is no memory
        p = ctypes.c_void_p()
        state["refused"] += state["full"]
        rc = lib.hipMalloc(ctypes.byref(p), TOO_MUCH if state["full"] else n)
        return p.value if rc == 0 else None

    xyz, tets = jittered_kuhn(5, seed=1)[:2]
    out = {}
    for full in (False, True):
        ctx = F.fepic_create(device=0, cg_tol=1e-12, preconditioner=F.FEPIC_PC_AUX if pc == "aux" else F.FEPIC_PC_JACOBI)
        try:
            keep = F.fepic_set_allocator(ctx, alloc, lib.hipFree)
            F.fepic_upload_mesh(ctx, xyz, tets)
            rows = np.unique(F.fepic_get_matrix(ctx, 0)[0])
            n = F.fepic_get_topology_sizes(ctx)["n_edges"]
            e = np.zeros(n)
            e[rows] = inputs.random_field_dofs(n, 1.0, 3)[rows]
            F.fepic_set_fields(ctx, e, e)
            state["full"] = full
            F.fepic_step(ctx, 1e-10)
            state["full"] = False
            out[full] = F.fepic_get_fields(ctx)[0]
        finally:
            state["full"] = False
            F.fepic_destroy(ctx)
        del keep
    assert state["refused"] > 0
    # two forms of the same solve, each to a residual of 1e-12
    assert np.linalg.norm(out[True] - out[False]) <= 1e-9 * np.linalg.norm(out[False])
