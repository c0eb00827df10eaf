"""The counting sort's scan at the edges of its two forms (every block sums the blocks before
it; or, past 12,288 blocks of 1,024 tets, one block scans the sums), by the launcher itself: no
mesh of 12.6M tets has to be built.  Live particles come out grouped by tet with all their
words, the counts are left zero, and the live count arrives on both sides.
"""
import ctypes

import numpy as np
import pytest

from gpu_common import announce, have_gpu, require_lib

pytestmark = pytest.mark.gpu
LINE = 12288 * 1024


class PArrays(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("tet", "l1", "l2", "l3", "u0", "u1", "u2", "id")]


class AbHistIo(ctypes.Structure):
    _fields_ = [("hin", ctypes.c_void_p), ("hout", ctypes.c_void_p), ("stride", ctypes.c_int64),
                ("min", ctypes.c_void_p), ("mout", ctypes.c_void_p)]


@pytest.mark.parametrize("n_tets", [1, 1024, 1025, 300_000, LINE - 1, LINE, LINE + 1, LINE + 5000])
def test_sort(n_tets):
    if not have_gpu():
        pytest.fail("GPU tests need an MI355X")
    F = require_lib()
    import torch

    announce(f"sort over {n_tets} tets")
    sort = getattr(ctypes.CDLL(F.LIB_PATH),
                   "_ZN5fepic11launch_sortIfEEvP12ihipStream_tNS_7PArraysIT_EES5_llPiS6_S6_S6_S6_NS_8AbHistIoE")
    P = ctypes.c_void_p
    sort.argtypes = [P, PArrays, PArrays, ctypes.c_int64, ctypes.c_int64, P, P, P, P, P, AbHistIo]
    sort.restype = None
    n = 5000
    rng = np.random.default_rng(n_tets % 1000)
    tet = rng.integers(0, n_tets, n).astype(np.int32)
    tet[:: 3] = n_tets - 1 - rng.integers(0, min(n_tets, 7), len(tet[:: 3]))   # the last tets, several each
    tet[:: 11] = -1
    words = {k: rng.normal(size=n).astype(np.float32) for k in ("l1", "l2", "l3", "u0", "u1", "u2")}
    words = {"tet": tet, **words, "id": np.arange(n, dtype=np.int64)}
    dev = {k: torch.from_numpy(v.copy()).to("cuda") for k, v in words.items()}
    out = {k: torch.zeros_like(v) for k, v in dev.items()}
    blocks = (n_tets + 1023) // 1024
    count, offset, sums, live = (torch.zeros(k, dtype=torch.int32, device="cuda") for k in (n_tets, n_tets, blocks + 1, 1))
    host = torch.zeros(1, dtype=torch.int32, pin_memory=True)
    sums[blocks] = 77   # not the scan's
    pack = lambda d: PArrays(*(d[f].data_ptr() for f, _ in PArrays._fields_))
    torch.cuda.synchronize()
    want = words["id"][tet >= 0]
    for _ in range(2):   # again from the counts as they were left
        sort(torch.cuda.current_stream().cuda_stream, pack(dev), pack(out), n, n_tets, count.data_ptr(),
             offset.data_ptr(), sums.data_ptr(), live.data_ptr(), host.data_ptr(), AbHistIo())
        torch.cuda.synchronize()
        assert host.item() == live.item() == len(want)
        assert int(count.abs().max()) == 0 and int(sums[blocks]) == 77
        got = {k: v.cpu().numpy()[: len(want)] for k, v in out.items()}
        assert np.all(np.diff(got["tet"]) >= 0)
        assert np.array_equal(np.sort(got["id"]), want)
        for k, v in words.items():
            assert np.array_equal(got[k], v[got["id"]]), k
