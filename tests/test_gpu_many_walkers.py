"""More walkers than wavefronts fit in one launch (GPU): 2^26 + 64, as 2^20 + 1
instances of 64 walkers on a 2 x 2 lattice (10.5 GB of workspace).  Through the
C entry points, since a million instances' geometry is not asked for one by
one; the first, a middle and the last instance match the oracle bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1402_2328_amd import rewl
from paper_1402_2328_amd import workloads as WL
from tests.parity import oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu
N_INST = 2 ** 20 + 1


@pytest.fixture(scope="module")
def batch():
    cfg = WL.config(WL.ISING, 2, n_windows=1, walkers_per_window=64, seed=4)
    one = WL.rewl_params_of(cfg)
    arr = (rewl.rewl_params * N_INST)()
    C.memmove(arr, bytes(one) * N_INST, C.sizeof(arr))
    L = rewl.lib()
    size = L.rewl_workspace_bytes(C.cast(arr, C.c_void_p), N_INST, None, None)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    h = C.c_void_p()
    rc = L.rewl_init(C.cast(arr, C.c_void_p), N_INST, None, None, C.c_void_p(ws.data_ptr()), size,
                     C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(h))
    assert rc == 0, rc
    yield L, h, cfg
    L.rewl_destroy(h)


def _walker(L, h, instance, slot):
    spins, H, lng = np.zeros(4, np.int8), np.zeros(5, np.uint32), np.zeros(5)
    E, att, cid = C.c_int32(), C.c_uint64(), C.c_int32()
    p = lambda a: a.ctypes.data_as(C.c_void_p)
    assert L.rewl_get_walker(h, instance, slot, p(spins), C.byref(E), p(H), p(lng), C.byref(att), C.byref(cid)) == 0
    return dict(spins=spins, E=E.value, H=H, lng=lng, attempts=att.value)


@pytest.mark.parametrize("shape", [(0, 0), (0, 1)], ids=["lanes", "wavefronts"])
def test_more_than_2_to_the_26_walkers(batch, shape):
    L, h, cfg = batch
    assert L.rewl_set_launch(h, -1, shape[0], shape[1], -1, -1, None) == 0
    before = _walker(L, h, 0, 0)["attempts"]
    assert L.rewl_run_sweeps(h, 70) == 0
    for i in (0, N_INST // 2, N_INST - 1):
        sim = oracle_sim(cfg, instance=i)
        for _ in range(before // 70 + 1):
            sim.sweep(70)
        for slot in (0, 1, 63):
            a, b = _walker(L, h, i, slot), sim.walker(slot)
            assert a["E"] == b["E"] and a["attempts"] == b["attempts"], (i, slot)
            assert np.array_equal(a["spins"], b["spins"]), (i, slot)
            assert np.array_equal(a["H"], b["H"]), (i, slot)
            assert np.array_equal(a["lng"].view(np.uint64), b["lng"].view(np.uint64)), (i, slot)
