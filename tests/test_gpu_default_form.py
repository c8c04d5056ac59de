"""Default form of a batch, one wavefront or one lane per walker (GPU), on both
sides of the lines: by lattice size up to a workgroup per compute unit, by
walkers per workgroup in batches of very many instances.  The state of the
first and the last instance matches the oracle bit for bit."""
import pytest
import torch

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,L,q,h,m,n,wave", [
    # 64 walkers, one workgroup, per instance: up to 3072 + 128 L walkers
    (WL.ISING, 8, 2, 4, 16, 64, True), (WL.ISING, 8, 2, 4, 16, 65, False), (WL.ISING, 8, 2, 4, 16, 112, False),
    (WL.ISING, 16, 2, 4, 16, 80, True), (WL.ISING, 16, 2, 4, 16, 81, False),
    (WL.ISING, 32, 2, 4, 16, 112, True), (WL.ISING, 32, 2, 4, 16, 113, False),
    (WL.ISING, 48, 2, 4, 16, 112, True), (WL.ISING, 48, 2, 4, 16, 113, False),
    (WL.POTTS, 8, 10, 4, 16, 64, True), (WL.POTTS, 8, 10, 4, 16, 65, False),
    (WL.POTTS, 24, 3, 4, 16, 88, True), (WL.POTTS, 24, 3, 4, 16, 89, False),
    # more workgroups than compute units
    (WL.ISING, 8, 2, 4, 4, 448, True), (WL.ISING, 8, 2, 4, 4, 449, False),
    # many instances: 5 of L = 8 per SIMD, and beyond, where 4.75 is the line
    (WL.ISING, 8, 2, 5, 1, 5120, True), (WL.ISING, 8, 2, 5, 1, 5121, False), (WL.ISING, 8, 2, 4, 1, 5121, True),
    (WL.POTTS, 8, 2, 5, 1, 5121, False), (WL.POTTS, 8, 3, 5, 1, 5121, True),
])
def test_default_form(model, L, q, h, m, n, wave):
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    cfg = WL.config(model, L, q=q, n_windows=h, walkers_per_window=m)
    ctx = gpu_context([cfg] * n)
    (plan,) = ctx.set_launch().values()
    assert (plan["walkers_per_group"] == 1) == wave, plan
    ctx.run_cycles(2, 300)
    for i in (0, n - 1):
        sim = oracle_sim(cfg, instance=i)
        oracle_cycle(sim, 300)
        oracle_cycle(sim, 300)
        compare_state(ctx, i, sim)
