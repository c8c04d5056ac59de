"""Default page of large batches (GPU): as few turns per compute unit as the
smallest page allows, then the largest page that keeps them.  The state of a
few instances matches the oracle bit for bit."""
import pytest
import torch

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


# 64 walkers, one workgroup, per instance; LDS per walker 4 B per lattice word
# and 12 B per bin; 163840 B per compute unit in pieces of 1280 B
@pytest.mark.parametrize("L,per_cu,page", [
    (16, 5, 32),    # 64 + 384 B: 5 fit
    (16, 6, 16),    # 64 + 192 B: 10 fit
    (20, 3, 32),    # 80 + 768 B: three take 165120 B
    (32, 4, 32),    # 128 + 384 B: 4 fit
    (32, 5, 16),    # five take 166400 B
    (32, 6, 16),    # 128 + 192 B: 8 fit
    (16, 11, 16),   # two turns of six, 64 + 192 B
    (64, 4, 64),    # 512 + 192 B: 3 fit; two turns of two, 512 + 768 B
])
def test_default_page_of_a_large_batch(L, per_cu, page):
    cfg = WL.config(WL.ISING, L, n_windows=16, walkers_per_window=4)
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count - 3
    ctx = gpu_context([cfg] * n)
    (plan,) = ctx.set_launch().values()
    assert plan["page_bins"] == page, plan
    ctx.run_cycles(2, 600)
    for i in (0, n // 2, n - 1):
        sim = oracle_sim(cfg, instance=i)
        oracle_cycle(sim, 600)
        oracle_cycle(sim, 600)
        compare_state(ctx, i, sim)


@pytest.mark.parametrize("model,L,q,h,wave", [
    (WL.ISING, 12, 2, 6, True), (WL.ISING, 12, 2, 8, False),
    (WL.POTTS, 6, 10, 5, True), (WL.POTTS, 6, 10, 6, False),
])
def test_default_form_of_many_small_instances(model, L, q, h, wave):
    """Up to 7 (Potts 5.5) walkers per instance have a wavefront each."""
    cfg = WL.config(model, L, q=q, n_windows=h, walkers_per_window=1)
    n = 1700
    ctx = gpu_context([cfg] * n)
    (plan,) = ctx.set_launch().values()
    assert (plan["walkers_per_group"] == 1) == wave, plan
    ctx.run_cycles(2, 700)
    for i in (0, n - 1):
        sim = oracle_sim(cfg, instance=i)
        oracle_cycle(sim, 700)
        oracle_cycle(sim, 700)
        compare_state(ctx, i, sim)
