"""Both forms of the histogram in the page of the lane-per-walker sweep (GPU):
whole counts in batches of at least a workgroup per SIMD (1024) whose ln g and
H exceed the last-level cache, else increments (but for L = 32, whose loop
always keeps counts).  Against the oracle, bit for bit, on both sides of that
line: one and two lattice words per row, L a power of two and not, with and
without the random number wavefront, workgroups of 64 and of fewer lanes."""
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


# 12 bytes per bin and walker; the line is at 302 MB and 1024 workgroups
@pytest.mark.parametrize("L,h,m,n", [
    (31, 1, 64, 1030), (31, 1, 64, 600),    # 761 MB; 443 MB in 600 workgroups of 64
    (16, 1, 64, 1600), (16, 2, 33, 40),     # 316 MB
    (40, 4, 16, 1030), (40, 3, 16, 20),     # 724 MB
    (64, 1, 32, 1030),                      # 1621 MB
])
@pytest.mark.parametrize("precision", [WL.FP64, WL.FP32C])
@pytest.mark.parametrize("page,group,producer", [(16, 64, 0), (16, 40, 1), (64, 24, 0)])
def test_counts_and_increments(L, h, m, n, precision, page, group, producer):
    cfg = WL.config(WL.ISING, L, n_windows=h, walkers_per_window=m, precision=precision, seed=8)
    ctx = gpu_context([cfg] * n)
    (plan,) = ctx.set_launch(page_bins=page, walkers_per_group=group, rng_producer=producer).values()
    assert plan["page_bins"] == page
    for _ in range(2):
        ctx.run_cycles(1, 2000)
    slots = list(range(0, h * m, 7)) + [h * m - 1]
    for i in (0, n - 1):
        sim = oracle_sim(cfg, instance=i)
        for _ in range(2):
            oracle_cycle(sim, 2000)
        compare_state(ctx, i, sim, slots=slots)
    ctx.close()
