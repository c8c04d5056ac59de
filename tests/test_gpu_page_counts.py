"""Histogram counts that travel with their ln g through the page of the
lane-per-walker sweep (Ising L = 32), against the oracle: every page size that
shifts, workgroups of 64 and of fewer lanes, with and without the random
number wavefront, both precisions, several launches, and windows that freeze
while others go on.  Histograms, energies and ln g bit for bit.  L = 31, whose
page gathers increments, goes through the same."""
import numpy as np
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [31, 32])
@pytest.mark.parametrize("precision", [WL.FP64, WL.FP32C])
@pytest.mark.parametrize("page,group,producer", [(16, 64, 0), (16, 40, 1), (32, 7, 0), (64, 64, 1)])
def test_counts_follow_the_page(L, precision, page, group, producer):
    cfg = WL.config(WL.ISING, L, n_windows=24, walkers_per_window=3, precision=precision,
                    flat=(1, 50), lnf_final=0.6, seed=5)
    ctx, sim = gpu_context([cfg]), oracle_sim(cfg)
    (plan,) = ctx.set_launch(page_bins=page, walkers_per_group=group, rng_producer=producer).values()
    assert plan["page_bins"] == page and plan["walkers_per_group"] == group
    frozen = []
    for _ in range(6):
        ctx.run_cycles(1, 8000)
        oracle_cycle(sim, 8000)
        frozen.append(int(np.sum(ctx.status(0)["frozen"])))
        compare_state(ctx, 0, sim)
    assert any(0 < f < 24 for f in frozen), frozen
