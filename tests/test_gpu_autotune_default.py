"""The tuner knows the default plan (GPU): of a batch of very many instances of
few walkers, set to lanes before, it finds the wavefront form again, which is
about twice as fast here (28 800 walkers of q = 10 Potts L = 6 of 3)."""
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


def test_the_default_plan_is_a_candidate():
    cfg = WL.config(WL.POTTS, 6, q=10, n_windows=3, walkers_per_window=1, lnf_final=1e-12)
    ctx = gpu_context([cfg] * 9600)
    (default,) = ctx.set_launch().values()
    assert default["walkers_per_group"] == 1
    ctx.set_launch(page_bins=32, rng_producer=0)
    (plan,) = (p for k, p in ctx.autotune(400, repeats=3).items() if k != "batching")
    assert plan == default
    ctx.run_cycles(2, 300)
    for i in (0, 9599):
        sim = oracle_sim(cfg, instance=i)
        oracle_cycle(sim, 300)
        oracle_cycle(sim, 300)
        compare_state(ctx, i, sim)
