"""No cycles asked for (GPU): the call returns and changes nothing, with the
graph and without."""
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_graph", [False, True])
def test_no_cycles(use_graph):
    cfg = WL.config(WL.ISING, 8, n_windows=3, walkers_per_window=2, seed=6)
    ctx, sim = gpu_context([cfg]), oracle_sim(cfg)
    for cycles in (0, 2, 0):
        ctx.run_cycles(cycles, 300, use_graph=use_graph)
        for _ in range(cycles):
            oracle_cycle(sim, 300)
        compare_state(ctx, 0, sim)
