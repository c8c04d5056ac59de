"""Exchange rounds in which an instance has few window pairs or none (GPU):
one window, and two or three windows in odd and even rounds.  Every wavefront
of an instance's block has to act on the same round number, also where nothing
but that number is written.  State, exchange statistics and counters against
the oracle, bit for bit, in a batch of instances with and without pairs."""
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 5, 64])
def test_rounds_without_pairs(m):
    cfgs = [WL.config(WL.ISING, 8, n_windows=1 + i % 3, walkers_per_window=m, seed=3, flips=200)
            for i in range(48)]
    ctx = gpu_context(cfgs)
    sims = [oracle_sim(c, instance=i) for i, c in enumerate(cfgs)]
    ctx.run_sweeps(200)
    for sim in sims:
        sim.sweep(200)
    for rnd in range(6):
        ctx.exchange()
        for i, sim in enumerate(sims):
            sim.exchange()
            assert ctx.status(i)["rounds"] == rnd + 1
    for i, sim in enumerate(sims):
        compare_state(ctx, i, sim)


@pytest.mark.parametrize("h,m", [(130, 1), (65, 9), (33, 33), (17, 64), (520, 2)])
def test_rounds_of_many_proposals(h, m):
    """Blocks of 256, 512 and 1024 threads with a last turn that is partly
    empty, and more than 256 pairs."""
    cfg = WL.config(WL.ISING, 40 if h > 300 else 24, n_windows=h, walkers_per_window=m, seed=3)
    ctx, sim = gpu_context([cfg]), oracle_sim(cfg)
    for _ in range(3):
        ctx.run_sweeps(150)
        ctx.exchange()
        sim.sweep(150)
        sim.exchange()
    compare_state(ctx, 0, sim)
