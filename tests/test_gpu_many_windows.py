"""End of a cycle and end of a run at the edges of their kernels (GPU): more
than 64 window pairs in an exchange round, 64 walkers per window, more than
256 windows in a join, window representatives that do not all fit in LDS,
odd walker counts in the pairwise sums, and windows that freeze together.

Every window counts as flat at its first check (flatness 0), so one cycle
merges, the second freezes, and the pieces, join and jackknife follow.  State
and unnormalised join bit for bit; the jackknife's mean within 1e-12 or 8 ulp
of the largest value (it goes through the platform's exp and log), its error
within 1e-8 relative.
"""
import numpy as np
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu

CASES = {
    "131_windows_64_walkers": WL.config(WL.ISING, 24, n_windows=131, walkers_per_window=64),
    "300_windows_3_walkers": WL.config(WL.ISING, 32, n_windows=300, walkers_per_window=3),
    "300_windows_5_walkers_fp32c": WL.config(WL.ISING, 32, n_windows=300, walkers_per_window=5,
                                             precision=WL.FP32C),
    "8193_bins_16_windows": WL.config(WL.POTTS, 64, q=4, n_windows=16, walkers_per_window=2),
    "8193_bins_1_window": WL.config(WL.POTTS, 64, q=4, n_windows=1, walkers_per_window=7),
    "one_walker": WL.config(WL.ISING, 8, n_windows=3, walkers_per_window=1),
}


@pytest.mark.parametrize("name", CASES)
def test_cycle_end_and_results_match_the_oracle(name):
    cfg = dict(CASES[name], flat=(0, 1), lnf_final=0.3, seed=9)
    F = 300
    ctx, sim = gpu_context([cfg]), oracle_sim(cfg)
    W = cfg["n_windows"] * cfg["walkers_per_window"]
    slots = sorted(set(np.linspace(0, W - 1, 60).astype(int).tolist()))
    for _ in range(2):
        ctx.run_sweeps(F)
        ctx.merge()
        ctx.exchange()
        oracle_cycle(sim, F)
        compare_state(ctx, 0, sim, slots=slots, windows=W < 2000)
    t, r, a = ctx.get_exchange_stats(0)
    for got, want in zip((t, r, a), sim.exchange_stats()):
        assert np.array_equal(got, want)
    assert ctx.status(0)["done"] == 1
    raw_g, joins_g = ctx.get_lng(0, normalise=False)
    raw_o, joins_o = sim.join(normalise=False)
    assert np.array_equal(joins_g, joins_o)
    assert np.array_equal(raw_g.view(np.uint64), raw_o.view(np.uint64))
    if cfg["walkers_per_window"] > 1 and np.isfinite(raw_o[0]) and cfg["n_windows"] > 1:
        mean_g, err_g = ctx.jackknife(0)
        mean_o, err_o = sim.jackknife()
        fin = np.isfinite(mean_o)
        assert np.array_equal(np.isfinite(mean_g), fin)
        tol = max(1e-12, 8 * np.finfo(float).eps * np.abs(mean_o[fin]).max())
        assert np.abs(mean_g[fin] - mean_o[fin]).max() < tol
        assert np.allclose(err_g, err_o, rtol=1e-8, atol=1e-11)
