"""Jackknife error bars at the edges of their kernels (GPU), values compared
with the oracle in every case: 8, 16 and 63 pieces left in (the loads go eight
at a time, past the left-out walker at either end of a group), 64 walkers per
window, more than 256 windows, and window representatives that do not all fit
in LDS (30 windows of L = 64 with an overlap of 9/10: 31 500 bins).  Ising
throughout, whose normalisation needs no particular bin visited.

Every window counts as flat at its first check, so the second cycle freezes
them all.  The mean within 1e-12 or 8 ulp of the largest value (it goes through
the platform's exp and log), the error within 1e-8 relative.  The
allocation-free form, where the instance fits, is the same bit for bit.
"""
import numpy as np
import pytest

from paper_1402_2328_amd import rewl
from paper_1402_2328_amd import workloads as WL
from tests.parity import gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu

CASES = {
    "9_walkers": WL.config(WL.ISING, 12, n_windows=3, walkers_per_window=9),
    "17_walkers_fp32c": WL.config(WL.ISING, 12, n_windows=3, walkers_per_window=17, precision=WL.FP32C),
    "131_windows_64_walkers": WL.config(WL.ISING, 24, n_windows=131, walkers_per_window=64),
    "300_windows_3_walkers": WL.config(WL.ISING, 32, n_windows=300, walkers_per_window=3),
    "300_windows_10_walkers_fp32c": WL.config(WL.ISING, 32, n_windows=300, walkers_per_window=10,
                                              precision=WL.FP32C),
    "representatives_beyond_lds": WL.config(WL.ISING, 64, n_windows=30, walkers_per_window=9, overlap=(9, 10)),
    "one_window": WL.config(WL.ISING, 16, n_windows=1, walkers_per_window=12),
}


@pytest.mark.parametrize("name", CASES)
def test_jackknife_matches_the_oracle(name):
    cfg = dict(CASES[name], flat=(0, 1), lnf_final=0.3, seed=9)
    ctx, sim = gpu_context([cfg]), oracle_sim(cfg)
    for _ in range(2):
        ctx.run_cycles(1, 300)
        oracle_cycle(sim, 300)
    assert ctx.status(0)["done"] == 1
    mean_g, err_g = ctx.jackknife(0)
    mean_o, err_o = sim.jackknife()
    fin = np.isfinite(mean_o)
    assert fin.sum() > 40 and (err_o[fin] > 0).sum() > 20    # something is compared
    assert np.array_equal(np.isfinite(mean_g), fin)
    tol = max(1e-12, 8 * np.finfo(float).eps * np.abs(mean_o[fin]).max())
    assert np.abs(mean_g[fin] - mean_o[fin]).max() < tol
    assert np.allclose(err_g, err_o, rtol=1e-8, atol=1e-11)
    g = ctx.geometry[0]
    reps = int((g["hi"] - g["lo"] + 1).sum())
    if (g["m"] + 2) * g["nbins"] + (reps + 31) // 32 * 32 <= 2 ** 19:
        mean_n, err_n = ctx.jackknife_noalloc(0)
        assert np.array_equal(mean_n, mean_g) and np.array_equal(err_n, err_g)
    else:
        with pytest.raises(rewl.RewlError):
            ctx.jackknife_noalloc(0)
