"""The sweep with one wavefront per walker (walkers_per_group = 1, and the
default of small batches) against the oracle, bit for bit (GPU).

The configurations sit where the form can go wrong: windows below, at and
just above the 64 bins of its register page and several pages wide, lattices
so small that most of 64 attempts share a site or a neighbour (down to L = 2,
where right and left neighbour are one site), the largest lattice, Potts
values up to 127, and sweeps that are no multiple of 64 attempts.
"""
import numpy as np
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


def _c(model, L, **kw):
    return WL.config(model, L, **dict(dict(walkers_per_window=2, seed=11, lnf_final=1e-4), **kw))


# one window over the whole range unless explicit windows (bins) are given
CASES = {
    "ising_L2": (_c(WL.ISING, 2), None),
    "ising_L3": (_c(WL.ISING, 3), None),
    "ising_L8_65_bins": (_c(WL.ISING, 8), None),
    "ising_L8_63_64_bins": (_c(WL.ISING, 8, n_windows=2), ([0, 2], [62, 64])),
    "ising_L8_fp32c": (_c(WL.ISING, 8, n_windows=3, precision=WL.FP32C), None),
    "ising_L16_257_bins": (_c(WL.ISING, 16), None),
    "ising_L16_257_bins_fp32c_1t": (_c(WL.ISING, 16, precision=WL.FP32C, schedule=WL.ONE_OVER_T), None),
    "ising_L17_290_bins": (_c(WL.ISING, 17, n_windows=1), None),
    "ising_L32_h2": (_c(WL.ISING, 32, n_windows=2), None),
    "ising_L64_h3": (_c(WL.ISING, 64, n_windows=3), None),
    "potts_q2_L9": (_c(WL.POTTS, 9, q=2), None),
    "potts_q3_L2": (_c(WL.POTTS, 2, q=3), None),
    "potts_q3_L6_73_bins": (_c(WL.POTTS, 6, q=3), None),
    "potts_q10_L12_h2": (_c(WL.POTTS, 12, q=10, n_windows=2), None),
    "potts_q127_L11_fp32c": (_c(WL.POTTS, 11, q=127, precision=WL.FP32C), None),
    "potts_q16_L64_h4": (_c(WL.POTTS, 64, q=16, n_windows=4, walkers_per_window=1), None),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("explicit", [False, True])
def test_wavefront_per_walker_matches_the_oracle(name, explicit):
    cfg, win = CASES[name]
    ctx = gpu_context([cfg], windows=[win] if win else None)
    if explicit:
        (plan,) = ctx.set_launch(walkers_per_group=1).values()
        assert plan["walkers_per_group"] == 1
        assert plan["workgroups"] == cfg["n_windows"] * cfg["walkers_per_window"]
    sim = oracle_sim(cfg, windows=win)
    for F in (1, 63, 64, 65, 130, 4001) + ((20000, 20000) if explicit else ()):
        ctx.run_cycles(1, F)
        oracle_cycle(sim, F)
        compare_state(ctx, 0, sim)


def test_frozen_windows_keep_moving_without_updates():
    cfg = _c(WL.ISING, 8, n_windows=3, lnf_final=0.3)
    ctx, sim = gpu_context([cfg]), oracle_sim(cfg)
    frozen = set()
    for _ in range(40):
        ctx.run_cycles(1, 1000)
        oracle_cycle(sim, 1000)
        st = ctx.status(0)
        frozen.add(int(np.sum(st["frozen"])))
        compare_state(ctx, 0, sim)
        if st["done"]:
            break
    assert frozen & {1, 2}   # some windows froze while others went on


def test_a_fused_batch_of_a_default_plan_takes_the_lane_form():
    """A fused launch runs every class with one lane per walker; back to
    per-class launches the small batch has one wavefront per walker again."""
    cfgs = [_c(WL.ISING, 8, n_windows=2), _c(WL.POTTS, 6, q=3, n_windows=2), _c(WL.ISING, 40, n_windows=2)]
    ctx = gpu_context(cfgs)
    sims = [oracle_sim(c, instance=i) for i, c in enumerate(cfgs)]
    for fused in (0, 1, 0):
        plan = ctx.set_batching(fused=fused)
        groups = [p["walkers_per_group"] for k, p in plan.items() if k != "batching"]
        assert all((g == 1) == (fused == 0) for g in groups), plan
        ctx.run_cycles(2, 777)
        for i, sim in enumerate(sims):
            oracle_cycle(sim, 777)
            oracle_cycle(sim, 777)
            compare_state(ctx, i, sim)


@pytest.mark.parametrize("model,L,q", [(WL.ISING, 18, 2), (WL.POTTS, 18, 5)])
def test_many_walkers_on_lattices_of_more_than_256_sites(model, L, q):
    """Above 4096 walkers such lattices are swept with counts in place of lane
    masks: 65 instances of 64 walkers, the last compared in full."""
    cfg = _c(model, L, q=q, walkers_per_window=64)
    ctx = gpu_context([cfg] * 65)
    (plan,) = ctx.set_launch(walkers_per_group=1).values()
    assert plan["workgroups"] == 65 * 64
    ctx.run_cycles(2, 1500)
    sim = oracle_sim(cfg, instance=64)
    for _ in range(2):
        oracle_cycle(sim, 1500)
    compare_state(ctx, 64, sim)
