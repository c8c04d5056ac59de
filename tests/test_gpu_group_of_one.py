"""One walker per workgroup (GPU): a lane launch where a page, a producer or a
lattice form is asked for, one wavefront per walker where none is; and what a
plan reports, set again, is the same plan."""
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import compare_state, gpu_context, oracle_cycle, oracle_sim

pytestmark = pytest.mark.gpu


def _c(model, L, **kw):
    return WL.config(model, L, **dict(dict(n_windows=3, walkers_per_window=2, seed=21), **kw))


# lds: 4 B per lattice word and 12 B per page bin of the one walker, 8 B per
# site for the neighbour table, and a producer's two buffers of 16 blocks (16
# B each, at a 16-byte boundary) and flag (16 B)
@pytest.mark.parametrize("cfg,shape,lds", [
    (_c(WL.ISING, 16), dict(page_bins=16), 64 + 192 + 512 + 16),
    (_c(WL.ISING, 32), dict(page_bins=32, rng_producer=0), 128 + 384),
    (_c(WL.ISING, 40, precision=WL.FP32C), dict(page_bins=16, rng_producer=1), 320 + 192 + 512 + 16),
    (_c(WL.POTTS, 8, q=5), dict(page_bins=32, rng_producer=0, potts_nibbles=1), 32 + 384 + 512),
    (_c(WL.POTTS, 8, q=5), dict(page_bins=32, rng_producer=1, potts_nibbles=2), 32 + 384 + 512 + 16),
    (_c(WL.POTTS, 8, q=5), dict(page_bins=32, rng_producer=0, potts_nibbles=0), 64 + 384),
])
def test_a_lane_launch_of_one_walker_per_workgroup(cfg, shape, lds):
    ctx, sim = gpu_context([cfg]), oracle_sim(cfg)
    (plan,) = ctx.set_launch(walkers_per_group=1, **shape).values()
    assert plan["walkers_per_group"] == 1 and plan["workgroups"] == 6, plan
    assert {k: plan[k] for k in shape} == shape, plan
    assert plan["lds_bytes"] == lds, plan
    for _ in range(3):
        ctx.run_cycles(1, 1500)
        oracle_cycle(sim, 1500)
    compare_state(ctx, 0, sim)


@pytest.mark.parametrize("shape", [dict(), dict(walkers_per_group=1), dict(rng_producer=0),
                                   dict(walkers_per_group=1, page_bins=32), "tuned"])
def test_a_reported_plan_set_again_is_the_same_plan(shape):
    cfgs = [_c(WL.ISING, 16), _c(WL.ISING, 36), _c(WL.POTTS, 8, q=5)]
    ctx = gpu_context(cfgs)
    if shape == "tuned":
        ctx.autotune(500)
        plan = ctx.set_batching()
    else:
        plan = ctx.set_launch(**shape)
    wave = dict(page_bins=0, walkers_per_group=1, rng_producer=-1, potts_nibbles=-1)
    if shape in (dict(), dict(walkers_per_group=1)):
        assert all({k: p[k] for k in wave} == wave for p in plan.values()), plan
    ctx.set_launch(page_bins=64, walkers_per_group=3, rng_producer=0, potts_nibbles=0)
    for cls, name in enumerate(ctx.CLASSES):
        again = ctx.set_launch(cls=cls, **{k: plan[name][k] for k in wave})
    assert again == plan
