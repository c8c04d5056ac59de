"""The sweep forms against each other where attempt numbers are unusual (GPU).

The lane form takes the attempt number as wave-uniform and handles two of the
Philox rounds apart for each upper half of it; the producer and wavefront
forms compute every block in full.  Across 2^32 attempts, and from a state
whose walkers have made different numbers of attempts (no run gives one),
all forms must end in the same state, bit for bit.
"""
import numpy as np
import pytest

from paper_1402_2328_amd import workloads as WL
from tests.parity import gpu_context, gpu_digest

pytestmark = pytest.mark.gpu

F0 = 1543
CASES = {
    "ising_L32": WL.config(WL.ISING, 32, n_windows=4, walkers_per_window=20, seed=3),
    "ising_L12_fp32c": WL.config(WL.ISING, 12, n_windows=2, walkers_per_window=7, seed=3, precision=WL.FP32C),
    "ising_L40": WL.config(WL.ISING, 40, n_windows=3, walkers_per_window=5, seed=3),
    "potts_q5_L10": WL.config(WL.POTTS, 10, q=5, n_windows=3, walkers_per_window=11, seed=3),
}
FORMS = {"lanes": dict(page_bins=32, rng_producer=0), "lanes_of_5": dict(walkers_per_group=5, rng_producer=0),
         "producer": dict(rng_producer=1), "wavefronts": dict(walkers_per_group=1)}


def _with_attempts(blob, walkers, values):
    """The checkpoint with the walkers' attempt numbers (found as the run of
    `walkers` 64-bit words equal to F0) replaced."""
    words = blob[: len(blob) // 8 * 8].view(np.uint64).copy()
    hit = np.flatnonzero(words == F0)
    runs = [i for i in hit if np.array_equal(words[i:i + walkers], np.full(walkers, F0, np.uint64))]
    assert len(runs) == 1
    words[runs[0]:runs[0] + walkers] = values
    return np.concatenate([words.view(np.uint8), blob[len(words) * 8:]])


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("what", ["across 2^32", "differing"])
def test_forms_agree(name, what):
    cfg = CASES[name]
    walkers = cfg["n_windows"] * cfg["walkers_per_window"]
    ctx = gpu_context([cfg])
    ctx.run_sweeps(F0)
    start = 2 ** 32 - 500
    values = np.full(walkers, start, np.uint64)
    if what == "differing":
        values += (np.arange(walkers) % 3 * 250).astype(np.uint64)
    blob = _with_attempts(ctx.checkpoint(), walkers, values)
    ctx.close()
    got = {}
    for form, shape in FORMS.items():
        c = gpu_context([cfg])
        c.set_launch(**shape)
        c.restore(blob)
        for flips in (499, 2, 1001):
            c.run_sweeps(flips)
        assert c.get_walker(0, walkers - 1)["attempts"] == int(values[-1]) + 1502
        got[form] = gpu_digest(c, 0)
        c.close()
    assert len(set(got.values())) == 1, got
