"""Copies that fill the chip (GPU): a property of the configuration and the
LDS, whatever page a lone instance has by default."""
import pytest

from paper_1402_2328_amd import workloads as WL

pytestmark = pytest.mark.gpu


# LDS of a workgroup of 64 walkers against 160 KiB per compute unit, 256 units
@pytest.mark.parametrize("cfg,copies", [
    (WL.POTTS_Q10_L20, 128),        # 64 (200 + 12 x 32) + 3200 B: 4 fit; 8 workgroups
    (WL.POTTS_Q10_L20_FP32C, 128),
    (WL.ISING_L32, 640),            # 64 (128 + 12 x 32) B: 5 fit, page 64 only 2; 2 workgroups
    (WL.config(WL.ISING, 64, n_windows=16, walkers_per_window=8), 384),    # 64 (512 + 12 x 16) B: 3
    (WL.config(WL.POTTS, 64, q=20, n_windows=16, walkers_per_window=8), 64),  # less than 64 walkers fit
])
def test_bench_replicas(cfg, copies):
    assert WL.bench_replicas(cfg) == copies
