"""Workgroup slots behind the fitted rays per tile: what a CU holds follows the precision (two waves per
SIMD in BF16, one in FP32) and the tuned wave count. The fitted tiles of a full stack run at once."""
import pytest

from paper_2302_01838_amd.tune import fit_rays_per_tile


@pytest.mark.parametrize("precision,waves,slots", [("bf16", 4, 512), ("bf16", 8, 256), ("bf16", 6, 256),
                                                   ("bf16", 2, 512), ("fp32", 2, 512), ("fp32", 4, 256),
                                                   ("fp32", 3, 256), ("fp32", 1, 512)])
def test_slots_follow_precision_and_waves(precision, waves, slots):
    rnd = 3 * waves  # S = 20
    entry = dict(rays_per_tile=3 * rnd, waves=waves)
    fit = lambda rays, objects: fit_rays_per_tile(entry, 20, rays, objects, precision)
    for m in (1, 2, 3, 4):
        assert fit(rnd * m * (slots - 5), 10) == rnd * m      # exactly the slots
        assert fit(rnd * m * (slots - 5) + 1, 10) == (rnd * (m + 1) if m < 4 else entry["rays_per_tile"])
