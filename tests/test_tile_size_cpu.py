"""Rays per tile from a stack's capacity: the binding's rule over the tuned hidden-32 shape, and the
library's own, seen through the workspace size (a stack's tiles bound its partials)."""
import ctypes
import os

import pytest

import paper_2302_01838_amd as vm
from paper_2302_01838_amd.tune import fit_rays_per_tile


@pytest.mark.parametrize("rays,objects,waves,want", [
    (120, 1, 4, 12), (6000, 50, 4, 24), (6132, 2, 4, 12), (6133, 2, 4, 24), (6145, 2, 4, 24),
    (16368, 50, 4, 36), (17532, 50, 4, 36), (17533, 50, 4, 48), (23376, 50, 4, 48),
    (23377, 50, 4, 36), (1 << 26, 50, 4, 36), (0, 50, 4, 36),
    (120, 1, 2, 6), (16368, 50, 2, 36), (18132, 50, 2, 42), (60000, 50, 2, 36)])
def test_fit_of_the_tuned_tile(rays, objects, waves, want):
    got = fit_rays_per_tile(dict(rays_per_tile=36, waves=waves), 20, rays, objects)
    assert got == want
    rnd = 3 * waves
    assert got % rnd == 0 and got <= 48
    if got != 36:  # a tile that is not the tuned one fits, and no shorter one does
        assert -(-rays // got) + objects // 2 <= 512
        assert got == rnd or -(-rays // (got - rnd)) + objects // 2 > 512


@pytest.mark.skipif(not os.path.exists(vm.library_path()), reason="library not built")
@pytest.mark.parametrize("precision,rays,objects,hidden,want", [
    (vm.VMAP_BF16, 120, 1, 32, 24), (vm.VMAP_BF16, 12000, 24, 32, 24), (vm.VMAP_BF16, 12001, 24, 32, 48),
    (vm.VMAP_BF16, 24024, 24, 32, 72), (vm.VMAP_BF16, 48001, 24, 32, 48), (vm.VMAP_BF16, 120, 1, 16, 24),
    (vm.VMAP_BF16, 120, 1, 64, 48), (vm.VMAP_FP32, 6000, 50, 32, 24), (vm.VMAP_FP32, 7000, 50, 32, 48),
    (vm.VMAP_FP32, 1 << 20, 50, 32, 48)])
def test_library_tile_from_capacity(precision, rays, objects, hidden, want):
    lib = vm.load_library()
    kw = dict(max_objects=objects, hidden=hidden, max_hidden=hidden, max_samples_per_ray=10,
              max_rays=rays, precision=precision, rays_per_tile_wide=want)
    size = lambda rpt: lib.vmap_workspace_bytes(ctypes.byref(vm.default_config(rays_per_tile=rpt, **kw)))
    assert size(0) == size(want) > 0
    for other in (24, 48, 72, 96):
        if hidden != 64 and -(-rays // other) != -(-rays // want):
            assert size(other) != size(0)
