"""Bytes that a layered stack's workspace takes per sample row: activations of five layers, with the
deltas of every layer while those nine stay below 64 GiB, and with two buffers of deltas beyond, as
large stacks need."""
import ctypes
import os

import pytest

import paper_2302_01838_amd as vm

pytestmark = pytest.mark.skipif(not os.path.exists(vm.library_path()), reason="library not built")


@pytest.mark.parametrize("hidden", [256, 512, 1024])
def test_bytes_per_row(hidden):
    lib = vm.load_library()
    S = 64
    tile = 1 << 15  # few tiles, so that the rows dominate

    def size(rows):
        cfg = vm.default_config(max_objects=1, hidden=hidden, max_hidden=hidden, max_samples_per_ray=S,
                                max_rays=rows // S, precision=vm.VMAP_BF16, rays_per_tile=tile, rays_per_tile_wide=tile)
        return lib.vmap_workspace_bytes(ctypes.byref(cfg))

    limit = (64 << 30) // (9 * 2 * hidden) // S * S  # rows whose nine layers just fit 64 GiB
    assert size(limit) > 0
    small = 1 << 14
    other = 2 * 16 + 1  # z, dz and the row tiles' losses
    params = 4 * (hidden * 32 + 3 * hidden * hidden)
    for a, b, layers in ((small, limit, 9), (limit + S, 2 * limit, 7)):
        tiles = (b - a) / S / tile + 1
        per_row = (size(b) - size(a)) / (b - a)
        assert 2 * layers * hidden + 32 <= per_row <= 2 * layers * hidden + other + 1.1 * params * tiles / (b - a) + 1
    assert size(limit + S) < size(limit)
