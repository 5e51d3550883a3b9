"""Stop and resume in a stack of another capacity (Sec. 3.2): a checkpoint of a stack sized for its
objects, restored into a larger one (a map that grows) or a larger one's into a smaller, continues
bitwise as the first would have. An object's gradient is summed tile by tile, and the default tile
follows capacity, so the checkpoint carries the tile sizes. A stack created with its own keeps them."""
import numpy as np
import pytest

import scenes
from vmap_testlib import same_state, scaled, snapshot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402

LARGE = dict(max_objects=200, max_rays=1 << 17)


def _scene():
    sc = scaled(scenes.make_scene("k50_uneven"), 10)
    return sc, [scenes.make_batch(sc, s) for s in range(4)]


def _stack(sc, precision, widths, capacity, **kw):
    o = vm.ObjectSet(B=sc.B, precision=precision, hidden=min(widths), max_hidden=max(widths),
                     max_samples_per_ray=sc.S, **capacity, **kw)
    for i, ob in enumerate(sc.objects):
        o.add(ob.norm_centre, ob.norm_scale, hidden=widths[i % len(widths)], seed=ob.seed)
    return o


def _resume(tmp_path, sc, batches, first, second, graph=False):
    """Steps 1-2 in `first`, 3-4 in both from there; whether losses and states stay equal."""
    for b in batches[:2]:
        first.step(vm.DeviceBatch(b))
    path = str(tmp_path / "ckpt.npz")
    first.save(path)
    second.step(vm.DeviceBatch(batches[3]))  # a stack in use, whose launches and graphs exist
    second.set_graph_mode(graph)
    second.step(vm.DeviceBatch(batches[3]))
    second.load(path)
    for b in batches[2:]:
        db = vm.DeviceBatch(b)
        if not torch.equal(first.step(db).view(torch.int32), second.step(db).view(torch.int32)):
            return False
    ids = range(sc.n_objects)
    a, b = snapshot(first, ids), snapshot(second, ids)
    return all(same_state(a[k], b[k]) for k in ids)


@pytest.mark.parametrize("precision,widths", [("fp32", (32,)), ("bf16", (32,)), ("bf16", (16, 32)),
                                              ("fp32", (64,)), ("bf16", (32, 64)), ("bf16", (32, 128)),
                                              ("bf16", (256,))])
@pytest.mark.parametrize("grow", [True, False])
def test_resume_in_another_capacity(tmp_path, precision, widths, grow):
    sc, batches = _scene()
    small = dict(max_objects=sc.n_objects, max_rays=max(b["ray_offsets"][-1] for b in batches))
    first, second = (_stack(sc, precision, widths, c) for c in ((small, LARGE) if grow else (LARGE, small)))
    tiles = first.tiles
    same = _resume(tmp_path, sc, batches, first, second, graph=grow)
    assert same
    n = 2 if max(widths) > 32 else 1  # (a stack without wide objects has no wide tile to hand on)
    assert second.tiles[:n] == tiles[:n] and first.tiles == tiles


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_resume_with_pinned_tiles(tmp_path, precision):
    sc, batches = _scene()
    small = dict(max_objects=sc.n_objects, max_rays=max(b["ray_offsets"][-1] for b in batches))
    first, second = (_stack(sc, precision, (32,), c, rays_per_tile=24) for c in (small, LARGE))
    same = _resume(tmp_path, sc, batches, first, second)
    assert same
    other = _stack(sc, precision, (32,), LARGE, rays_per_tile=36)
    other.load(str(tmp_path / "ckpt.npz"))
    assert other.tiles[0] == 36


def test_checkpoint_without_tiles_loads(tmp_path):
    sc, batches = _scene()
    first = _stack(sc, "fp32", (32,), dict(max_objects=sc.n_objects, max_rays=4096))
    first.step(vm.DeviceBatch(batches[0]))
    path = str(tmp_path / "ckpt.npz")
    first.save(path)
    with np.load(path) as z:
        np.savez(path, **{k: z[k] for k in z.files if k != "rays_per_tile"})
    second = _stack(sc, "fp32", (32,), LARGE)
    tiles = second.tiles
    second.load(path)
    assert second.tiles == tiles
    ids = range(sc.n_objects)
    a, b = snapshot(first, ids), snapshot(second, ids)
    assert all(np.array_equal(a[k][0], b[k][0]) for k in ids)


def test_narrow_checkpoint_leaves_a_wide_stacks_wide_tile(tmp_path):
    sc, batches = _scene()
    small = dict(max_objects=sc.n_objects, max_rays=max(b["ray_offsets"][-1] for b in batches))
    first = _stack(sc, "bf16", (32,), small)
    wide = vm.ObjectSet(B=sc.B, precision="bf16", hidden=32, max_hidden=128, max_samples_per_ray=sc.S, **LARGE)
    for ob in sc.objects:
        wide.add(ob.norm_centre, ob.norm_scale, hidden=32, seed=ob.seed)
    tile = wide.tiles[1]
    same = _resume(tmp_path, sc, batches, first, wide)
    assert same and wide.tiles == (first.tiles[0], tile)
