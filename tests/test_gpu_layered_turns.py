"""A layered stack of so large a capacity that its deltas take two buffers in turn, each layer's weight
gradient launched by itself (and hidden 256 without its one-launch chain): losses, renders, gradients
and states bitwise those of a small stack, in training steps and through the autograd split."""
import numpy as np
import pytest

import scenes
from vmap_testlib import same_state, scaled, snapshot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("hidden,max_rays", [(256, 234000), (512, 117000), (1024, 58500)])
def test_two_delta_buffers(hidden, max_rays):
    """(about 55 GB of workspace: nine layers would pass 64 GiB)"""
    sc = scaled(scenes.make_scene("k50_uneven"), 6)
    ids = list(range(7))
    n_rays = {k: (1, 13, 64, 100, 257, 3, 40)[k] for k in ids}
    runs = []
    for cap in (512, max_rays):
        objs = vm.ObjectSet(max_objects=8, B=sc.B, hidden=hidden, max_hidden=hidden, precision="bf16", max_rays=cap,
                            max_samples_per_ray=64, rays_per_tile=24, rays_per_tile_wide=24)
        for k in ids:
            # a hidden-32 object beside the layered ones
            objs.add(sc.objects[k].norm_centre, sc.objects[k].norm_scale, hidden=32 if k == 3 else hidden, seed=k)
        out = []
        for s in range(2):
            db = vm.DeviceBatch(scenes.make_batch(sc, s, object_ids=ids, n_rays=n_rays))
            out += [x.cpu().numpy() for x in objs.forward(db)]
            out.append(objs.step(db).cpu().numpy())
            out += [objs.get_state(k, vm.STATE_GRAD) for k in ids]
            out.append(objs.backward(db, torch.ones(len(ids))).cpu().numpy())
            objs.adam_step(db)
        runs.append((out, snapshot(objs, ids), objs.workspace.numel()))
        objs.close()
        del objs
        torch.cuda.empty_cache()
    (a, sa, small), (b, sb, large) = runs
    assert large > 50 << 30 and small < 1 << 30
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    assert all(same_state(sa[k], sb[k]) for k in ids)
