"""Layered products at the batch sizes between one and two rounds of 256 x 256 blocks on the chip's CUs,
where the block size changes from wide to narrow and back: an object's losses, renders, gradient and
state are bitwise those it has alone (narrow blocks), at hidden 512 and 1024."""
import dataclasses

import numpy as np
import pytest

import scenes
from vmap_testlib import same_state, snapshot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("hidden,rays,objects", [(512, 1600, 3), (512, 1984, 3), (512, 2600, 3), (512, 103, 20),
                                                 (1024, 1380, 2), (1024, 1750, 2), (1024, 2100, 2)])
def test_rows_of_one_and_two_rounds(hidden, rays, objects):
    base = scenes.make_scene("k50_uneven")
    sc = dataclasses.replace(base, S=9, n_strat=4,
                             objects=[dataclasses.replace(o, hidden=hidden) for o in base.objects[:objects]])
    n_rays = {k: rays for k in range(objects)}
    n_rays[0] = 37
    runs = []
    for members in ([0], list(range(objects))):
        objs = vm.ObjectSet(max_objects=objects, B=sc.B, hidden=hidden, precision="bf16",
                            max_rays=sum(n_rays.values()), max_samples_per_ray=sc.S)
        for ob in sc.objects:
            objs.add(ob.norm_centre, ob.norm_scale, seed=ob.seed)
        db = vm.DeviceBatch(scenes.make_batch(sc, 0, object_ids=members, n_rays={k: n_rays[k] for k in members}))
        renders = [x[: n_rays[0]].cpu().numpy() for x in objs.render(db)]
        loss = objs.step(db).cpu().numpy()[:1]
        runs.append(renders + [loss, objs.get_state(0, vm.STATE_GRAD)] + snapshot(objs, [0])[0])
    for a, b in zip(*runs):
        assert same_state([a], [b])
    assert np.any(runs[0][4])
