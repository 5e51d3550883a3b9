"""The tile kernel's own tile table at the batch sizes where its form changes: up to 64 objects a
wave keeps it in registers, beyond that it lies in LDS, and past about 500 objects without the ray
offsets and object ids. Against the separate work-list launch, bitwise: both sum the same partials
in the same order. Workgroups of one to eight waves, and a grid smaller than the tile count (a
workgroup's later tiles read the table again)."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("n,waves,grid", [(1, 4, 0), (63, 3, 0), (64, 4, 7), (64, 2, 0), (65, 4, 0),
                                          (65, 1, 11), (600, 4, 0), (600, 4, 40)])
def test_table_forms_match_split_launches(precision, n, waves, grid):
    sc = scenes.make_scene("tiny_k4")
    pool = scenes.make_batch(sc, 0, object_ids=[0], n_rays={0: 9 * n + 60})
    counts = (np.arange(n) * 7919) % 10  # zero to nine rays, zero-ray objects among them
    counts[0] = 59                       # several tiles
    counts[-1] += 1
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offs[-1])
    batch = {k: pool[k][:R] for k in ("rays_o", "rays_d", "t", "depth", "rgb", "mask")}
    batch.update(object_ids=np.arange(n, dtype=np.int32)[::-1].copy(), ray_offsets=offs, S=pool["S"])
    sets = []
    for split in (False, True):
        o = vm.ObjectSet(max_objects=n, B=sc.B, precision=precision, max_rays=R + 7,
                         max_samples_per_ray=sc.S, rays_per_tile=24, split_step=split)
        ob = sc.objects[0]
        for k in range(n):
            o.add(ob.norm_centre, ob.norm_scale, seed=1000 + k)
        o.set_launch(waves, grid)
        sets.append(o)
    db = vm.DeviceBatch(batch)
    for _ in range(2):
        losses = [o.step(db).cpu().numpy() for o in sets]
        assert np.array_equal(losses[0], losses[1])
    assert np.all(np.isfinite(losses[0])) and losses[0].sum() > 0
    for k in {0, 1 % n, n // 2, n - 1}:
        for w in (vm.STATE_PARAMS, vm.STATE_ADAM_M, vm.STATE_ADAM_V, vm.STATE_GRAD):
            assert np.array_equal(sets[0].get_state(k, w), sets[1].get_state(k, w)), (k, w)
        assert sets[0].get_state(k, vm.STATE_STEP) == sets[1].get_state(k, vm.STATE_STEP)
    assert sets[0].step_info() == sets[1].step_info()
