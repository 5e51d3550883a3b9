"""BF16 workgroups of five to eight waves, which have a CU to themselves, at the batch sizes where the
tile table's form changes: in the waves' registers and in LDS (up to 64 objects), in LDS without the
ray offsets and object ids beyond. Against the separate work-list launch, bitwise (the same partials in
the same order), over two steps and with a grid smaller than the tile count, whose workgroups' later
tiles read the table again."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("waves", [5, 8])
@pytest.mark.parametrize("n,grid", [(1, 0), (64, 0), (64, 7), (65, 0), (65, 11)])
def test_wide_workgroups_match_split_launches(waves, n, grid):
    sc = scenes.make_scene("tiny_k4")
    pool = scenes.make_batch(sc, 0, object_ids=[0], n_rays={0: 9 * n + 60})
    counts = (np.arange(n) * 7919) % 10
    counts[0] = 59
    counts[-1] += 1
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offs[-1])
    batch = {k: pool[k][:R] for k in ("rays_o", "rays_d", "t", "depth", "rgb", "mask")}
    batch.update(object_ids=np.arange(n, dtype=np.int32)[::-1].copy(), ray_offsets=offs, S=pool["S"])
    sets = []
    for split in (False, True):
        o = vm.ObjectSet(max_objects=n, B=sc.B, precision="bf16", max_rays=R + 7,
                         max_samples_per_ray=sc.S, rays_per_tile=24, split_step=split)
        for k in range(n):
            o.add(sc.objects[0].norm_centre, sc.objects[0].norm_scale, seed=1000 + k)
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
    assert sets[0].step_info() == sets[1].step_info()
