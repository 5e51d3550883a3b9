"""Objects of more tiles than a gradient sum takes in one run (32): the optimiser kernels sum four
quarters of an object's tiles, each in a kernel of its own shape, and must agree bitwise. The fused
training step against backward and adam_step, for a stack of hidden 32 (one parameter per thread)
and one with a hidden-128 object beside a hidden-32 one (units of k_reduce_adam_wide)."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("hidden", [32, 128])
@pytest.mark.parametrize("tiles", [1, 32, 33, 35, 36, 100])
def test_step_equals_split_for_many_tiles(hidden, tiles):
    sc = scenes.make_scene("tiny_k4")
    rays = 24 * tiles - 5
    batch = scenes.make_batch(sc, 0, object_ids=[0, 1], n_rays={0: rays, 1: 30})
    db = vm.DeviceBatch(batch)
    sets = []
    for _ in range(2):
        o = vm.ObjectSet(max_objects=2, B=sc.B, hidden=32, max_hidden=hidden, precision="bf16",
                         max_rays=rays + 30, max_samples_per_ray=sc.S, rays_per_tile=24,
                         rays_per_tile_wide=24)
        for k, h in enumerate((hidden, 32)):
            o.add(sc.objects[k].norm_centre, sc.objects[k].norm_scale, hidden=h, seed=7 + k)
        sets.append(o)
    step, split = sets
    for _ in range(2):
        l1 = step.step(db).cpu().numpy()
        l2 = split.forward(db, renders=False)[0].cpu().numpy()
        split.backward(db, torch.ones(2))
        split.adam_step(db)
        assert np.allclose(l1, l2, rtol=1e-6)  # (hidden 128 renders in another kernel)
        for k in range(2):
            for w in (vm.STATE_GRAD, vm.STATE_PARAMS, vm.STATE_ADAM_M, vm.STATE_ADAM_V):
                a, b = step.get_state(k, w), split.get_state(k, w)
                assert np.array_equal(a, b), (k, w)
            assert np.any(step.get_state(k, vm.STATE_GRAD))
