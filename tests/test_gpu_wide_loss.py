"""Losses of the forward pass and of the training step are the same sums, also where two kernels
compute them (hidden 128): a batch's losses before a step, bitwise those the step reports. Tiles of
one sub-tile and of several rounds of four, with ragged ends."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("hidden,precision", [(32, "fp32"), (32, "bf16"), (64, "fp32"), (64, "bf16"), (128, "bf16"),
                                              (256, "bf16"), (512, "bf16")])
@pytest.mark.parametrize("rpt_wide", [0, 3, 24, 96])
def test_forward_and_step_losses_agree(hidden, precision, rpt_wide):
    sc = scenes.make_scene("tiny_k4")
    n_rays = {0: 1, 1: 7, 2: 100, 3: 233}
    objs = vm.ObjectSet(max_objects=4, B=sc.B, hidden=hidden, precision=precision, max_rays=sum(n_rays.values()),
                        max_samples_per_ray=sc.S, rays_per_tile=rpt_wide if hidden == 32 else 0,
                        rays_per_tile_wide=rpt_wide)
    for ob in sc.objects:
        objs.add(ob.norm_centre, ob.norm_scale, seed=ob.seed)
    for s in range(2):
        db = vm.DeviceBatch(scenes.make_batch(sc, s, n_rays=n_rays))
        loss = objs.forward(db, renders=False)[0]
        assert torch.equal(loss.view(torch.int32), objs.step(db).view(torch.int32))
        assert float(loss.min()) > 0
