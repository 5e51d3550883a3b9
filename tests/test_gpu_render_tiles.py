"""Rendering without losses takes tiles of its own, by the batch's rays: the renders are bitwise those of
the forward pass with losses, whose tiles are the training step's, in stacks of any capacity and tile,
with hidden 16 and wider objects beside hidden 32 and any launch shape."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("S,rays", [(1, 3), (7, 700), (10, 61), (33, 500), (64, 2600)])
@pytest.mark.parametrize("kw", [dict(), dict(max_rays=1 << 16), dict(rays_per_tile=5), dict(rays_per_tile=1000),
                                dict(hidden=64), dict(waves=1), dict(waves=3, grid=5)], ids=str)
def test_renders_are_those_of_the_forward_pass(precision, S, rays, kw):
    kw = dict(kw)
    waves, grid = kw.pop("waves", 4), kw.pop("grid", 0)
    hidden = kw.pop("hidden", 32)
    rng = np.random.default_rng(S)
    counts = np.array([rays, 0, rays // 3, 1, 17])
    R = int(counts.sum())
    d = rng.standard_normal((R, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    batch = dict(object_ids=np.array([4, 1, 0, 3, 2], np.int32), S=S,
                 ray_offsets=np.concatenate([[0], np.cumsum(counts)]).astype(np.int32),
                 rays_o=(rng.uniform(-0.2, 0.2, (R, 3)) - 1.5 * d).astype(np.float32), rays_d=d.astype(np.float32),
                 t=np.sort(rng.uniform(0.5, 2.5, (R, S)), 1).astype(np.float32),
                 depth=rng.uniform(1, 2, R).astype(np.float32), rgb=rng.uniform(0, 1, (R, 3)).astype(np.float32),
                 mask=np.ones(R, np.float32))
    kw.setdefault("max_rays", R)
    objs = vm.ObjectSet(max_objects=5, B=scenes.make_scene("tiny_k4").B, hidden=16, max_hidden=hidden, precision=precision,
                        max_samples_per_ray=S, autotune=False, **kw)
    for k in range(5):
        objs.add((0, 0, 0), 1.0, hidden=(32, 16, hidden, 32, hidden)[k], seed=k)
    objs.set_launch(waves, grid)
    db = vm.DeviceBatch(batch)
    loss, *want = objs.forward(db)
    assert float(loss.max()) > 0
    for a, b in zip(want, objs.render(db)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert objs.step_info()[2] == 0
    assert torch.equal(loss, objs.step(db))
