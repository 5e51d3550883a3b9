"""Gradient and loss sums of objects of many tiles, whose partials are spread over extra workgroups
(more than 64 tiles, batches of few objects): the training step, the step with a separate work list,
backward with adam_step, and k_reduce_adam_wide (a stack that may hold hidden-128 objects), which all
add in the same order and must agree bitwise; the objects of few tiles beside them too."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402

RPT = 4
BATCHES = {  # tiles per batch object
    "one": [500], "edges": [64, 65, 66, 32, 33, 128, 129, 257], "last": [3] * 54 + [300], "many": [70] * 20 + [0, 1],
    "past": [2] * 70 + [90]}  # (more rows than the extra ones are worth: not spread)


def _batch(sc, tiles, poison=None):
    counts = [RPT * t - (1 if t > 2 and t % 2 else 0) for t in tiles]
    pool = scenes.make_batch(sc, 0, object_ids=[0], n_rays={0: sum(counts)})
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    batch = {k: pool[k].copy() for k in ("rays_o", "rays_d", "t", "depth", "rgb", "mask")}
    if poison is not None:  # a ray of the object's last tile
        batch["rays_o"][offs[poison + 1] - 1] = np.inf
    batch.update(object_ids=np.arange(len(tiles), dtype=np.int32)[::-1].copy(), ray_offsets=offs, S=pool["S"])
    return batch


def _stack(sc, tiles, precision, hidden, max_hidden=None, **kw):
    o = vm.ObjectSet(max_objects=len(tiles), B=sc.B, hidden=hidden, max_hidden=max_hidden, precision=precision,
                     max_rays=RPT * sum(tiles), max_samples_per_ray=sc.S, rays_per_tile=RPT, **kw)
    for k in range(len(tiles)):
        o.add(sc.objects[0].norm_centre, sc.objects[0].norm_scale, hidden=hidden, seed=7 + k)
    return o


@pytest.mark.parametrize("precision,hidden", [("fp32", 32), ("bf16", 32), ("bf16", 16)])
@pytest.mark.parametrize("name", list(BATCHES))
def test_spread_sums_agree(name, precision, hidden):
    sc, tiles = scenes.make_scene("tiny_k4"), BATCHES[name]
    db = vm.DeviceBatch(_batch(sc, tiles))
    sets = [_stack(sc, tiles, precision, hidden), _stack(sc, tiles, precision, hidden, split_step=True),
            _stack(sc, tiles, precision, hidden)]
    if precision == "bf16":
        sets.append(_stack(sc, tiles, precision, hidden, max_hidden=128, split_step=True, rays_per_tile_wide=RPT))
    n = len(tiles)
    for _ in range(2):
        losses = [o.step(db) for o in sets[:2] + sets[3:]]
        split = sets[2]
        losses.append(split.forward(db, renders=False)[0])
        grad = split.backward(db, torch.ones(n)).cpu().numpy()
        split.adam_step(db)
        for x in losses[1:]:
            assert torch.equal(losses[0].view(torch.int32), x.view(torch.int32))
        for j in range(n):
            k = n - 1 - j
            g = split.get_state(k, vm.STATE_GRAD)
            assert np.array_equal(grad[j, : g.size], g) and not grad[j, g.size:].any()
    for k in range(n):
        rays = tiles[n - 1 - k] > 0
        for w in (vm.STATE_GRAD, vm.STATE_PARAMS, vm.STATE_ADAM_M, vm.STATE_ADAM_V):
            states = [o.get_state(k, w) for o in sets]
            assert all(np.array_equal(states[0], s) for s in states[1:]), (k, w)
            assert np.any(states[0]) == rays or w == vm.STATE_PARAMS
        assert {o.get_state(k, vm.STATE_STEP) for o in sets} == {2 if rays else 0}
    # the weight images followed: a query reads them
    pts = np.random.default_rng(0).uniform(-0.3, 0.3, (100, 3)).astype(np.float32) + sc.objects[0].norm_centre
    q = [o.query(0, pts)[0] for o in sets]
    assert all(torch.equal(q[0], x) for x in q[1:])


@pytest.mark.parametrize("split_step", [False, True])
def test_skip_of_a_spread_object(split_step):
    """An object of many tiles whose last tile is not finite is skipped whole and counted once."""
    sc, tiles = scenes.make_scene("tiny_k4"), [70, 3, 200, 100]
    good, bad = _batch(sc, tiles), _batch(sc, tiles, poison=2)
    sets = [_stack(sc, tiles, "bf16", 32, split_step=split_step) for _ in range(2)]
    for o, b in zip(sets, (good, bad)):
        o.step(vm.DeviceBatch(b))
    assert sets[1].step_info()[1] == 1 and sets[0].step_info()[1] == 0
    for j in range(4):
        k = 3 - j
        steps = [o.get_state(k, vm.STATE_STEP) for o in sets]
        assert steps == [1, 0 if j == 2 else 1]
        same = np.array_equal(*[o.get_state(k, vm.STATE_PARAMS) for o in sets])
        assert same == (j != 2)
