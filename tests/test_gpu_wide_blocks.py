"""256 x 256 product blocks of the layered path (taken by batches of many rows) against the 128 x 128
blocks (taken by the same objects alone): losses, gradients and states bit for bit, at row counts
around the blocks' edges and the 64-row chunks of the weight gradients."""
import dataclasses

import numpy as np
import pytest

import scenes
from vmap_testlib import make_pair, same_state, snapshot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("S,rays", [(1, [1, 63, 64, 65, 127, 129, 255, 256, 257, 511, 513]),
                                    (7, [1, 9, 10, 18, 36, 37, 73, 74, 147])])
def test_wide_blocks_equal_narrow_ones(S, rays):
    print(f"[wide blocks] S={S}", flush=True)
    base = scenes.make_scene("k50_uneven")
    sc = dataclasses.replace(base, S=S, n_strat=max(1, S // 2),
                             objects=[dataclasses.replace(o, hidden=512) for o in base.objects])
    n_rays = {k: (rays[k] if k < len(rays) else 500) for k in range(sc.n_objects)}
    ids = list(range(len(rays)))
    runs = []
    for members in (ids, list(range(sc.n_objects))):
        objs, _ = make_pair(sc, "bf16", max_rays=sum(n_rays.values()))
        batch = scenes.make_batch(sc, 0, object_ids=members, n_rays={k: n_rays[k] for k in members})
        loss = objs.step(vm.DeviceBatch(batch)).cpu().numpy()[: len(ids)]
        runs.append((loss, [objs.get_state(k, vm.STATE_GRAD) for k in ids], snapshot(objs, ids)))
    (la, ga, sa), (lb, gb, sb) = runs
    assert np.array_equal(la.view(np.uint32), lb.view(np.uint32))
    for k in ids:
        assert np.any(ga[k]) and np.array_equal(ga[k].view(np.uint32), gb[k].view(np.uint32)), k
        assert same_state(sa[k], sb[k]), k
