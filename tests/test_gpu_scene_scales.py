"""The pairs of a scene are those of the FP64 slab test in any units: scenes and directions scaled so that
the FP32 test before it meets denormal and vanishing products, and overflowing ones."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


@pytest.mark.parametrize("size", [1e-42, 1e-38, 1e-30, 1e-20, 1e-6, 1.0, 1e15, 1e30])
@pytest.mark.parametrize("speed", [1e-38, 1e-20, 1.0, 1e20, 1e37])
def test_pairs_in_any_units(size, speed):
    rng = np.random.default_rng(5)
    n, R = 12, 700
    with np.errstate(all="ignore"):
        c = (rng.uniform(-2, 2, (n, 3)) * size).astype(np.float32)
        s = np.maximum((rng.uniform(0.1, 0.8, n) * size).astype(np.float32), np.float32(1e-45))
        o = (rng.uniform(-3, 3, (R, 3)) * size).astype(np.float32)
        d = rng.uniform(-0.7, 0.7, (R, 3)) - o / size
        d = (d / np.linalg.norm(d, axis=1, keepdims=True) * speed).astype(np.float32)
    d[rng.uniform(size=(R, 3)) < 0.05] = 0
    objs = vm.ObjectSet(max_objects=n, B=np.ones((3, 16), np.float32), max_rays=n * R, max_samples_per_ray=4)
    want = 0
    for k in range(n):
        objs.add(c[k], float(s[k]), seed=k)
        # (the library's half extent is the reciprocal of the reciprocal it keeps)
        h = 1.0 / (1.0 / np.float64(s[k]))
        with np.errstate(all="ignore"):
            t0, t1 = oracle.ray_box(o, d, c[k].astype(np.float64) - h, c[k].astype(np.float64) + h)
        want += int((t1 > np.maximum(t0, 0.0)).sum())
    out = objs.render_scene(o, d, S=2)
    assert int(out[4]) == want > 0
