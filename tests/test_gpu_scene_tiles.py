"""Scene rendering at the sizes where its layouts change: the pairs of images of 32 rays or fewer (one
word of bits per object, the scanned counts in place of bases), of more objects than a workgroup of the
pair kernels takes (64), and the tile length, which follows the pairs found. A ray's render does not
depend on its tile, so stacks of other tiles and capacities give the same image bitwise; the pairs
are those of the FP64 slab test whatever the FP32 test before it settles."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402

B = (np.random.default_rng(3).standard_normal((3, 16)) * 4).astype(np.float32)


def _objects(n):
    rng = np.random.default_rng(n)
    return rng.uniform(-2, 2, (n, 3)).astype(np.float32), rng.uniform(0.2, 0.9, n).astype(np.float32)


def _rays(R, centres):
    """Rays from points around towards the objects' centres, in turn."""
    rng = np.random.default_rng(R)
    o = rng.uniform(-4, 4, (R, 3))
    d = centres[np.arange(R) % len(centres)] + rng.uniform(-0.3, 0.3, (R, 3)) * (np.arange(R)[:, None] > 0) - o
    return o.astype(np.float32), (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)


def _stack(n, precision, max_rays, **kw):
    c, s = _objects(n)
    o = vm.ObjectSet(max_objects=n, B=B, precision=precision, max_rays=max_rays, max_samples_per_ray=20, **kw)
    for k in range(n):
        o.add(c[k], float(s[k]), seed=k)
    return o


def _bits(out):
    return [x.cpu().numpy().view(np.uint32) for x in out]


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("R,n", [(1, 3), (31, 40), (32, 65), (33, 65), (64, 130), (257, 64), (20000, 9), (60000, 65)])
def test_image_does_not_depend_on_the_tiles(precision, R, n):
    c, s = (x.astype(np.float64) for x in _objects(n))
    ro, rd = _rays(R, c)
    hits = [t1 > np.maximum(t0, 0.0) for t0, t1 in
            (oracle.ray_box(ro, rd, c[k] - s[k], c[k] + s[k]) for k in range(n))]
    pairs = int(sum(h.sum() for h in hits))
    assert pairs > 0
    cases = [dict(max_rays=4 * max(pairs, 16)), dict(max_rays=1 << 20), dict(max_rays=pairs, rays_per_tile=36),
             dict(max_rays=pairs, rays_per_tile=1), dict(max_rays=2 * pairs, rays_per_tile=1000)]
    first = None
    for kw in cases:
        objs = _stack(n, precision, **kw)
        out = objs.render_scene(ro, rd, S=20, occ_threshold=0.2)
        assert int(out[4]) == pairs, kw
        assert objs.step_info()[2] == 0
        if kw.get("rays_per_tile") == 36:  # other launch shapes
            objs.set_launch(2, 5)
            assert all(np.array_equal(a, b) for a, b in zip(_bits(out), _bits(objs.render_scene(ro, rd, S=20, occ_threshold=0.2))))
        first = first or _bits(out)
        assert all(np.array_equal(a, b) for a, b in zip(first, _bits(out))), kw
    # a ray without a pair has no object, and a pick is one of the ray's pairs
    kid = first[3].view(np.int32)
    met = np.stack(hits)
    assert np.all(kid[~met.any(0)] == -1)
    assert np.all(met[kid[kid >= 0], np.nonzero(kid >= 0)[0]])


def test_pairs_of_grazing_and_axis_parallel_rays():
    """Rays along the axes, in the faces' planes, through edges and a rounding step beside them, from
    inside and on a face, with zero, denormal and huge direction components."""
    c, s = (x.astype(np.float64) for x in _objects(5))
    f32 = np.float32
    o, d = [], []
    for k in range(5):
        for a in range(3):
            for face in (c[k, a] - s[k], c[k, a] + s[k], c[k, a]):
                for q in (f32(face), np.nextafter(f32(face), f32(9)), np.nextafter(f32(face), f32(-9))):
                    for b in range(3):
                        for sign in (1.0, -1.0):
                            for tilt in (0.0, 1e-40, 1e-7, 1e3):
                                p = c[k].astype(f32)
                                p[a] = q
                                e = np.zeros(3, f32)
                                e[b] = sign
                                e[(b + 1) % 3] = tilt
                                far = p.copy()
                                far[b] -= f32(3 * sign)
                                o += [p, far]
                                d += [e, e]
    o, d = np.stack(o), np.stack(d)
    objs = _stack(5, "fp32", 1 << 17)
    for t_min in (0.0, 0.1, 2.5):
        t_min = float(f32(t_min))
        want = 0
        for k in range(5):
            with np.errstate(all="ignore"):
                t0, t1 = oracle.ray_box(o, d, c[k] - s[k], c[k] + s[k])
            want += int((t1 > np.maximum(t0, t_min)).sum())
        out = objs.render_scene(o, d, S=4, t_min=t_min)
        assert int(out[4]) == want > 0
