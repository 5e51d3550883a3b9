"""Sample depths of a ray are placed by counting smaller keys, or by the sorting network where a
workgroup holds a NaN: both against the oracle's draws, put in order on the host, over rays per
workgroup that fill it exactly and not, ties (sigma 0: every normal sample is t_s) and NaNs."""
import numpy as np
import pytest

import oracle
import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2302_01838_amd as vm  # noqa: E402


def _network(x):
    """Rows of x (padded with +inf to a power of two) through the bitonic network of minima and
    maxima that drop NaNs."""
    S = x.shape[1]
    P = 1 << (S - 1).bit_length()
    v = np.full((x.shape[0], P), np.inf, np.float32)
    v[:, :S] = x
    i = np.arange(P)
    k = 2
    while k <= P:
        j = k // 2
        while j:
            o = v[:, i ^ j]
            v = np.where(((i & j) == 0) == ((i & k) == 0), np.fmin(v, o), np.fmax(v, o))
            j //= 2
        k *= 2
    return v[:, :S]


@pytest.mark.parametrize("S,n_strat", [(1, 0), (2, 1), (3, 3), (20, 10), (20, 0), (31, 7), (64, 32)])
@pytest.mark.parametrize("sigma", [0.0, 0.03])
def test_places(S, n_strat, sigma):
    per = (512 - 63) // S  # rays per workgroup
    sc = scenes.make_scene("tiny_k4")
    objs = vm.ObjectSet(max_objects=1, B=sc.B, hidden=32, max_rays=16, max_samples_per_ray=8)
    for R in (1, per, per + 1, 3 * per - 1):
        rng = np.random.default_rng(R)
        tn = rng.uniform(0.3, 1.0, R).astype(np.float32)
        tf = (tn + rng.uniform(0.5, 3.0, R)).astype(np.float32)
        depth = np.where(rng.uniform(size=R) < 0.8, rng.uniform(tn + 0.1, tf), 0.0).astype(np.float32)
        t = objs.sample_rays(tn, tf, depth, S, n_strat, sigma=sigma, seed=5).cpu().numpy()
        with np.errstate(divide="ignore", invalid="ignore"):
            ref = oracle.depth_guided_samples(tn, tf, depth, S, n_strat, sigma, 5)
        np.testing.assert_allclose(t, ref, rtol=2.5e-7, atol=0)
        # one ray with a NaN start: its stratified samples are NaN, and the other rays' places do not
        # change with the route
        tn[R // 2] = np.nan
        u = objs.sample_rays(tn, tf, depth, S, n_strat, sigma=sigma, seed=5).cpu().numpy()
        others = np.arange(R) != R // 2
        assert np.array_equal(u[others].view(np.uint32), t[others].view(np.uint32))
        if n_strat == S:  # nothing but NaNs and padding: the network's own result
            want = _network(np.full((1, S), np.nan, np.float32))
            np.testing.assert_array_equal(u[R // 2], want[0])
        elif sigma == 0.0:
            ts = depth[R // 2] if depth[R // 2] > 0 else tf[R // 2]
            x = np.full((1, S), ts, np.float32)
            x[0, :n_strat] = np.nan
            np.testing.assert_array_equal(u[R // 2], _network(x)[0])
