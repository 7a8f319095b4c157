"""Guided sampling forms a point's faces once per point in LDS when a block of
2048 samples covers few enough points, else once per sample: the same FP64
operations, so a point with S samples and S copies of it with one sample each
give the same terms bit for bit.  Sample counts around the limit (258 points
per block), points split over blocks, more samples than a block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [1, 3])
@pytest.mark.parametrize("n,S", [(1, 1), (700, 7), (600, 8), (520, 9), (300, 13), (3, 2047), (3, 2049), (2, 5000)])
def test_terms_do_not_depend_on_the_grouping(c0_tree, n, S, D):
    import torch
    import paper_2207_05009_amd as lq
    print(f"[gpu] guided samples, {n} points x {S}, {D} x {D} bins", flush=True)
    oct_ = lq.Octree(c0_tree, "f32")
    rng = np.random.default_rng(100 * S + D)
    G = 5
    x = rng.uniform(-3.0, 3.0, (n, 3)).astype(np.float32)      # beside, above, on the axes and inside the box
    x[::5] = rng.uniform(-0.9, 0.9, (len(x[::5]), 3))
    x[1::5, 0] = 1.0                                            # in a face's plane
    nrm = (-x + rng.normal(0.0, 0.4, (n, 3))).astype(np.float32)
    u = rng.random((n, S, 3), dtype=np.float32)
    w = rng.random(6 * G * G * D * D).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()   # noqa: E731
    args = (dev(w), G)
    kw = dict(defensive=0.2, want_terms=True, dir_res=D)
    _, a = oct_.proxy_irradiance_guided(dev(x), dev(nrm), dev(u), *args, **kw)
    _, b = oct_.proxy_irradiance_guided(dev(np.repeat(x, S, 0)), dev(np.repeat(nrm, S, 0)), dev(u.reshape(n * S, 1, 3)),
                                        *args, **kw)
    torch.cuda.synchronize()
    assert torch.equal(a.reshape(-1, 3), b.reshape(-1, 3))
    oct_.free()
