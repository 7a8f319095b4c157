"""GPU gradient of the surrogate where the training step's tiling changes:
one and several tiles of 64 samples per workgroup, a partial last tile, a last
workgroup with fewer tiles.  The gradient of a batch is the sum of those of
its parts, each part being the batch with the other rays moved off the
sphere: the same bfloat16 products, added in float32 in another order.  Every
partial sum is rounded by 2^-24 of itself, and for terms of random signs the
sum is no smaller than its partial sums' scale: about ten roundings deep,
6e-7 of a layer's norm, tested with 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 64, 65, 129, 256 * 64, 256 * 64 + 1, 3 * 256 * 64 - 70])
def test_gradient_is_the_sum_of_its_parts(n):
    import torch
    import paper_2207_05009_amd as lq
    print(f"[gpu] surrogate gradient by parts, {n} samples", flush=True)
    rng = np.random.default_rng(n)
    o = rng.normal(size=(n, 3))
    o = (o / np.linalg.norm(o, axis=1, keepdims=True) * 3.0).astype(np.float32)
    d = (rng.uniform(-0.8, 0.8, (n, 3)) - o).astype(np.float32)
    rgb = np.exp(rng.uniform(-3, 3, (n, 3))).astype(np.float32)
    sur = lq.Surrogate(seed=3)
    ot, dt, ct = (torch.from_numpy(a).cuda() for a in (o, d, rgb))
    loss, g = sur.grad(ot, dt, ct)
    part = rng.integers(0, 3, n)
    ref, ref_loss = np.zeros(g.numel()), 0.0
    for k in range(3):
        ok = ot.clone()
        ok[torch.from_numpy(part != k).cuda()] = torch.tensor([10.0, 10.0, 10.0], device="cuda")
        dk = dt.clone()
        dk[torch.from_numpy(part != k).cuda()] = torch.tensor([1.0, 0.0, 0.0], device="cuda")
        lk, gk = sur.grad(ok, dk, ct)
        ref += gk.cpu().numpy().astype(np.float64)
        ref_loss += lk
    g = g.cpu().numpy().astype(np.float64)
    assert loss == pytest.approx(ref_loss, rel=1e-5)
    off = 0
    for i, k in ((128, 64), (64, 64), (64, 64), (64, 64), (64, 3)):
        for a, b in ((off, off + i * k), (off + i * k, off + i * k + k)):     # weights, biases
            assert np.linalg.norm(ref[a:b]) > 0
            assert np.linalg.norm(g[a:b] - ref[a:b]) <= 1e-5 * np.linalg.norm(ref[a:b]), (n, a)
        off += i * k + k
