"""Loading, building and reading back a tree on a card that holds little beside
it: none needs device memory in proportion to the float32 values of all leaves,
and a tree without room for its brick tables answers without them."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

MB = 1 << 20


class Filled:
    """The card's memory taken, but for about `free` bytes, while in scope."""

    def __init__(self, free):
        self.free = free

    def __enter__(self):
        import torch
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        self.held, piece = [], 16 << 30
        while piece >= 2 * MB:
            left = torch.cuda.mem_get_info()[0] - self.free
            if left < piece:
                piece //= 2
                continue
            try:
                self.held.append(torch.empty(piece, dtype=torch.uint8, device="cuda"))
            except torch.cuda.OutOfMemoryError:
                piece //= 2
        print(f"[gpu] {torch.cuda.mem_get_info()[0] / MB:.0f} MB of the card left", flush=True)
        return self

    def __exit__(self, *exc):
        import torch
        del self.held
        torch.cuda.empty_cache()


def test_download_needs_no_room_for_the_whole_result():
    import torch
    from paper_2207_05009_amd import lumiq
    n, g = 3 << 20, torch.Generator(device="cuda").manual_seed(5)
    codes = torch.arange(n, dtype=torch.int32, device="cuda") * 5     # below 8^8
    sigma, sh = torch.rand(n, generator=g, device="cuda"), torch.randn((n, 3, 9), generator=g, device="cuda")
    tree = lumiq.octree_from_leaves(8, 2, codes, sigma, sh, storage="f32")
    before = (sigma.cpu().numpy(), sh.cpu().numpy())                  # 340 MB of values
    del codes, sigma, sh
    with Filled(200 * MB):
        out = tree.download()
    assert np.array_equal(out["sigma"], before[0]) and np.array_equal(out["sh"], before[1])
    tree.free()


def test_load_needs_no_room_for_a_copy_of_the_leaves():
    import torch
    from paper_2207_05009_amd import lumiq
    t = inputs.random_tree(7, 0.5, seed=3, sh_degree=4)               # 1.05M leaves: 512 MB of rows, 304 MB of values
    tables = 64 * len(t.child) + 2048 * 4096                          # both child tables, bricks
    with Filled(512 * t.n_leaves + tables + 150 * MB):
        tree = lumiq.Octree(t, "f32")
        out = tree.download()
    assert np.array_equal(out["sigma"], t.sigma) and np.array_equal(out["sh"].reshape(t.sh.shape), t.sh)
    tree.free()


def test_build_gives_its_scratch_back_before_the_rows():
    import torch
    from paper_2207_05009_amd import lumiq
    n, g = 3 << 20, torch.Generator(device="cuda").manual_seed(6)
    codes = torch.arange(n, dtype=torch.int32, device="cuda") * 5
    sigma, sh = torch.rand(n, generator=g, device="cuda"), torch.randn((n, 3, 9), generator=g, device="cuda")
    tree = lumiq.octree_from_leaves(8, 2, codes, sigma, sh)           # 403 MB of rows; 120 MB of scratch before them
    need, ref = tree.info()["device_bytes"], tree.download()
    tree.free()
    with Filled(need + 50 * MB):
        tree = lumiq.octree_from_leaves(8, 2, codes, sigma, sh)
    out = tree.download()
    assert all(np.array_equal(out[k], ref[k]) for k in ref)
    tree.free()


def test_tree_without_room_for_bricks_answers_the_same():
    """600,000 leaves scattered over depth 10, nearly each in a brick of its own:
    1.2 GB of bricks beside 0.2 GB of other tables.  The octree march visits the
    same leaves over the same segments; only a segment that starts at an edge or a
    corner may round differently, within a few float32 ulp of each of its terms."""
    import torch
    from paper_2207_05009_amd import lumiq
    g = torch.Generator(device="cuda").manual_seed(8)
    codes = torch.unique(torch.randint(0, 1 << 30, (600000,), generator=g, device="cuda")).to(torch.int32)
    n = codes.numel()
    sigma = torch.rand(n, generator=g, device="cuda") * 60.0
    sh = torch.randn((n, 3, 9), generator=g, device="cuda")
    bricks = 2048 * torch.unique(codes >> 9).numel()
    trees = [lumiq.octree_from_leaves(10, 2, codes, sigma, sh, storage="f16")]
    need = trees[0].info()["device_bytes"] - bricks
    with Filled(need + 300 * MB):
        trees.append(lumiq.octree_from_leaves(10, 2, codes, sigma, sh, storage="f16"))
        assert trees[1].info()["device_bytes"] <= need
    o, d = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in inputs.rays.room_to_proxy(1 << 18, 9))
    u = torch.rand((4096, 8, 3), generator=g, device="cuda")
    up = torch.tensor([0.0, 0.0, 1.0], device="cuda").expand(4096, 3).contiguous()
    p = torch.rand((4096, 3), generator=g, device="cuda") * 4.0 - 2.0
    p[:, 2] = -1.5
    for model in ("linear", "exp"):
        res = [[*t.query(o, d, model=model), *t.query_image(o, d, 512, 512, model=model),
                *lumiq.query_multi([t, t, trees[0]], [0, 1000, 1000, 1 << 18], o, d, model=model),
                t.proxy_irradiance(p, up, u, model=model)[0]] for t in trees]
        torch.cuda.synchronize()
        for a, b in zip(*res):
            assert float(a.sum()) > 0
            assert float((a == b).float().mean()) > 0.999 and torch.allclose(a, b, rtol=1e-5, atol=1e-6)
    for t in trees:
        t.free()
