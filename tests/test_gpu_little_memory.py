"""Loading and reading back a tree on a card that holds little beside it: neither
needs device memory in proportion to the float32 values of all leaves."""
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
        self.held = []
        while torch.cuda.mem_get_info()[0] > self.free + 4 * MB:
            left = torch.cuda.mem_get_info()[0] - self.free
            self.held.append(torch.empty(min(left, 16 << 30) // (2 * MB) * 2 * MB or 2 * MB, dtype=torch.uint8,
                                         device="cuda"))
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
