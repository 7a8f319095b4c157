"""A tree whose leaf rows hold more than 2^32 words (57 million leaves, float32,
SH degree 4: 128 words a row, 76 of them values): it loads, its last leaves
answer as they do in a tree of their own, and its densities come back."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LAST = 4096                      # the leaves of a cube of 16^3 cells
N = 13916 * LAST                 # 57.0M; 76 N > 2^32


def test_tree_of_more_than_2_to_32_words():
    import torch
    from paper_2207_05009_amd import lumiq
    assert 76 * N > 2 ** 32
    print(f"[gpu] {N} leaves of degree 4, {N * 512 / 2 ** 30:.1f} GiB of rows", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    codes = torch.arange(N, dtype=torch.int32, device="cuda")
    sigma = torch.rand(N, generator=g, device="cuda") * 5.0 + 0.2
    sh = torch.empty((N, 3, 25), device="cuda")
    for a in range(0, N, 1 << 22):
        sh[a:a + (1 << 22)].uniform_(-1.0, 1.0, generator=g)
    small = lumiq.octree_from_leaves(10, 4, codes[-LAST:].contiguous(), sigma[-LAST:].contiguous(),
                                     sh[-LAST:].contiguous())
    big = lumiq.octree_from_leaves(10, 4, codes, sigma, sh)
    del sh
    torch.cuda.empty_cache()
    assert big.info()["n_leaves"] == N
    # rays that start within the last cube and leave it into cells that hold no leaf: toward +x, +y and +z
    v = N - LAST
    cell = [sum(((v >> (3 * b + a)) & 1) << b for b in range(10)) for a in range(3)]
    lo = torch.tensor([-1.0 + 2.0 * c / 1024 for c in cell], device="cuda")
    o = lo + torch.rand((20000, 3), generator=g, device="cuda") * (32.0 / 1024)
    d = torch.rand((20000, 3), generator=g, device="cuda") + 0.05
    ra, rb = (t.query(o, d, flags=lumiq.LQ_NO_EARLY_TERM) for t in (small, big))
    torch.cuda.synchronize()
    assert float(ra[0].sum()) > 0 and torch.equal(ra[0], rb[0]) and torch.equal(ra[1], rb[1])
    out = np.zeros(N, np.float32)
    lumiq.check(lumiq.lib().lq_octree_download(big.handle, None, out.ctypes.data, None))
    assert np.array_equal(out, sigma.cpu().numpy())
    small.free()
    big.free()
