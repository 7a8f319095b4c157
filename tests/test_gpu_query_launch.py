"""Launch forms of the emission query: one lane per ray without counters for a
batch that fits the resident blocks, chunks of rays from shared counters for a
larger one, whole 8 x 8 tiles for a camera batch.  A ray's result does not
depend on them: a batch of any size gives the bits that the same rays give in
batches of one, of a wave and in a large one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _batch(n, seed):
    rng = np.random.default_rng(seed)
    o = rng.normal(size=(n, 3))
    o = o / np.linalg.norm(o, axis=1, keepdims=True) * rng.uniform(0.3, 4.0, (n, 1))
    d = rng.uniform(-1.2, 1.2, (n, 3)) - o
    d[::97] = -o[::97]                       # through the centre
    d[5::101, 0] = 0.0                       # along planes of cells
    return o.astype(np.float32), d.astype(np.float32)


@pytest.mark.parametrize("storage,model", [("f32", "linear"), ("f16", "exp")])
def test_batch_size_does_not_change_a_ray(c0_tree, storage, model):
    import torch
    import paper_2207_05009_amd as lq
    oct_ = lq.Octree(c0_tree, storage)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    top = 1 << 21                            # beyond every resident grid: chunks from the counters
    o, d = (torch.from_numpy(a).cuda() for a in _batch(top, 3))
    ref, ref_a = oct_.query(o, d, model=model)
    assert float(ref.sum()) > 0
    sizes = [1, 2, 63, 64, 65, 127, 128, 129, 4095, 4096, 65535, 65536, 65537]
    for waves in (3, 4, 5, 8):               # the resident lanes at these waves per SIMD, and one more
        sizes += [cus * 4 * waves * 64 + k for k in (-1, 0, 1)]
    for n in sizes:
        print(f"[gpu] query {storage} {model}, {n} rays", flush=True)
        a = 7 if n < top - 7 else 0          # a slice that starts inside a chunk
        rgb, alpha = oct_.query(o[a:a + n].contiguous(), d[a:a + n].contiguous(), model=model)
        assert torch.equal(rgb, ref[a:a + n]) and torch.equal(alpha, ref_a[a:a + n]), n
    for i in (0, 97, 106, 1234):             # batches of one
        rgb, alpha = oct_.query(o[i:i + 1].contiguous(), d[i:i + 1].contiguous(), model=model)
        assert torch.equal(rgb[0], ref[i]) and torch.equal(alpha[0], ref_a[i]), i
    oct_.free()


@pytest.mark.parametrize("w,h", [(1, 1), (7, 9), (8, 8), (9, 8), (64, 1), (1, 65), (257, 131), (1283, 721), (2048, 1027)])
def test_camera_tiles_do_not_change_a_ray(c0_tree, w, h):
    import torch
    import paper_2207_05009_amd as lq
    print(f"[gpu] camera batch {w} x {h}", flush=True)
    oct_ = lq.Octree(c0_tree, "f32")
    x, y = np.meshgrid((np.arange(w) + 0.5) / w - 0.5, (np.arange(h) + 0.5) / h - 0.5)
    d = np.stack([x, y, np.full_like(x, 1.3)], -1).reshape(-1, 3).astype(np.float32)
    o = np.tile(np.float32([0.1, -0.2, -3.0]), (w * h, 1))
    ot, dt = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    rgb, alpha = oct_.query_image(ot, dt, w, h)
    ref, ref_a = oct_.query(ot, dt)
    assert torch.equal(rgb.reshape(-1, 3), ref) and torch.equal(alpha.reshape(-1), ref_a)
    oct_.free()
