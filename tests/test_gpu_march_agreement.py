"""The production query (brick tables) against the trace of the pruned octree, which
records its leaves: the same leaves over the same segments, so the same bits,
except where a segment starts at an edge or a corner, whose tie may be represented
by another axis: the segment is then off by a few float32 ulp, transmittance by
1e-6 and radiance by 1e-5 of itself (the bounds of the same comparison on the CPU).
At the depths that the CPU comparison does not reach."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu


def _compare(tree, depth, n):
    import torch
    from paper_2207_05009_amd import lumiq
    o, d = (np.concatenate(v) for v in zip(inputs.rays.sphere_to_cube(n, 5), inputs.rays.room_to_proxy(n, 6),
                                           inputs.rays.adversarial(depth, 7, 20000)))
    o, d = (torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda() for a in (o, d))
    for model in ("linear", "exp"):
        rgb, alpha = tree.query(o, d, model=model)
        tr = tree.trace(o, d, model=model, flags=lumiq.LQ_TRACE_PRUNED)
        torch.cuda.synchronize()
        assert int(tr["n_comp"].sum()) > n
        same = (rgb == tr["rgb"]).all(1) & (alpha == tr["alpha"])
        assert float(same[:2 * n].float().mean()) > 0.9999 and float(same.float().mean()) > 0.9
        go = (tr["alpha"] - 0.9).abs() >= 1e-5            # the stop test may go either way there
        assert float((alpha - tr["alpha"]).abs()[go].max()) < 1e-6
        top = tr["rgb"].max(1).values.clamp_min(2e-3)
        assert bool(((rgb - tr["rgb"]).abs().max(1).values <= 1e-5 * top)[go].all())
    tree.free()


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_full_size_luminaire(c1_tree, storage):
    from paper_2207_05009_amd import lumiq
    print(f"[gpu] marches agree, depth 9, {storage}", flush=True)
    _compare(lumiq.Octree(c1_tree, storage), 9, 1 << 20)


def test_depth_10():
    import torch
    from paper_2207_05009_amd import lumiq
    print("[gpu] marches agree, depth 10, scattered leaves and a solid corner", flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)
    codes = torch.unique(torch.cat([torch.randint(0, 1 << 30, (1 << 20,), generator=g, device="cuda"),
                                    torch.arange(1 << 21, device="cuda")])).to(torch.int32)
    n = codes.numel()
    tree = lumiq.octree_from_leaves(10, 3, codes, torch.rand(n, generator=g, device="cuda") * 20.0,
                                    torch.randn((n, 3, 16), generator=g, device="cuda"), storage="bf16")
    _compare(tree, 10, 1 << 19)
