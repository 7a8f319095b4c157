"""An error that an earlier call of the program left with the HIP runtime (here an
allocation that was refused) is not the loader's, the builder's nor the
download's."""
import ctypes as C
import glob
import os

import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu


def test_load_build_and_download_after_a_refused_allocation():
    import torch
    from paper_2207_05009_amd import lumiq
    lumiq.lib()
    torch.zeros(1, device="cuda")
    hip = C.CDLL(glob.glob(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so*"))[0])
    p = C.c_void_p()

    def refused():
        assert hip.hipMalloc(C.byref(p), C.c_size_t(1 << 50)) != 0

    print("[gpu] load and download with an error left over", flush=True)
    t = inputs.random_tree(5, 0.1, seed=4, sh_degree=1)
    refused()
    tree = lumiq.Octree(t, "f16")
    refused()
    out = tree.download()
    assert np.array_equal(out["child"], t.child) and out["sigma"].shape == t.sigma.shape
    codes = torch.from_numpy(inputs.morton3(*t.leaf_cells.T).astype(np.int32)).cuda()
    sigma, sh = torch.from_numpy(t.sigma).cuda(), torch.from_numpy(t.sh).cuda()
    torch.cuda.synchronize()
    refused()
    built = lumiq.octree_from_leaves(5, 1, codes, sigma, sh, storage="f16")
    assert built.info() == tree.info()               # brick tables included
    hip.hipGetLastError()
    tree.free()
    built.free()
