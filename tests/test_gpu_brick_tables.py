"""The device-built brick tables (csrc/bricks.hip) against their definition,
cell by cell (brick_tables of the CPU test of the march): depths around the
brick and top-grid levels, sparse, dense and single-leaf trees, leaves in the
grid's corners."""
import ctypes as C
import glob
import os

import numpy as np
import pytest

import inputs
from tests.test_brick_march_cpu import brick_tables

pytestmark = pytest.mark.gpu


def _cells(depth, p_occ):
    t = inputs.random_tree(depth, p_occ, seed=depth + 7)
    return t.child, t.leaf_cells


@pytest.mark.parametrize("depth,p_occ", [(1, 0.5), (2, 0.3), (3, 0.02), (4, 0.003), (4, 0.5), (5, 0.0005), (6, 0.00002),
                                         (6, 0.01), (7, 0.000005)])
def test_tables_are_their_definition(depth, p_occ):
    import torch
    from paper_2207_05009_amd import lumiq
    print(f"[gpu] brick tables, depth {depth}, occupancy {p_occ}", flush=True)
    child, cells = _cells(depth, p_occ)
    build = lumiq.lib()["_ZN2lq12build_bricksEPKiiPPjPmPPKjS7_"]      # lq::build_bricks
    dev = torch.from_numpy(np.ascontiguousarray(child, dtype=np.int32)).cuda()
    torch.cuda.synchronize()
    buf, size, top, bricks = C.c_void_p(), C.c_size_t(), C.c_void_p(), C.c_void_p()
    assert build(C.c_void_p(dev.data_ptr()), depth, C.byref(buf), C.byref(size), C.byref(top), C.byref(bricks)) == 0
    out = np.zeros(size.value // 4, np.uint32)
    hip = C.CDLL(glob.glob(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so*"))[0])
    assert hip.hipMemcpy(C.c_void_p(out.ctypes.data), buf, size, 2) == 0
    assert hip.hipFree(buf) == 0
    ref_top, ref = brick_tables(depth, np.asarray(cells))
    at = (top.value - buf.value) // 4
    assert (bricks.value - buf.value) == 0 and at == ref.size
    assert np.array_equal(out[at:], ref_top)
    assert np.array_equal(out[:at].reshape(ref.shape), ref)
