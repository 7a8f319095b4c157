"""The benchmark's roofline record: only bytes that every launch has to move, so
neither the steps of the octree march (which the timed kernel does not take) nor
its leaf rows enter the fraction, and it stays below 1."""
import numpy as np
import pytest

import bench


class _Counts(np.ndarray):
    def numel(self):
        return self.size


def _counts(n, v):
    return np.full(n, v, np.int64).view(_Counts)


class _Tree:
    def __init__(self, n, steps):
        self.out = {"count": _counts(n, 5), "n_comp": _counts(n, 5), "n_steps": _counts(n, steps)}

    def trace(self, o, d, model, flags):
        return self.out


class _Lumiq:
    LQ_TRACE_PRUNED = 8


@pytest.mark.parametrize("ms", [0.05, 0.8, 3.0])
def test_roofline_fraction_is_of_the_bytes_every_launch_moves(ms):
    n = 1 << 20
    o = np.zeros((n, 3), np.float32)
    few, many = (bench.variant_record(_Lumiq, _Tree(n, k), o, o, "linear", 9, 4, ms) for k in (19, 28))
    assert few["roofline_frac"] == many["roofline_frac"] == round(40 * n / (ms * 1e-3) / 8e12, 4) < 1.0
    assert many["octree_work"]["bytes_per_launch"] - few["octree_work"]["bytes_per_launch"] == 9 * 4 * n
    assert few["traffic"] is None and few["traffic_frac"] is None


def test_measured_traffic_has_a_fraction_of_its_own():
    rec = bench.roofline_record(1 << 22, 0.82, 0.76e9)
    assert rec["traffic_frac"] == round(0.76e9 / 0.82e-3 / 8e12, 4)
    assert rec["roofline_frac"] == round(40 * (1 << 22) / 0.82e-3 / 8e12, 4)
