"""GPU parity of the distillation kernel's forms (csrc/distill.hip): exponents
relative to the voxel's centre or to each sample's maximum, logarithms of
products of DC terms or of each term, 8, 16 and 32 unrolled blobs, sample
counts around the block of 16 and the product of 4.  Each against the oracle
in FP64, with the bound of the other distillation tests: float32 rounding of
the sums and of exp2 / log2, 1e-4 relative."""
import numpy as np
import pytest

import inputs
from inputs.trees import field_params
from oracle import distill as od

pytestmark = pytest.mark.gpu
RTOL = 1e-4


@pytest.fixture(scope="module")
def lq():
    import torch
    import paper_2207_05009_amd as lq
    assert torch.cuda.is_available()
    lq.lib()
    return lq


def _centred(p, depth):
    """The host's rule: no exponent changes by more than 64 in half a voxel diagonal."""
    half = 0.5 * np.sqrt(3.0) * 2.0 / (1 << depth)
    far = np.sqrt(((1.0 + np.abs(p["centres"])) ** 2).sum(1))
    return bool((np.log2(np.e) / (2.0 * np.asarray(p["radii"]) ** 2) * half * (2.0 * far + half)).max() <= 64.0)


@pytest.mark.parametrize("emission", ["plain", "faint", "bright"])
@pytest.mark.parametrize("radius,n_blobs,n_shells,samples", [
    (0.3, 8, 0, 16), (0.3, 9, 2, 17), (0.3, 17, 8, 3), (0.3, 1, 1, 5),
    (0.03, 8, 3, 1), (0.03, 16, 1, 4), (0.03, 32, 2, 33), (0.002, 3, 1, 8)])
def test_forms_match_oracle(lq, radius, n_blobs, n_shells, samples, emission):
    import torch
    depth = 4
    p = field_params(inputs.TreeSpec(depth=depth, n_blobs=n_blobs, n_shells=n_shells, sh_degree=1, seed=40 + n_blobs,
                                     occupancy=0.3))
    p["radii"] = np.random.default_rng(n_blobs).uniform(1.0, 1.5, n_blobs) * radius
    e = np.array(p["emission"], dtype=np.float64)
    if emission == "faint":
        e[0] = 1e-9                               # below 2^-24
    elif emission == "bright":
        e[-1] = p["l_max"] * (1.0 - 2.0 ** -13)   # within 2^-12 of the ceiling
    p["emission"] = e
    assert _centred(p, depth) == (radius > 0.1)
    print(f"[gpu] radius {radius}, {n_blobs} blobs, {n_shells} shells, {samples} samples, {emission}", flush=True)
    codes, sig, sh = lq.distill_leaves(p, depth, 0.01, samples, 5)
    torch.cuda.synchronize()
    g_codes = codes.cpu().numpy().view(np.uint32).astype(np.uint64)
    assert g_codes.size > 0
    f = od.field_from_params(p)
    o_codes, amb = od.centre_occupancy(f, depth)
    assert np.all(np.isin(np.setxor1d(g_codes, o_codes), amb))
    o_sig, o_sh = od.average_samples(f, depth, g_codes, samples, 5)
    es = np.abs(sig.cpu().numpy() - o_sig) / np.maximum(np.abs(o_sig), 1e-3)
    eh = np.abs(sh.cpu().numpy() - o_sh) / np.maximum(np.abs(o_sh), 1e-2)
    assert es.max() <= RTOL and eh.max() <= RTOL, (es.max(), eh.max())


@pytest.mark.parametrize("depth,n_blobs,n_shells,radius", [(1, 2, 0, 0.5), (2, 5, 1, 0.5), (6, 16, 0, 0.3), (6, 9, 8, 0.05),
                                                           (7, 32, 2, 0.15)])
def test_kept_voxels_match_oracle(lq, depth, n_blobs, n_shells, radius):
    """The kept voxels are a decision: words of 64 centres decided at once by
    bounds, with amplitudes of both signs, agree with the oracle's centres
    (other than those it names ambiguous)."""
    p = field_params(inputs.TreeSpec(depth=depth, n_blobs=n_blobs, n_shells=n_shells, sh_degree=0, seed=60 + depth,
                                     occupancy=0.3))
    rng = np.random.default_rng(n_blobs)
    p["radii"] = rng.uniform(1.0, 2.0, n_blobs) * radius
    p["amps"] = np.array(p["amps"]) * np.where(np.arange(n_blobs) % 3 == 1, -1.0, 1.0)
    print(f"[gpu] kept voxels, depth {depth}, {n_blobs} blobs, {n_shells} shells", flush=True)
    codes, _, _ = lq.distill_leaves(p, depth, 0.01, 1, 5)
    g_codes = codes.cpu().numpy().view(np.uint32).astype(np.uint64)
    o_codes, amb = od.centre_occupancy(od.field_from_params(p), depth)
    assert g_codes.size > 0 and np.all(np.diff(g_codes.astype(np.int64)) > 0)
    assert np.all(np.isin(np.setxor1d(g_codes, o_codes), amb))


def test_radiances_far_below_the_ceiling(lq):
    """Radiances of 1e-6 under a ceiling of 8e6: the DC term's argument is
    1e-13 per sample, and its product over four samples would leave float32's
    range.  The bound is that of the forms above."""
    p = field_params(inputs.TreeSpec(depth=4, n_blobs=5, n_shells=1, sh_degree=0, seed=44, occupancy=0.3))
    p["radii"] = np.full(5, 0.3)
    p["l_max"] = 8e6
    p["emission"] = np.full((5, 3), 1e-6) * np.arange(1, 6)[:, None]
    print("[gpu] distillation, radiances far below the ceiling", flush=True)
    codes, sig, sh = lq.distill_leaves(p, 4, 0.01, 9, 5)
    g_codes = codes.cpu().numpy().view(np.uint32).astype(np.uint64)
    o_sig, o_sh = od.average_samples(od.field_from_params(p), 4, g_codes, 9, 5)
    eh = np.abs(sh.cpu().numpy() - o_sh) / np.maximum(np.abs(o_sh), 1e-2)
    assert g_codes.size > 0 and eh.max() <= RTOL, eh.max()
