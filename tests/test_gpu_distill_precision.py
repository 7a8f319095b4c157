"""Precision of the distillation's sample loop (csrc/distill.hip) where its forms
meet: with one sample per voxel nothing averages the rounding of the exponents,
the exponentials and the logarithms.  Against the oracle in FP64, with bounds that
follow from the instructions' own errors: exp2 and rcp one ulp (2^-23), the other
operations half of one (2^-24)."""
import numpy as np
import pytest

import inputs
from inputs.trees import field_params
from oracle import distill as od

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _distilled(p, depth, samples, seed):
    import torch
    from paper_2207_05009_amd import lumiq
    codes, sig, sh = lumiq.distill_leaves(p, depth, 0.01, samples, seed)
    torch.cuda.synchronize()
    codes = codes.cpu().numpy().view(np.uint32).astype(np.uint64)
    ref = od.average_samples(od.field_from_params(p), depth, codes, samples, seed)
    return sig.cpu().numpy(), sh.cpu().numpy().reshape(len(codes), 3, -1), ref[0], ref[1].reshape(len(codes), 3, -1)


@pytest.mark.parametrize("change", [7.3, 7.7, 30.0, 62.0])
def test_weights_are_as_precise_as_their_exponentials(change):
    """Two blobs near the centre, every voxel kept: far from both, on the plane
    between them, both weights count while the exponents change by up to `change`
    within half a voxel.  An exponent below 8 is rounded by 2^-22 at most, a
    larger one, when taken relative to the voxel's centre, by up to 2^-19."""
    depth = 6
    p = field_params(inputs.TreeSpec(depth=depth, n_blobs=2, n_shells=0, sh_degree=1, seed=3, occupancy=0.3))
    p["centres"] = np.array([[0.02, 0.03, -0.04], [-0.03, 0.02, 0.05]])
    half = 0.5 * np.sqrt(3.0) * 2.0 / (1 << depth)
    far = np.sqrt(((1.0 + np.abs(p["centres"])) ** 2).sum(1))
    p["radii"] = np.sqrt(np.log2(np.e) * half * (2.0 * far + half) / (2.0 * change))
    p["amps"] = np.array([12.0, -12.0])
    p["log_base"], p["sigma_max"] = 0.0, 1e9
    p["hi"] = np.ones((2, 3, 3)) * np.array([1.0, -1.0])[:, None, None]
    print(f"[gpu] distillation, exponents change by {change}", flush=True)
    sig, sh, ref_sig, ref_sh = _distilled(p, depth, 1, 9)
    assert len(sig) > 0.9 * 8 ** depth                   # but for those by the negative blob
    eps = 2 * U + 4 * U * np.log(2.0)                    # an exponential: its own ulp, its exponent's rounding
    # w1 - w2: 2 w1 w2 (e1 + e2), the common 1 / s (sum, rcp, product), the result
    bound = 0.5 * 2 * eps + 4 * U + U
    err = np.abs(sh[:, :, 1:] - ref_sh[:, :, 1:]).max()
    print(f"[gpu] w1 - w2 off by {err:.2e}, bound {bound:.2e}", flush=True)
    assert err <= bound
    # ln density = sum a g: 24 times a term's error, the argument of exp2 (below 32), exp2
    log_err = np.abs(sig / ref_sig - 1.0).max()
    assert log_err <= 24.0 * (eps + 3 * U) + 2.0 ** -20 * np.log(2.0) + 2 * U, log_err


@pytest.mark.parametrize("bright", [0.05, 0.45, 0.499, 0.501, 0.9, 1.0 - 2.0 ** -10, 1.0 - 2.0 ** -14])
def test_dc_near_the_ceiling(bright):
    """One blob of radiance bright * l_max: the DC coefficient is a constant,
    2 sqrt(pi) ln(E / (l_max - E)).  Up to half the ceiling the difference is taken
    of rounded sums (a rounding of E times E / (l_max - E)); above, from the blobs'
    own differences, which cancel nothing."""
    depth = 4
    p = field_params(inputs.TreeSpec(depth=depth, n_blobs=1, n_shells=0, sh_degree=1, seed=5, occupancy=0.3))
    p["radii"] = np.array([0.4])
    p["emission"] = np.float32(bright * p["l_max"]) * np.ones((1, 3))
    print(f"[gpu] distillation, radiance at {bright} of the ceiling", flush=True)
    _, sh, _, ref = _distilled(p, depth, 1, 9)
    ratio = float(p["emission"][0, 0] / (p["l_max"] - p["emission"][0, 0]))
    # the quotient: E, the difference, their products, rcp (one ulp); log2 (one ulp), the scaled result
    amplified = ratio if bright <= 0.5 else 0.0
    scale = 2.0 * np.sqrt(np.pi)
    bound = scale * (amplified + 8.0) * U + scale * np.log(2.0) * 2 * U * max(1.0, abs(np.log2(ratio))) + 2 * U * scale * abs(np.log(ratio))
    err = np.abs(sh[:, :, 0] - ref[:, :, 0]).max()
    print(f"[gpu] DC off by {err:.2e}, bound {bound:.2e}", flush=True)
    assert err <= bound


def test_infinite_ceiling():
    """E / l_max is 0 for an infinite l_max: every DC coefficient is -inf, also
    where a blob's weight vanishes."""
    import torch
    from paper_2207_05009_amd import lumiq
    p = field_params(inputs.TreeSpec(depth=4, n_blobs=6, n_shells=2, sh_degree=1, seed=6, occupancy=0.3))
    p["radii"] = np.full(6, 0.02)
    p["l_max"] = np.inf
    print("[gpu] distillation without a ceiling", flush=True)
    _, sig, sh = lumiq.distill_leaves(p, 4, 0.01, 20, 3)
    torch.cuda.synchronize()
    assert len(sig) > 0 and bool(torch.isfinite(sig).all()) and bool(torch.isfinite(sh[:, :, 1:]).all())
    assert bool((sh[:, :, 0] == -np.inf).all())
