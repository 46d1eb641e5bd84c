"""The fused displaced bilinears (all p in one pass over z-lines) against the oracle's definition.

Sizes sit where the lane mapping changes: z-lines of 2, odd ones, ones that fill a workgroup or leave most of it
idle, the first that no longer fits (the one-hop launches), every rhs subset size.  Tolerance: an FP64 sum of N
products differs from another order's by at most about N eps of the sum of magnitudes, and the p-fold link products
add 3p roundings; both lie far below 1e-13 of |y| |x| for the sizes here (N <= 6e4 terms of random sign).
"""

import numpy as np
import pytest

import synth
from oracle import fs as ofs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,p_max", [((4, 4, 2, 4), 1), ((3, 5, 7, 3), 6), ((2, 3, 17, 5), 0), ((2, 2, 33, 3), 9),
                                        ((2, 2, 64, 2), 50), ((2, 2, 256, 2), 3), ((2, 2, 257, 2), 3),
                                        ((6, 4, 129, 2), 2), ((2, 2, 64, 2), 63)])
@pytest.mark.parametrize("device", [False, True])
def test_bilinear_against_oracle(dims, p_max, device):
    import torch

    from paper_2212_04430_amd import _lib as L
    U = synth.gauge_field(dims, eps=0.4, seed=2)
    y, x = synth.random_spinor(dims, seed=5, n=2)
    ctx = L.fs_create(dims, 0, 0)
    try:
        L.fs_upload_gauge(ctx, U)
        if device:
            got = L.fs_bilinear(ctx, p_max, torch.from_numpy(y).cuda(), torch.from_numpy(x).cuda())
        else:
            got = L.fs_bilinear(ctx, p_max, y, x)
    finally:
        L.fs_destroy(ctx)
    ref = ofs.bilinears(U, dims, y, x, range(16), p_max).T
    assert np.abs(got - ref).max() <= 1e-13 * np.linalg.norm(y) * np.linalg.norm(x)


@pytest.mark.parametrize("dims,nr", [((4, 4, 4, 4), 1), ((4, 4, 4, 4), 2), ((4, 2, 18, 4), 8), ((2, 4, 24, 2), 16),
                                     ((4, 4, 66, 2), 4)])
def test_rhs_subsets_agree(dims, nr):
    """Samples of an estimate in blocks of nr against blocks of another size (another subset of systems per
    workgroup): the solves agree to 1e-12, so the samples do to 1e-10 of the largest."""
    from paper_2212_04430_amd import _lib as L
    ctx = L.fs_create(dims, 0, 0)
    try:
        L.fs_upload_gauge(ctx, synth.gauge_field(dims, eps=0.3, seed=1))
        X = []
        for block in (nr, 4 if nr != 4 else 1):
            sp = L.solve_params(0.2, tol=1e-12, storage="f64", batched=1, rhs_block=block)
            X.append(L.fs_estimate(ctx, L.fs_est_params(3, 5, 0, min(8, dims[2] - 1), sp), [0.0, 0.4],
                                   want_samples=True)[1])
    finally:
        L.fs_destroy(ctx)
    assert np.abs(X[0] - X[1]).max() <= 1e-10 * np.abs(X[1]).max()
