"""The operator on canonical spinors where its tiles can go wrong, against the oracle's operator.

Extents that tiles do not divide, that one tile spans, that exceed a workgroup along x, two-site axes, both launch
sizes (one and four waves per workgroup), both link forms of FP32, and spinors that overlap or are not 16-byte
aligned.  Tolerances relative to max |reference|, as for the block-layout stencils: the storage's unit roundoff times
the eight-term sum (FP64 1e-13, FP32 2e-6, FP16 4e-3, BF16 3e-2).
"""

import numpy as np
import pytest

import synth
from oracle import lattice as lat

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-13, "f32": 2e-6, "f16": 4e-3, "bf16": 3e-2}


@pytest.mark.parametrize("dims,n", [((2, 2, 2, 2), 1), ((5, 3, 7, 4), 2), ((300, 2, 3, 2), 1), ((66, 3, 2, 5), 1),
                                    ((17, 9, 11, 13), 6), ((16, 16, 8, 9), 9), ((258, 8, 4, 4), 5)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("scale", [1.0, 0.9])
def test_against_oracle(dims, n, storage, scale):
    import torch

    from paper_2212_04430_amd import _lib as L
    U = synth.gauge_field(dims, eps=0.5, seed=4) * scale  # 0.9: not special unitary, whole links
    psi = synth.random_spinor(dims, seed=6, n=n)
    ctx = L.fs_create(dims, 1, 0)
    try:
        L.fs_upload_gauge(ctx, U)
        got = L.fs_apply_dirac(ctx, 0.1, 0.3, storage, torch.from_numpy(psi).cuda()).cpu().numpy()
    finally:
        L.fs_destroy(ctx)
    for i in {0, n - 1}:
        ref = lat.wilson_apply(U, psi[i], 0.1, 0.3, dims, True)
        assert np.abs(got[i] - ref).max() <= TOL[storage] * np.abs(ref).max()


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_overlap_and_alignment(storage):
    """In place, shifted by less than a spinor, and from an odd multiple of 8 bytes: as from separate buffers."""
    import ctypes as C

    import torch

    from paper_2212_04430_amd import _lib as L
    dims = (6, 4, 5, 4)
    V = int(np.prod(dims))
    U = synth.gauge_field(dims, eps=0.5, seed=4)
    psi = torch.from_numpy(synth.random_spinor(dims, seed=6)).cuda()
    ctx = L.fs_create(dims, 0, 0)
    try:
        L.fs_upload_gauge(ctx, U)
        ref = L.fs_apply_dirac(ctx, 0.1, 0.3, storage, psi)
        n = 24 * V
        for src, dst in ((0, 0), (0, 8), (8, 0), (1, n + 2), (0, n + 1)):
            buf = torch.zeros(2 * n + 16, dtype=torch.float64, device="cuda")
            buf[src:src + n] = torch.view_as_real(psi).reshape(-1)
            p = buf.data_ptr()
            torch.cuda.synchronize()
            assert L._lib.fs_apply_dirac(ctx, 0.1, 0.3, L.PREC[storage], C.c_void_p(p + 8 * src),
                                         C.c_void_p(p + 8 * dst), 1, 1) == 0
            got = torch.view_as_complex(buf[dst:dst + n].clone().reshape(V, 4, 3, 2))
            assert float((got - ref).abs().max()) <= TOL[storage] * float(ref.abs().max())
    finally:
        L.fs_destroy(ctx)
