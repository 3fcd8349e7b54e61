"""Refinement's residual and triangular products with their contractions in parts, at
the edges of the split: 127, 128 and 129 unknowns (15 to 17 chunks of 8: one part or
two, the last cut), 255 and 257 (the same for the triangular products), 1100 (many
parts), one frame, a whole tile of frames and one more, in FP32 and FP64, by plans with
and without R.  Two steps converge to the image's own rounding: 1e-7 of each frame
in complex64, 1e-9 in complex128 (condition number at most about 1e4).
"""
import numpy as np
import pytest

import oracle
from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRIDS = {127: (127, 1), 128: (16, 8), 129: (43, 3), 255: (17, 15), 257: (257, 1), 1100: (44, 25)}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("F", [1, 64, 129])
@pytest.mark.parametrize("N", list(GRIDS))
def test_refined_images_match_oracle(N, F, prec):
    from paper_2410_06129_amd import pinv as P
    nx, ny = GRIDS[N]
    enc = synth.small_case(seed=1100 + N, nx=nx, ny=ny, C=2, K=N, F=1).enc
    cdt = np.complex64 if prec == "fp32" else np.complex128
    d = synth.unit_complex_noise((F, enc.M), np.random.default_rng(N)).astype(cdt)
    ref = d.astype(np.complex128) @ oracle.Build(enc, rel=1e-2).recon_matrix().T
    ctx = P.pinv_context_create(0)
    try:
        for flags in (0, P.FLAG_NO_R):
            plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG,
                                P.FP32 if prec == "fp32" else P.FP64, P.FLAG_UNCACHED | flags)
            P.pinv_plan_wait(plan)
            x = torch.full((F, N), float("nan"), dtype=getattr(torch, str(np.dtype(cdt))), device="cuda")
            P.pinv_apply(ctx, plan, torch.from_numpy(d).cuda(), x, refine_steps=2)
            torch.cuda.synchronize()
            P.pinv_plan_release(plan)
            err = np.linalg.norm(x.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
            assert err.max() <= (1e-7 if prec == "fp32" else 1e-9), (flags, err.max())
    finally:
        P.pinv_context_destroy(ctx)
