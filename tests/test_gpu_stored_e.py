"""Products that read a stored encoding matrix.

FP64 plans of 640 unknowns or more store E^H before the W product: R element by
element against the oracle on both sides of that size, over every factor an element
can have (coils, species, off-resonance, a voxel mask) and sample counts on and off
the 64-column tiles.  1e-9 of the largest element, as for every FP64 R.

The shared-trajectory Gram stores F^H where R's or W's memory holds it: two coils of an
FP32 plan just do, one coil does not; sizes on and off the 64-voxel tiles and 8-sample
chunks.  1e-12 of the largest element (FP64 sums of at most 1000 unit-size terms).

Refinement of FP32 plans forms E^H d through a stored F^H where gridding does not: a
map, species, odd voxel and sample counts, one frame and 64 frames of one coil more,
a contraction in splits, and columns in two slabs.  Two steps converge to the image's
own rounding to complex64: 1e-7 of each frame."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = {
    "n639": dict(seed=901, nx=71, ny=9, C=2, K=330, F=1),
    "n640": dict(seed=902, nx=32, ny=20, C=2, K=320, F=1),
    "n641_one_coil": dict(seed=903, nx=641, ny=1, C=1, K=705, F=1),
    "n646_species_b0": dict(seed=904, nx=17, ny=19, C=3, K=217, F=1, species=[0.0, 170.0], b0=True),
    "mask": dict(seed=905, nx=32, ny=30, C=3, K=255, F=1, b0=True),
}


@pytest.mark.parametrize("form", ["3m", "4m"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_r_matches_oracle(name, form):
    from paper_2410_06129_amd import pinv as P
    enc = synth.small_case(**SHAPES[name]).enc
    if name == "mask":
        enc = dataclasses.replace(enc, voxels=synth.circular_mask(32, 30, 0.96))
    assert (enc.N >= 640) == (name != "n639") and enc.M >= enc.N
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP64, P.FLAG_UNCACHED,
                            cprod=P.CPROD_3M if form == "3m" else P.CPROD_4M)
        P.pinv_plan_wait(plan)
        R = torch.full((enc.N, enc.M), float("nan"), dtype=torch.complex128, device="cuda")
        P.pinv_plan_copy_buffer(plan, P.BUF_R, R)
        torch.cuda.synchronize()
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)
    ref = oracle.Build(enc, rel=1e-2).recon_matrix()
    assert np.max(np.abs(R.cpu().numpy() - ref)) <= 1e-9 * np.max(np.abs(ref))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("coils", [1, 2])
@pytest.mark.parametrize("nx,ny,K", [(1, 1, 9), (8, 8, 64), (13, 5, 131), (16, 12, 200)])
def test_shared_gram_matches_oracle(nx, ny, K, coils, prec):
    from paper_2410_06129_amd import pinv as P
    enc = synth.small_case(seed=910 + K, nx=nx, ny=ny, C=coils, K=K, F=1, b0=True).enc
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG,
                            {"fp64": P.FP64, "fp32": P.FP32, "bf16x3": P.BF16X3}[prec], P.FLAG_UNCACHED)
        P.pinv_plan_wait(plan)
        assert P.pinv_plan_info_get(plan)["gram_form"] == P.GRAM_SHARED
        G = torch.full((enc.N, enc.N), float("nan"), dtype=torch.complex128, device="cuda")
        P.pinv_plan_copy_buffer(plan, P.BUF_GRAM, G)
        torch.cuda.synchronize()
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)
    Go = oracle.gram(enc)
    assert np.max(np.abs(G.cpu().numpy() - Go)) <= 1e-12 * np.max(np.abs(Go))


REFINED = {
    "one_frame": dict(seed=921, nx=13, ny=11, C=3, K=301, F=1, b0=True),
    "one_coil_65": dict(seed=922, nx=12, ny=9, C=1, K=333, F=65),
    "map_one_coil": dict(seed=923, nx=16, ny=8, C=1, K=500, F=3, b0=True),
    "species_map": dict(seed=924, nx=11, ny=12, C=4, K=700, F=17, species=[0.0, 170.0], b0=True),
    "mask": dict(seed=925, nx=15, ny=14, C=5, K=201, F=26, b0=True),
    "slabs": dict(seed=926, nx=24, ny=24, C=8, K=600, F=3600, species=[0.0, 170.0], b0=True),
}


@pytest.mark.parametrize("name", list(REFINED))
def test_refined_images_match_oracle(name):
    from paper_2410_06129_amd import pinv as P
    enc = synth.small_case(**REFINED[name]).enc
    if name == "mask":
        enc = dataclasses.replace(enc, voxels=synth.circular_mask(15, 14, 0.97))
    F = REFINED[name]["F"]
    if name == "slabs":   # F^H and its product with every frame and coil: 512 MB
        assert 16 * enc.N * (enc.K + F * enc.C) > 512 << 20
    d = synth.unit_complex_noise((F, enc.M), np.random.default_rng(9)).astype(np.complex64)
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
        P.pinv_plan_wait(plan)
        x = torch.full((F, enc.N), float("nan"), dtype=torch.complex64, device="cuda")
        P.pinv_apply(ctx, plan, torch.from_numpy(d).cuda(), x, refine_steps=2)
        torch.cuda.synchronize()
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)
    x = x.cpu().numpy().astype(np.complex128)
    assert np.all(np.isfinite(x.view(np.float64)))
    pick = slice(None, None, 97 if F > 1000 else 1)
    ref = d[pick].astype(np.complex128) @ oracle.Build(enc, rel=1e-2).recon_matrix().T
    err = np.linalg.norm(x[pick] - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print(f"{name}: {err.max():.1e}")
    assert err.max() <= 1e-7
