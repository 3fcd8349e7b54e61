"""Refinement whose E^H d is formed by gridding: images against the oracle.

Shapes: grids of whole 8-cell tiles (2 n a multiple of 8) and cut ones (odd n), the
shortest side taken (16 voxels), non-square ones, samples on grid cells exactly
(Cartesian, where windows start on a cell), beyond the Nyquist range (windows that wrap
around the grid), all around one point (a tile's list in many segments) and a number that
is no multiple of the 16 of a chunk; species, a voxel mask, coils and none, frames that fill
a 64-row tile and do not.

Tolerance: two steps of refinement converge (each reduces the error by the condition
number, at most about 1.6e4, times 2^-24), so what is left is the image's own rounding
to complex64, 2^-24 at most per value, and the last correction's: 1e-7 of each frame.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    "odd": dict(seed=1002, nx=31, ny=29, C=3, K=1201, F=22),
    "wide": dict(seed=1003, nx=64, ny=16, C=2, K=2003, F=32),
    "one_coil": dict(seed=1004, nx=32, ny=29, C=1, K=1300, F=65),
    "species": dict(seed=1005, nx=28, ny=29, C=4, K=1700, F=5, species=[0.0, 140.0]),
    "mask": dict(seed=1006, nx=34, ny=33, C=4, K=2000, F=3),
    "cartesian": dict(seed=1007, nx=30, ny=30, C=2, K=1300, F=7),
    "wrapped": dict(seed=1008, nx=27, ny=32, C=3, K=1500, F=6),
    "dense": dict(seed=1009, nx=28, ny=28, C=2, K=3001, F=4),
}


def encoding(name):
    w = synth.small_case(**CASES[name])
    enc, rng = w.enc, np.random.default_rng(CASES[name]["seed"])
    if name == "mask":
        enc = dataclasses.replace(enc, voxels=synth.circular_mask(34, 33, 0.97))
    if name == "cartesian":
        enc = dataclasses.replace(enc, k=np.concatenate([synth.cartesian_full(30, 30)] * 2)[:enc.K])
    if name == "wrapped":
        enc = dataclasses.replace(enc, k=(rng.random((enc.K, 2)) - 0.5) * [80.0, 100.0])
    if name == "dense":
        k = enc.k.copy()
        k[1000:] = (rng.random((enc.K - 1000, 2)) - 0.5) * 3.0
        enc = dataclasses.replace(enc, k=k)
    return enc


@pytest.fixture(scope="module")
def P():
    from paper_2410_06129_amd import pinv
    return pinv


@pytest.fixture(scope="module")
def ctx(P):
    c = P.pinv_context_create(0)
    yield c
    P.pinv_context_destroy(c)


def refined(P, ctx, enc, d):
    plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
    P.pinv_plan_wait(plan)
    dd = torch.from_numpy(d).cuda()
    x = torch.full((d.shape[0], enc.N), float("nan"), dtype=torch.complex64, device="cuda")
    P.pinv_apply(ctx, plan, dd, x, refine_steps=2)
    torch.cuda.synchronize()
    P.pinv_plan_release(plan)
    return x.cpu().numpy().astype(np.complex128)


@pytest.mark.parametrize("name", list(CASES))
def test_refined_images_match_oracle(P, ctx, name):
    enc = encoding(name)
    # 1.75 times gridding's multiply-adds in the direct sum, and at least 1e7
    rows, img = CASES[name]["F"] * enc.C * enc.S, enc.nx * enc.ny
    direct = 3 * rows * enc.K * enc.V
    assert direct >= max(1e7, 1.75 * rows * (1058 * enc.K + 3 * img * (4 * enc.nx + 2 * enc.ny)))
    rng = np.random.default_rng(7)
    d = synth.unit_complex_noise((CASES[name]["F"], enc.M), rng).astype(np.complex64)
    x = refined(P, ctx, enc, d)
    R = oracle.Build(enc, rel=1e-2).recon_matrix()
    ref = d.astype(np.complex128) @ R.T
    err = np.linalg.norm(x - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print(f"{name}: {err.max():.1e}")
    assert err.max() <= 1e-7


def test_a_frame_with_infinities_stays_alone(P, ctx):
    enc = encoding("odd")
    d = synth.unit_complex_noise((22, enc.M), np.random.default_rng(8)).astype(np.complex64)
    good = refined(P, ctx, enc, d)
    d[3, 1234] = np.inf
    x = refined(P, ctx, enc, d)
    assert not np.any(np.isfinite(x[3]))
    assert np.array_equal(np.delete(x, 3, 0), np.delete(good, 3, 0))


def test_noalloc_takes_what_the_region_holds(P, ctx):
    """The call asks for at most 531 of the fixed region's 537 MB (the refinement vectors'
    177 and up to four parts of the direct sum), and E^H d is formed beside the vectors,
    with room for shorter passes over the grids only: it is not refused, and agrees with
    the allocating call to the images' rounding (two of them: 2e-7)."""
    F = 5400
    enc = synth.small_case(seed=1010, nx=32, ny=32, C=2, K=600, F=1).enc
    plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
    P.pinv_plan_wait(plan)
    g = torch.Generator(device="cuda").manual_seed(3)
    d = torch.view_as_complex(torch.randn(F, enc.M, 2, device="cuda", generator=g))
    x, y = (torch.full((F, enc.N), float("nan"), dtype=torch.complex64, device="cuda") for _ in range(2))
    P.pinv_apply(ctx, plan, d, x, refine_steps=2)
    P.pinv_apply_noalloc(ctx, plan, d, y, refine_steps=2)
    torch.cuda.synchronize()
    P.pinv_plan_release(plan)
    err = torch.linalg.vector_norm(y - x, dim=1) / torch.linalg.vector_norm(x, dim=1)
    assert float(err.max()) <= 2e-7
