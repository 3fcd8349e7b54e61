"""FP32 products on f16 pieces: R against the oracle, beside the same plan on
FP32 matrix instructions.

Shapes sit at the edges of the 128 x 128 tiles and 32-column chunks: N = 256 and
384 (whole tiles), 274, 289 and 340 (ragged: padded rows of W^T and a second slab
of conj(E)), M a multiple of the tile and not, with several coils, a voxel mask,
species and an off-resonance map; each just past the size where this path starts.

Tolerance: a value is held within 2^-24 relative (rms) in two f16 pieces and
within 2^-25 in FP32, and both accumulate in FP32, so R may be at most twice as
far from the oracle as the FP32 instructions leave it (the factor's three
pieces and the longer sums between roundings make it better in general).
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = {
    "n256": dict(seed=301, nx=16, ny=16, C=8, K=600, F=3),
    "n289_odd": dict(seed=302, nx=17, ny=17, C=12, K=1501, F=3),
    "n384_whole": dict(seed=303, nx=32, ny=12, C=2, K=1024, F=3),
    "n340_b0": dict(seed=304, nx=10, ny=17, C=8, K=1650, F=3, species=[0.0, 170.0], b0=True),
}


@pytest.fixture(scope="module")
def P():
    from paper_2410_06129_amd import pinv
    return pinv


@pytest.fixture(scope="module")
def ctx(P):
    c = P.pinv_context_create(0)
    yield c
    P.pinv_context_destroy(c)


def get_r(P, ctx, enc, **kw):
    plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED, **kw)
    P.pinv_plan_wait(plan)
    R = torch.full((enc.N, enc.M), float("nan"), dtype=torch.complex64, device="cuda")
    P.pinv_plan_copy_buffer(plan, P.BUF_R, R)
    torch.cuda.synchronize()
    P.pinv_plan_release(plan)
    return R.cpu().numpy().astype(np.complex128)


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("name", list(SHAPES) + ["n289_mask"])
def test_r_matches_oracle(P, ctx, name):
    w = synth.small_case(**SHAPES["n289_odd" if name == "n289_mask" else name])
    enc = w.enc
    if name == "n289_mask":   # 274 of a 20 x 19 grid's voxels
        base = synth.small_case(seed=305, nx=20, ny=19, C=14, K=1451, F=3).enc
        enc = dataclasses.replace(base, voxels=synth.circular_mask(20, 19, 0.96))
    assert enc.N ** 2 * enc.M >= (3e8 if enc.N % 32 == 0 else 1.5e9)
    ref = oracle.Build(enc, rel=1e-2).recon_matrix()
    e_half, e_fp32 = rel(get_r(P, ctx, enc), ref), rel(get_r(P, ctx, enc, cprod=P.CPROD_4M), ref)
    print(f"{name}: N={enc.N} M={enc.M} f16 pieces {e_half:.2e}, FP32 {e_fp32:.2e}")
    assert e_half <= 2.0 * e_fp32


@pytest.mark.parametrize("amp", [1e-15, 1e15])
def test_r_scales_with_the_coils(P, ctx, amp):
    """Sensitivities far from 1: every power of two is carried beside the
    pieces, so R only scales by 1 / amp (amp rounded to a power of two)."""
    enc = synth.small_case(**SHAPES["n289_odd"]).enc
    a = 2.0 ** round(np.log2(amp))
    r1 = get_r(P, ctx, enc)
    ra = get_r(P, ctx, dataclasses.replace(enc, coil=enc.coil * a))
    assert np.all(np.isfinite(ra))
    assert rel(ra * a, r1) < 1e-12


def test_products_are_unbiased(P, ctx):
    """The matrix instruction's cut-off products must leave no mean error in R:
    over the 8.4e6 entries of a 32 x 32, 4-coil R, independent errors average to
    2.4e-4 of their size; 1e-3 is four times that (a third of the bias that sums
    of one sign leave)."""
    enc = synth.small_case(seed=306, nx=32, ny=32, C=4, K=2048, F=3).enc
    plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP64, P.FLAG_UNCACHED)
    R = torch.empty((enc.N, enc.M), dtype=torch.complex128, device="cuda")
    P.pinv_plan_copy_buffer(plan, P.BUF_R, R)
    torch.cuda.synchronize()
    P.pinv_plan_release(plan)
    d = get_r(P, ctx, enc) - R.cpu().numpy()
    bias = abs(d.mean()) / np.sqrt(np.mean(np.abs(d) ** 2))
    print(f"mean error / rms error {bias:.1e}")
    assert bias < 1e-3


# ---------------------------------------------------------------------------
# applies of more than 32 frames
# ---------------------------------------------------------------------------
# Each value is within 2^-23 of the FP32 operand it stands for (two pieces), the
# dropped products of the second pieces are 2^-22 at most, and a segment's FP32
# sum rounds every 32 of at most 4096 columns: over random frames these add up to
# a few 2^-23; 2e-6 is 16 of them.
APPLY_TOL = 2e-6

APPLY_SHAPES = {
    # N ragged, M odd (8-byte loads of R and the data), one and two passes of frames
    "odd": (dict(seed=311, nx=17, ny=17, C=3, K=1173, F=3), (300, 2100)),
    # several segments with a short last one; frames below, at and past a tile
    "long": (dict(seed=312, nx=32, ny=20, C=2, K=4210, F=3), (56, 64, 65, 129)),
}


@pytest.mark.parametrize("flag", ["fp32", "r_fp64"])
@pytest.mark.parametrize("name", list(APPLY_SHAPES))
def test_apply_matches_own_r(P, ctx, name, flag):
    kw, frames = APPLY_SHAPES[name]
    enc = synth.small_case(**kw).enc
    N, M = enc.N, enc.M
    flags = P.FLAG_UNCACHED | (P.FLAG_R_FP64 if flag == "r_fp64" else 0)
    plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, flags)
    try:
        R = torch.empty((N, M), dtype=torch.complex64, device="cuda")
        P.pinv_plan_copy_buffer(plan, P.BUF_R, R)
        torch.cuda.synchronize()
        Rt = R.cpu().numpy().astype(np.complex128).T
        rng = np.random.default_rng(7)
        for F in frames:
            assert F * N * M >= 3e8   # below, the FP32 tiles run
            d = (rng.standard_normal((F, M)) + 1j * rng.standard_normal((F, M))).astype(np.complex64)
            d[1] *= np.float32(2.0 ** -90)    # every frame has a scale of its own
            d[2] *= np.float32(2.0 ** 90)
            d[3] = 0
            d[4, ::2] *= np.float32(1e-6)     # a wide range within one frame
            ref = d.astype(np.complex128) @ Rt
            x = torch.full((F, N), float("nan"), dtype=torch.complex64, device="cuda")
            dd = torch.from_numpy(d).cuda()
            P.pinv_apply(ctx, plan, dd, x)
            torch.cuda.synchronize()
            xs = x.cpu().numpy().astype(np.complex128)
            assert np.all(xs[3] == 0)
            keep = np.arange(F) != 3
            err = np.linalg.norm(xs - ref, axis=1)[keep] / np.linalg.norm(ref, axis=1)[keep]
            print(f"{name} {flag} F={F}: {err.max():.2e}")
            assert err.max() < APPLY_TOL
            # an infinity stays in its frame
            dd[5, M // 2] = complex(float("inf"), 0.0)
            y = torch.empty_like(x)
            P.pinv_apply(ctx, plan, dd, y)
            torch.cuda.synchronize()
            ok = torch.arange(F, device="cuda") != 5
            assert torch.equal(x[ok], y[ok]) and not torch.isfinite(torch.view_as_real(y[5])).any()
    finally:
        P.pinv_plan_release(plan)
