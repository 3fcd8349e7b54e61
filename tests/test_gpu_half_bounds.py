"""Where FP32 plans leave f16 pieces for FP32 instructions: R on both sides of each bound
against the oracle, beside the same plan on FP32 instructions (4M), whose error R may
double at most (a value is held within 2^-24 rms in two pieces, 2^-25 in FP32)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    from paper_2410_06129_amd import pinv
    return pinv


@pytest.fixture(scope="module")
def ctx(P):
    c = P.pinv_context_create(0)
    yield c
    P.pinv_context_destroy(c)


def get_r(P, ctx, enc, lam=1e-2, **kw):
    plan = P.pinv_build(ctx, enc, lam, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED, **kw)
    P.pinv_plan_wait(plan)
    R = torch.full((enc.N, enc.M), float("nan"), dtype=torch.complex64, device="cuda")
    P.pinv_plan_copy_buffer(plan, P.BUF_R, R)
    torch.cuda.synchronize()
    P.pinv_plan_release(plan)
    return R.cpu().numpy().astype(np.complex128)


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def on_pieces(P, enc, lam=1e-2):
    """Plans of an N that is no multiple of 32 pad W's rows on f16 pieces."""
    assert enc.N % 32
    return (P.pinv_encoding_key(enc, lam, prec=P.FP32)[1]
            != P.pinv_encoding_key(enc, lam, prec=P.FP32, cprod=P.CPROD_4M)[1])


@pytest.mark.parametrize("nx,ny", [(17, 15), (20, 13)])   # 255 and 260 unknowns
def test_fewest_unknowns(P, ctx, nx, ny):
    enc = synth.small_case(seed=321, nx=nx, ny=ny, C=8, K=2900, F=1).enc
    assert enc.N ** 2 * enc.M >= 1.5e9 and on_pieces(P, enc) == (enc.N >= 256)
    ref = oracle.Build(enc, rel=1e-2).recon_matrix()
    e_auto, e_4m = rel(get_r(P, ctx, enc), ref), rel(get_r(P, ctx, enc, cprod=P.CPROD_4M), ref)
    print(f"N={enc.N}: {e_auto:.2e}, FP32 {e_4m:.2e}")
    assert e_auto <= 2.0 * e_4m


def test_maps_outside_the_mask_have_no_effect(P, ctx):
    """Sensitivities of voxels that are no unknowns (an unregularised ratio of coil images
    in the background) leave R as it is."""
    base = synth.small_case(seed=322, nx=20, ny=19, C=14, K=1451, F=1).enc
    vox = synth.circular_mask(20, 19, 0.96)
    outside = np.setdiff1d(np.arange(380), vox)
    r = []
    for filler in (0.0, 1e12, float("inf"), float("nan")):
        coil = base.coil.copy()
        coil[:, outside] = filler
        enc = dataclasses.replace(base, coil=coil, voxels=vox)
        assert on_pieces(P, enc)
        r.append(get_r(P, ctx, enc))
    assert np.all(np.isfinite(r[0])) and np.linalg.norm(r[0]) > 0
    for other in r[1:]:
        assert np.array_equal(r[0], other)


@pytest.mark.parametrize("lam", [1e-5, 1e-3])
def test_no_further_than_fp32(P, ctx, lam):
    """Short contractions round little, so E's own rounding is most of the error: one, into
    two pieces (2^-24), against those of FP32 tables and their products."""
    enc = synth.small_case(seed=324, nx=16, ny=16, C=8, K=1000, F=1).enc
    ref = oracle.Build(enc, rel=lam).recon_matrix()
    e_auto = rel(get_r(P, ctx, enc, lam), ref)
    e_4m = rel(get_r(P, ctx, enc, lam, cprod=P.CPROD_4M), ref)
    print(f"{e_auto:.2e}, FP32 {e_4m:.2e}")
    assert e_auto <= e_4m


def ramp(shape, axis, bits):
    """Powers of two from 1 down to 2^-bits along an axis, in a shuffled order."""
    n = shape[axis]
    w = 2.0 ** -np.round(bits * np.random.default_rng(5).permutation(n) / max(n - 1, 1))
    return w.reshape([-1 if i == axis else 1 for i in range(len(shape))])


@pytest.mark.parametrize("axis,bits,lam,pieces", [
    (1, 0, 1e-3, True), (1, 9, 1e-3, True), (1, 14, 1e-3, False), (1, 23, 1e-3, False), (1, 10, 1.0, False),
    (0, 4, 1e-3, True), (0, 14, 1e-3, False), (0, 23, 1e-3, False),
    (1, 0, 8.0, True), (1, 0, 12.0, False), (1, 0, 1e4, False),
])
def test_uneven_sensitivities(P, ctx, axis, bits, lam, pieces):
    """Sensitivities that differ between voxels (axis 1) or coils (axis 0) by up to 2^bits,
    and large shifts: no row of R, and no coil's columns, may be further from the FP64
    plan's than twice the FP32 instructions leave the worst of them."""
    base = synth.small_case(seed=323, nx=19, ny=17, C=8, K=1900, F=1).enc
    enc = dataclasses.replace(base, coil=base.coil * ramp(base.coil.shape, axis, bits))
    assert on_pieces(P, enc, lam) == pieces
    plan = P.pinv_build(ctx, enc, lam, P.LAMBDA_REL_MEAN_DIAG, P.FP64, P.FLAG_UNCACHED)
    ref = torch.empty((enc.N, enc.M), dtype=torch.complex128, device="cuda")
    P.pinv_plan_copy_buffer(plan, P.BUF_R, ref)
    torch.cuda.synchronize()
    P.pinv_plan_release(plan)
    ref = ref.cpu().numpy().reshape(enc.N, enc.C, enc.K)

    def worst(**kw):
        d = get_r(P, ctx, enc, lam, **kw).reshape(ref.shape) - ref
        return [max(np.sqrt((np.abs(d) ** 2).sum(ax) / (np.abs(ref) ** 2).sum(ax)))
                for ax in ((1, 2), (0, 2))]
    auto, fp32 = worst(), worst(cprod=P.CPROD_4M)
    print(f"rows {auto[0]:.1e} {fp32[0]:.1e} coils {auto[1]:.1e} {fp32[1]:.1e}")
    assert auto[0] <= 2.0 * fp32[0] and auto[1] <= 2.0 * fp32[1]


def images(P, ctx, enc, d, lam, mode, **kw):
    plan = P.pinv_build(ctx, enc, lam, mode, P.FP32, P.FLAG_UNCACHED | P.FLAG_R_FP64, **kw)
    P.pinv_plan_wait(plan)
    R = torch.empty((enc.N, enc.M), dtype=torch.complex64, device="cuda")
    P.pinv_plan_copy_buffer(plan, P.BUF_R, R)
    x = torch.full((d.shape[0], enc.N), float("nan"), dtype=torch.complex64, device="cuda")
    P.pinv_apply(ctx, plan, d, x)
    torch.cuda.synchronize()
    P.pinv_plan_release(plan)
    return x, R


def test_4m_keeps_an_fp64_formed_r_on_fp32(P, ctx):
    """AUTO's applies of many frames run on f16 pieces, 4M's on FP32 instructions, with the
    same R; each has its own cache key."""
    enc = synth.small_case(seed=325, nx=32, ny=32, C=4, K=2048, F=1).enc
    g = torch.Generator(device="cuda").manual_seed(1)
    d = torch.view_as_complex(torch.randn(100, enc.M, 2, device="cuda", generator=g))
    assert 100 * enc.N * enc.M >= 3e8
    x, R = images(P, ctx, enc, d, 1e-2, P.LAMBDA_REL_MEAN_DIAG)
    y, S = images(P, ctx, enc, d, 1e-2, P.LAMBDA_REL_MEAN_DIAG, cprod=P.CPROD_4M)
    assert torch.equal(R, S) and not torch.equal(x, y)
    assert float(torch.linalg.vector_norm(x - y) / torch.linalg.vector_norm(x)) < 5e-6
    key = [P.pinv_encoding_key(enc, 1e-2, prec=P.FP32, flags=P.FLAG_R_FP64, cprod=c)[0]
           for c in (P.CPROD_AUTO, P.CPROD_4M)]
    assert key[0] != key[1]


def test_applies_of_uneven_sensitivities(P, ctx):
    """Every second of 48 coils sees one half of the image, the others the other half and at
    2^-20 of the first, so that a voxel's whole value comes from samples far below the
    largest in their row: each half may be twice as far from R data as the FP32
    instructions (4M) leave it."""
    n, C, F = 24, 48, 300
    rng = np.random.default_rng(6)
    k = rng.uniform(-n / 2, n / 2, (100, 2))
    coil = synth.unit_complex_noise((C, n * n), rng)
    left = np.arange(n * n) % n < n // 2
    coil[0::2, ~left] = 0
    coil[1::2, left] = 0
    coil[1::2] *= 2.0 ** -20
    enc = synth.Encoding(n, n, k, t=None, coil=coil)
    assert F * enc.N * enc.M >= 3e8
    d = oracle.forward(enc, synth.unit_complex_noise((F, enc.N), rng))
    d = torch.from_numpy(d.astype(np.complex64)).cuda()
    err = {}
    for form in (P.CPROD_AUTO, P.CPROD_4M):
        x, R = images(P, ctx, enc, d, 2.0 ** -40, P.LAMBDA_ABS, cprod=form)
        ref = d.to(torch.complex128) @ R.to(torch.complex128).T.contiguous()
        e, ref = (v.reshape(F, n, n) for v in (x.to(torch.complex128) - ref, ref))
        err[form] = [float(torch.linalg.vector_norm(e[..., s]) / torch.linalg.vector_norm(ref[..., s]))
                     for s in (slice(0, n // 2), slice(n // 2, n))]
    print(err)
    for auto, fp32 in zip(err[P.CPROD_AUTO], err[P.CPROD_4M]):
        assert auto <= 2.0 * fp32
