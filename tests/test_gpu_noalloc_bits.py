"""pinv_apply_noalloc gives pinv_apply's results bit for bit, also where the fixed region
holds less than the allocating call takes: E^H d in shorter passes over the grids or in
slabs of F^H, and contractions in parts beside vectors that nearly fill the region."""
import pytest

from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

REGION = 512 << 20

CASES = {
    # f16 pieces and gridding, nothing short
    "pieces": (dict(seed=1401, nx=32, ny=32, C=4, K=2000, F=1), 200, 1, {}),
    # the refinement vectors take half of the region: shorter passes over the grids
    "grids": (dict(seed=1402, nx=32, ny=32, C=2, K=600, F=1), 5400, 2, {}),
    # slabs of F^H (a map, so no gridding)
    "slabs": (dict(seed=1403, nx=32, ny=32, C=4, K=5000, F=1, b0=True), 900, 1, {}),
    # a Gram over all rows: the residual's data vector (16 F M bytes) fills the region
    "parts": (dict(seed=1404, nx=32, ny=32, C=16, K=32250, F=1), 64, 1, dict(gram="FULL")),
}


@pytest.mark.parametrize("name", list(CASES))
def test_bits(name):
    from paper_2410_06129_amd import pinv as P
    kw, F, steps, opts = CASES[name]
    enc = synth.small_case(**kw).enc
    if name == "parts":   # no room for the triangular products' 8 parts beside the vectors
        vectors = 16 * F * enc.M + 16 * F * enc.N
        assert vectors < REGION < vectors + 8 * 16 * F * enc.N
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED,
                            **({"gram": P.GRAM_FULL} if opts else {}))
        P.pinv_plan_wait(plan)
        g = torch.Generator(device="cuda").manual_seed(3)
        d = torch.view_as_complex(torch.randn(F, enc.M, 2, device="cuda", generator=g))
        x, y = (torch.full((F, enc.N), float("nan"), dtype=torch.complex64, device="cuda") for _ in range(2))
        P.pinv_apply(ctx, plan, d, x, refine_steps=steps)
        P.pinv_apply_noalloc(ctx, plan, d, y, refine_steps=steps)
        torch.cuda.synchronize()
        assert torch.all(torch.isfinite(torch.view_as_real(x)))
        assert torch.equal(x, y)
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)
