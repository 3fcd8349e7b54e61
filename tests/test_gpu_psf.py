"""Point-spread-function Gram at the edges of its sample splits: fewer samples than
one split's 32, one more, a ragged last split, offset grids of one and of several
64 x 64 tiles (up to 64 x 64 offsets is one), against the oracle within 1e-12 of the
largest element (FP64 sums of at most 1500 unit-size terms)."""
import numpy as np
import pytest

import oracle
from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,K", [(2, 2, 31), (3, 2, 33), (5, 6, 64), (9, 7, 65), (32, 3, 1023),
                                     (33, 5, 527), (40, 33, 1500)])
def test_short_splits_match_oracle(nx, ny, K):
    from paper_2410_06129_amd import pinv as P
    rng = np.random.default_rng(800 + K)
    enc = synth.Encoding(nx, ny, (rng.random((K, 2)) - 0.5) * [nx, ny])
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP64,
                            P.FLAG_UNCACHED | P.FLAG_NO_R, gram=P.GRAM_PSF)
        P.pinv_plan_wait(plan)
        G = torch.full((enc.N, enc.N), float("nan"), dtype=torch.complex128, device="cuda")
        P.pinv_plan_copy_buffer(plan, P.BUF_GRAM, G)
        torch.cuda.synchronize()
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)
    Go = oracle.gram(enc)
    assert np.max(np.abs(G.cpu().numpy() - Go)) <= 1e-12 * np.max(np.abs(Go))
