"""Blocked factorisation: L^-1 at the edges of its blocks, steps and launch forms.

Orders 1 to 17 and 63 to 129 sit at the edges of the 16-column sub-blocks, the
32-row tiles and the 64-column blocks; 1105 (18 blocks) is the first size tested
whose trailing updates start with more than 256 tiles of 64 x 64 and end with fewer;
1280 and 1281 are 20 and 21 blocks, the last order on one stream and the first with
a look-ahead.  Random samples and two coils; lambda at 1e-2 of the mean diagonal
bounds the condition number near 1e3.

Tolerance: the factor's backward error is at most about N 2^-53 (1.4e-13 at 1281),
the condition number raises it to 1.4e-10, and both sides have one: 1e-9.
"""
import numpy as np
import pytest

from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRIDS = {1: (1, 1), 15: (5, 3), 16: (4, 4), 17: (17, 1), 63: (9, 7), 64: (8, 8), 65: (13, 5),
         127: (127, 1), 129: (43, 3), 1105: (65, 17), 1280: (40, 32), 1281: (61, 21)}


@pytest.fixture(scope="module")
def P():
    from paper_2410_06129_amd import pinv
    return pinv


@pytest.fixture(scope="module")
def ctx(P):
    c = P.pinv_context_create(0)
    yield c
    P.pinv_context_destroy(c)


def encoding(N, zero=None):
    nx, ny = GRIDS[N]
    rng = np.random.default_rng(700 + N)
    coil = synth.coil_maps(nx, ny, 2, rng)
    if zero is not None:
        coil[:, zero] = 0.0
    k = (rng.random((N + 3, 2)) - 0.5) * [nx, ny]
    return synth.Encoding(nx, ny, k, coil=coil)


@pytest.mark.parametrize("nb", [64, 128])
@pytest.mark.parametrize("N", list(GRIDS))
def test_inverse_factor_at_block_edges(P, ctx, N, nb):
    plan = P.pinv_build(ctx, encoding(N), 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP64,
                        P.FLAG_UNCACHED | P.FLAG_KEEP_GRAM, nb=nb)
    try:
        P.pinv_plan_wait(plan)
        lam = P.pinv_plan_info_get(plan)["lambda_abs"]
        G, Li = (torch.full((N, N), float("nan"), dtype=torch.complex128, device="cuda") for _ in range(2))
        P.pinv_plan_copy_buffer(plan, P.BUF_GRAM, G)
        P.pinv_plan_copy_buffer(plan, P.BUF_LINV, Li)
        torch.cuda.synchronize()
    finally:
        P.pinv_plan_release(plan)
    A = np.tril(G.cpu().numpy(), -1)
    A = A + A.conj().T + np.diag(G.cpu().numpy().diagonal().real + lam)
    ref = np.linalg.solve(np.linalg.cholesky(A), np.eye(N))
    Li = Li.cpu().numpy()
    assert np.max(np.abs(np.triu(Li, 1)), initial=0.0) == 0.0
    assert np.max(np.abs(Li - ref)) <= 1e-9 * np.max(np.abs(ref))


@pytest.mark.parametrize("v", [0, 15, 16, 40, 63, 64, 100, 128])
def test_first_bad_column_is_reported(P, ctx, v):
    """A voxel that no coil sees has a zero row in the Gram matrix: with lambda = 0
    its pivot is exactly zero, the first that is not positive."""
    plan = P.pinv_build(ctx, encoding(129, zero=v), 0.0, P.LAMBDA_ABS, P.FP64, P.FLAG_UNCACHED)
    try:
        assert P.pinv_plan_wait_status(plan) == P.ERR_NOT_PD
        assert f"column {v}" in P.pinv_last_error()
    finally:
        P.pinv_plan_release(plan)
