"""pinv_apply recorded into a graph: its scratch belongs to the capture, so replays with
eager applies of other sizes between them give the eager results bit for bit (an f16-piece
apply, whose packed operands are scratch, and one without scratch)."""
import numpy as np
import pytest

from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("F", [1, 100])
def test_replays_equal_eager_applies(F):
    from paper_2410_06129_amd import pinv as P
    enc = synth.small_case(seed=1200, nx=32, ny=32, C=4, K=1000, F=1).enc
    assert (F * enc.N * enc.M >= 3e8) == (F == 100)   # f16 pieces
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
        P.pinv_plan_wait(plan)
        d = torch.zeros(F, enc.M, dtype=torch.complex64, device="cuda")
        x, y = (torch.full((F, enc.N), float("nan"), dtype=torch.complex64, device="cuda") for _ in range(2))
        other = torch.randn(F + 30, enc.M, dtype=torch.complex64, device="cuda")
        z = torch.empty(F + 30, enc.N, dtype=torch.complex64, device="cuda")
        P.pinv_apply(ctx, plan, d, y)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            P.pinv_apply(ctx, plan, d, x)
        rng = np.random.default_rng(5)
        for _ in range(4):
            d.copy_(torch.from_numpy(synth.unit_complex_noise((F, enc.M), rng).astype(np.complex64)))
            P.pinv_apply(ctx, plan, other, z)   # (would reuse the capture's scratch if it could)
            graph.replay()
            P.pinv_apply(ctx, plan, d, y)
            torch.cuda.synchronize()
            assert torch.equal(x, y)
        del graph
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)


def test_refined_apply_is_refused_under_capture():
    """Refused before anything is recorded, alone and in a group; the capture goes on."""
    from paper_2410_06129_amd import pinv as P
    enc = synth.small_case(seed=1201, nx=16, ny=12, C=2, K=300, F=1).enc
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
        P.pinv_plan_wait(plan)
        d = torch.randn(1, enc.M, dtype=torch.complex64, device="cuda")
        x, y = (torch.full((1, enc.N), float("nan"), dtype=torch.complex64, device="cuda") for _ in range(2))
        P.pinv_apply(ctx, plan, d, y)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for call in (lambda: P.pinv_apply(ctx, plan, d, x, refine_steps=1),
                         lambda: P.pinv_apply_grouped(ctx, [(plan, d, x)], 1)):
                with pytest.raises(P.PinvError) as e:
                    call()
                assert e.value.status == P.ERR_UNSUPPORTED
            P.pinv_apply(ctx, plan, d, x)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, y)
        P.pinv_apply(ctx, plan, d, x, refine_steps=1)   # not under capture
        torch.cuda.synchronize()
        del graph
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)


def test_scratch_of_gone_graphs_is_released():
    """Recorded again and again, graphs leave their scratch with the context; it goes back
    to the device on request, and later captures take new scratch."""
    from paper_2410_06129_amd import pinv as P
    F = 400
    enc = synth.small_case(seed=1202, nx=32, ny=32, C=4, K=4000, F=1).enc
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
        P.pinv_plan_wait(plan)
        d = torch.randn(F, enc.M, dtype=torch.complex64, device="cuda")
        x, y = (torch.full((F, enc.N), float("nan"), dtype=torch.complex64, device="cuda") for _ in range(2))
        P.pinv_apply(ctx, plan, d, y)
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())

        def record():
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                P.pinv_apply(ctx, plan, d, x)
            return graph

        def used():
            torch.cuda.synchronize()
            free, total = torch.cuda.mem_get_info()
            return total - free
        first = record()
        del first
        P.pinv_context_release_captures(ctx)
        before = used()
        graphs = [record() for _ in range(6)]
        scratch = 8 * (enc.N + F) * enc.M // 2    # at least half of R and the data, packed
        assert used() - before >= 5 * scratch
        del graphs
        P.pinv_context_release_captures(ctx)
        assert used() - before < scratch
        graph = record()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, y)
        del graph
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)
