"""The device memory a context keeps between calls: used beside captures of other streams,
by several threads and streams at once, and by encodings of many sizes."""
import threading

import numpy as np
import pytest

from paper_2410_06129_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    from paper_2410_06129_amd import pinv
    return pinv


def frames(F, M, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.view_as_complex(torch.randn(F, M, 2, device="cuda", generator=g))


def test_new_scratch_beside_another_streams_capture(P):
    """A capture in the strict mode (global: no thread may allocate or query) is open on one
    stream while another thread applies with scratch that the context does not hold yet:
    neither the apply nor the capture fails."""
    enc = synth.small_case(seed=1300, nx=32, ny=32, C=4, K=1000, F=1).enc
    ctx = P.pinv_context_create(0)
    try:
        plan = P.pinv_build(ctx, enc, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
        P.pinv_plan_wait(plan)
        d, side = frames(100, enc.M, 1), torch.cuda.Stream()
        x, want = (torch.empty(100, enc.N, dtype=torch.complex64, device="cuda") for _ in range(2))
        a = torch.zeros(64, device="cuda")
        torch.cuda.synchronize()
        failed = []

        def work():
            try:
                P.pinv_apply(ctx, plan, d, x, stream=side)
            except Exception as e:  # noqa: BLE001
                failed.append(e)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="global"):
            a += 1
            t = threading.Thread(target=work)
            t.start()
            t.join()
            a += 1
        assert not failed, failed
        torch.cuda.synchronize()
        a.zero_()
        graph.replay()
        P.pinv_apply(ctx, plan, d, want)
        torch.cuda.synchronize()
        assert torch.all(a == 2) and torch.equal(x, want)
        P.pinv_plan_release(plan)
    finally:
        P.pinv_context_destroy(ctx)
