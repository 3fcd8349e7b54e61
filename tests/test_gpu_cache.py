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


def device_used():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_many_sizes_do_not_add_up(P):
    """Plans of 20 sizes built and released in turn: the context keeps at most twice what
    was in use at once (and 256 MB in each of its two parts), not a block of every size."""
    ctx = P.pinv_context_create(0)
    try:
        encs = [synth.small_case(seed=1310 + i, nx=40, ny=32, C=8, K=int(6000 * 1.06 ** i), F=1).enc
                for i in range(20)]
        size = [2 * 8 * e.N * e.M for e in encs]        # W and R
        assert sum(size) > 3 * (2 * 1.3 * size[-1] + (512 << 20))
        base = device_used()
        for e in encs + encs[::-1]:
            plan = P.pinv_build(ctx, e, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
            P.pinv_plan_wait(plan)
            P.pinv_plan_release(plan)
        kept = device_used() - base
        print(f"kept {kept >> 20} MB of {sum(size) >> 20}")
        assert kept < 2 * 1.3 * size[-1] + (512 << 20)
        P.pinv_context_trim(ctx)
        assert device_used() - base < 256 << 20
    finally:
        P.pinv_context_destroy(ctx)


def test_idle_memory_stays_within_the_budget(P):
    """A context with room for three plans keeps no more than that of released ones."""
    encs = [synth.small_case(seed=1340 + i, nx=24, ny=24, C=4, K=3000 + 700 * i, F=1).enc for i in range(8)]
    foot = P.pinv_encoding_key(encs[-1], 1e-2, prec=P.FP64)[1]
    ctx = P.pinv_context_create(0, 2 * foot)
    try:
        base = device_used()
        for e in encs:
            plan = P.pinv_build(ctx, e, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP64, P.FLAG_UNCACHED)
            P.pinv_plan_wait(plan)
            P.pinv_plan_release(plan)
        assert device_used() - base < 3 * foot
    finally:
        P.pinv_context_destroy(ctx)


def test_threads_and_streams_share_the_memory(P):
    """Four threads, each on its own stream, build, apply and release plans of different
    sizes without waiting for the device in between: every image equals the one computed
    alone."""
    ctx = P.pinv_context_create(0)
    try:
        work = []
        for i in range(6):
            e = synth.small_case(seed=1350 + i, nx=16 + 4 * i, ny=24, C=4, K=900 + 150 * i, F=1).enc
            for F, steps in ((70 + 40 * i, 1), (3, 0)):
                d = frames(F, e.M, 10 * i + F)
                want = torch.empty(F, e.N, dtype=torch.complex64, device="cuda")
                work.append((e, d, steps, want))
        for e, d, steps, want in work:
            plan = P.pinv_build(ctx, e, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
            P.pinv_apply(ctx, plan, d, want, refine_steps=steps)
            torch.cuda.synchronize()
            P.pinv_plan_release(plan)
        failed = []

        def thread(k):
            try:
                torch.cuda.set_device(0)
                s = torch.cuda.Stream()
                order = np.random.default_rng(k).permutation(3 * len(work)) % len(work)
                outs = [torch.full_like(work[j][3], float("nan")) for j in order]
                torch.cuda.current_stream().synchronize()
                for j, x in zip(order, outs):
                    e, d, steps, _ = work[j]
                    plan = P.pinv_build(ctx, e, 1e-2, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED, stream=s)
                    P.pinv_apply(ctx, plan, d, x, refine_steps=steps, stream=s)
                    P.pinv_plan_release(plan)
                s.synchronize()
                for j, x in zip(order, outs):
                    if not torch.equal(x, work[j][3]):
                        failed.append((k, int(j)))
            except Exception as e:  # noqa: BLE001
                failed.append((k, repr(e)))
        threads = [threading.Thread(target=thread, args=(k,)) for k in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not failed, failed
    finally:
        P.pinv_context_destroy(ctx)
