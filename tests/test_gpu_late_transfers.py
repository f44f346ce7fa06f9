"""ficco_query_stats() of a run whose transfers start late: output blocks that wait for a kernel which stands behind more than
a second of other work on its stream. It waits for them, and gives the spans of all."""
import time

import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_transfers_behind_a_second_of_other_work(gpu):
    M, K, N, G = 1024, 256, 512, 4
    dev, cs, xs = gpu["dev"], gpu["cs"], gpu["xs"]
    g = torch.Generator(device=dev).manual_seed(1)
    A, W = (torch.randn(s, generator=g, device=dev).bfloat16() for s in ((M, K), (K, N)))
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=dev)
    peers = [torch.full((M // G, N), float("nan"), dtype=torch.bfloat16, device=dev) for _ in range(G)]
    plan = ficco.ficco_plan(M, K, N, G, 2, ficco.FICCO_FINE_PERSISTENT)
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_DIRECTION, ficco.FICCO_DIR_GEMM_RS)
        with torch.cuda.stream(cs):
            torch.cuda._sleep(1000000)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            torch.cuda._sleep(10000000)
            torch.cuda.synchronize()
            per_s = 10000000 / (time.perf_counter() - t0)
            ficco.ficco_run(plan, None, A, W, C, peers, cs, xs)
            quick = ficco.ficco_query_stats(plan)
            C.fill_(float("nan"))
            for p in peers:
                p.fill_(float("nan"))
            torch.cuda.synchronize()
            print("late transfers", flush=True)
            t0 = time.perf_counter()
            torch.cuda._sleep(int(1.3 * per_s))
            ficco.ficco_run(plan, None, A, W, C, peers, cs, xs)
            late = ficco.ficco_query_stats(plan)
            assert time.perf_counter() - t0 > 1.1, "the work in front of the run was too short for this test"
        assert late.n_copies == quick.n_copies == 2 * G and late.copy_span_us > 0 and late.copy_busy_us > 0
        assert torch.equal(torch.cat(peers).view(torch.int16), C.view(torch.int16)) and not torch.isnan(C.float()).any()
    finally:
        ficco.ficco_destroy(plan)
