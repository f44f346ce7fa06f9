"""Waits of launches with many workgroups, most of which learn that a piece has landed from the workgroup that saw it: row
pieces of one and of several tiles, column pieces, one launch per step, expert-parallel, and the packed fused schedule, where it is
the copies into the packed input that they wait for. Every run of a plan gets another activation over a poisoned landing buffer, with runs that wait for
flags and runs that wait for nothing in between, and each result is that of the product alone, bit for bit."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PERSISTENT, FUSED, COLUMNS = ficco.FICCO_FINE_PERSISTENT, ficco.FICCO_FINE_FUSED, ficco.FICCO_FINE_2D
CASES = [("rows", PERSISTENT, 4096, 320, 256, 8, 1), ("rows", PERSISTENT, 4096, 256, 1032, 4, 4), ("rows", PERSISTENT, 2048, 192, 2048, 2, 1),
         ("rows", ficco.FICCO_SERIAL, 2048, 192, 2048, 8, 1), ("fused", FUSED, 4096, 256, 1032, 8, 2), ("packed", FUSED, 4096, 256, 1032, 8, 2),
         ("columns", COLUMNS, 2048, 640, 2048, 8, 3), ("experts", PERSISTENT, 3000, 256, 2056, 8, 2)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%d-%dx%dx%d-%dx%d" % c)
def test_results_of_runs_that_pass_landings_on(gpu, case):
    kind, schedule, M, K, N, G, c = case
    dev, cs, xs = gpu["dev"], gpu["cs"], gpu["xs"]
    g = torch.Generator(device=dev).manual_seed(M + K + N + c)
    experts = 2 if kind == "experts" else 1
    W = torch.randn((experts * K, N), generator=g, device=dev).bfloat16()
    if kind == "experts":
        rows = [[100 + 37 * j, 0] for j in range(G)]
        rows[0][1] = M - sum(r[0] for r in rows)
        plan = ficco.ficco_plan_grouped(K, N, rows, c, schedule)
    else:
        plan = ficco.ficco_plan(M, K, N, G, c, schedule)
    try:
        if kind == "packed":
            ficco.ficco_plan_set(plan, ficco.FICCO_OPT_PACKING, 1)
        alone, flags = ficco.FICCO_MODE_GEMM_ONLY, -2
        for run, mode in enumerate((0, 0, alone, 0, flags, 0, 0)):
            if mode == flags and kind == "packed":
                continue
            A = torch.randn((M, K), generator=g, device=dev).bfloat16()
            A_src = A.cpu().pin_memory() if mode == flags else A      # transfers over the host link: the waits are for flags
            A_dev = A.clone() if mode == alone and kind != "columns" else torch.full_like(A, float("nan"))
            C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=dev)
            torch.cuda.synchronize()
            print(f"passed on {case} run {run} mode {mode}", flush=True)
            ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, alone if mode == alone else ficco.FICCO_MODE_PAIR)
            ficco.ficco_run(plan, None if mode == alone else A_src, A_dev, W, C, None, cs, xs)
            ficco.ficco_query_stats(plan)
            if mode == alone and kind == "columns":
                continue                                              # (the landing buffer is K-sliced there: no product to compare)
            want = torch.empty_like(C)
            split = M - rows[0][1] if kind == "experts" else M
            for e, (r0, r1) in enumerate(((0, split), (split, M))[:experts]):
                single = ficco.ficco_plan(r1 - r0, K, N, 1, 1, PERSISTENT)
                try:
                    ficco.ficco_plan_set(single, ficco.FICCO_OPT_MODE, alone)
                    ficco.ficco_run(single, None, A[r0:r1], W[e * K:(e + 1) * K], want[r0:r1], None, cs, xs)
                    ficco.ficco_query_stats(single)
                finally:
                    ficco.ficco_destroy(single)
            assert torch.equal(C.view(torch.int16), want.view(torch.int16)), (run, mode)
    finally:
        ficco.ficco_destroy(plan)
