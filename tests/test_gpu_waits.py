"""Waits for more pieces than a wavefront has lanes, and for slices of which some have landed: the whole output of a
launch over 80 shards (its wait list is 80 pieces), the join of a run whose 128 transfers no GEMM consumes, and column
pieces that are more than 64 slices. Compared with the resident row-piece run, bit for bit."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(gpu, M, K, N, G, c, schedule, mode=None):
    dev = gpu["dev"]
    g = torch.Generator(device=dev).manual_seed(M + K + N)
    A = torch.randn((M, K), generator=g, device=dev).bfloat16()
    W = torch.randn((K, N), generator=g, device=dev).bfloat16()
    A_dev = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device=dev)
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=dev)
    torch.cuda.synchronize()
    plan = ficco.ficco_plan(M, K, N, G, c, schedule)
    try:
        if mode is not None:
            ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, mode)
        print(f"waits {M}x{K}x{N} shards {G} pieces {c} schedule {schedule}", flush=True)
        for _ in range(2):
            ficco.ficco_run(plan, A, A_dev, W, C, None, gpu["cs"], gpu["xs"])
            ficco.ficco_query_stats(plan)
    finally:
        ficco.ficco_destroy(plan)
    return A, A_dev, C


def test_launch_that_waits_for_eighty_pieces(gpu):
    C = _run(gpu, 80 * 16, 128, 256, 80, 1, ficco.FICCO_SERIAL)[2]
    want = _run(gpu, 80 * 16, 128, 256, 1, 1, ficco.FICCO_FINE_PERSISTENT)[2]
    assert not torch.isnan(C.float()).any()
    assert torch.equal(C, want)


def test_join_of_128_transfers(gpu):
    A, A_dev, _ = _run(gpu, 8 * 16 * 16, 128, 64, 8, 16, ficco.FICCO_FINE_PERSISTENT, mode=ficco.FICCO_MODE_COPY_ONLY)
    assert torch.equal(A_dev, A)


def test_more_slices_than_lanes(gpu):
    C = _run(gpu, 256, 64 * 70, 256, 2, 70, ficco.FICCO_FINE_2D)[2]
    want = _run(gpu, 256, 64 * 70, 256, 2, 1, ficco.FICCO_FINE_PERSISTENT)[2]
    assert torch.equal(C, want)
