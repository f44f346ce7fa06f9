"""Waits for more pieces than a wavefront has lanes, and for slices of which some have landed: the whole output of a
launch over 80 shards (its wait list is 80 pieces), the join of a run whose 128 transfers no GEMM consumes, and column
pieces that are more than 64 slices. Compared with the resident row-piece run, bit for bit. And the limit of a wait for
more than 64 pieces."""
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


def test_limit_counts_from_the_last_landing_across_batches(gpu):
    """One long transfer after the other, the 64th and the 65th of a wait: the wavefront watches 64 pieces at a time, and the
    landing that ends the first batch starts the limit anew for the second. Each of the two takes half of what the run
    takes (measured first), the limit is three quarters of it: no piece is late, two together would be."""
    dev, K = gpu["dev"], 4096
    rows = [[8]] * 63 + [[1 << 16]] * 2
    M = sum(r[0] for r in rows)
    A = torch.randint(-1000, 1000, (M, K), dtype=torch.int16, device=dev).view(torch.bfloat16)
    A_dev = torch.zeros_like(A)
    W = torch.zeros((K, 8), dtype=torch.bfloat16, device=dev)
    C = torch.zeros((M, 8), dtype=torch.bfloat16, device=dev)
    torch.cuda.synchronize()
    plan = ficco.ficco_plan_grouped(K, 8, rows, 1, ficco.FICCO_SHARD)
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, ficco.FICCO_MODE_COPY_ONLY)
        for _ in range(3):
            ficco.ficco_run(plan, A, A_dev, W, C, None, gpu["cs"], gpu["xs"])
            wall_us = ficco.ficco_query_stats(plan).wall_us
        print(f"two pieces of {rows[-1][0] * K * 2 >> 20} MiB in {wall_us:.0f} us", flush=True)
        assert wall_us > 4000
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_SPIN_LIMIT_US, int(wall_us * 0.75))
        for _ in range(2):
            ficco.ficco_run(plan, A, A_dev, W, C, None, gpu["cs"], gpu["xs"])
            ficco.ficco_query_stats(plan)                    # raises if a wait has given up
    finally:
        ficco.ficco_destroy(plan)
    assert torch.equal(A_dev.view(torch.int16), A.view(torch.int16))


@pytest.mark.parametrize("big", [0, 7, 15])
def test_tile_that_waits_for_128_pieces(gpu, big):
    """One row tile per expert over 16 peers x 8 steps of ragged pieces, one peer's far larger than the others: the pieces of a
    tile's two batches land in another order than they are listed in."""
    dev, K, N = gpu["dev"], 1024, 264
    rows = [[13 if j == big else 1 + (j + e) % 3 for e in range(2)] for j in range(16)]
    rows[big][1] = 6000
    M = sum(map(sum, rows))
    g = torch.Generator(device=dev).manual_seed(big)
    A = torch.randn((M, K), generator=g, device=dev).bfloat16()
    W = torch.randn((2 * K, N), generator=g, device=dev).bfloat16()
    out = []
    for c, schedule in ((8, ficco.FICCO_FINE_PERSISTENT), (1, ficco.FICCO_SERIAL)):
        A_dev = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device=dev)
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=dev)
        torch.cuda.synchronize()
        plan = ficco.ficco_plan_grouped(K, N, rows, c, schedule)
        try:
            print(f"experts, {c} pieces a peer, peer {big} the largest", flush=True)
            for _ in range(2):
                ficco.ficco_run(plan, A, A_dev, W, C, None, gpu["cs"], gpu["xs"])
                ficco.ficco_query_stats(plan)
        finally:
            ficco.ficco_destroy(plan)
        out.append(C)
    assert not torch.isnan(out[1].float()).any()
    assert torch.equal(out[0], out[1])
