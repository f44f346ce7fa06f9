"""The 64x128 tile, which the library picks for launches that leave CUs idle with every larger one, on row pieces,
column pieces and the expert-parallel kernel, at the edges of the tile (one row, one column block, remainders, more k-tiles
than its ring of six stages and fewer): bit for bit what a forced 256x256 tile gives. And that it stays the library's own
choice: the option refuses it as before."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")


def test_option_refuses_the_tile():
    plan = ficco.ficco_plan(64, 64, 64, 1, 1, ficco.FICCO_FINE_PERSISTENT)
    try:
        for value in (-1, ficco.FICCO_TILE_256x192 + 1):
            with pytest.raises(ficco.FiccoError):
                ficco.ficco_plan_set(plan, ficco.FICCO_OPT_TILE, value)
    finally:
        ficco.ficco_destroy(plan)


def _run(gpu, make, tile, A, W, M, N):
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=gpu["dev"])
    A_dev = torch.full_like(A, float("nan"))
    torch.cuda.synchronize()
    plan = make()
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_TILE, tile)
        for _ in range(2):
            ficco.ficco_run(plan, A, A_dev, W, C, None, gpu["cs"], gpu["xs"])
            ficco.ficco_query_stats(plan)
        info = ficco.ficco_plan_info(plan)
    finally:
        ficco.ficco_destroy(plan)
    return C, (info.tile_m, info.tile_n)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,M,K,N,G,c", [
    ("rows", 512, 1024, 1024, 4, 1), ("rows", 8, 1024, 136, 8, 1), ("rows", 8 * 65, 1088, 264, 8, 1), ("rows", 2 * 64 * 4, 4096, 128, 2, 4),
    ("rows", 64, 384, 768, 1, 1), ("rows", 1024, 1024, 2040, 8, 2), ("columns", 512, 1024, 1024, 4, 3), ("columns", 130, 1088, 776, 2, 2),
    ("experts", 700, 1024, 520, 4, 2)])
def test_small_tile_has_the_bits_of_the_large_one(gpu, kind, M, K, N, G, c):
    g = torch.Generator(device=gpu["dev"]).manual_seed(M + K + N)
    A = torch.randn((M, K), generator=g, device=gpu["dev"]).bfloat16()
    W = torch.randn((2 * K if kind == "experts" else K, N), generator=g, device=gpu["dev"]).bfloat16()
    if kind == "experts":
        rows = [[M // (2 * G)] * 2 for _ in range(G)]
        rows[0][1] += M - sum(map(sum, rows))
        make = lambda: ficco.ficco_plan_grouped(K, N, rows, c, ficco.FICCO_FINE_PERSISTENT)
    else:
        make = lambda: ficco.ficco_plan(M, K, N, G, c, ficco.FICCO_FINE_PERSISTENT if kind == "rows" else ficco.FICCO_FINE_2D)
    print(f"small tile {kind} {M}x{K}x{N} {G}x{c}", flush=True)
    got, tile = _run(gpu, make, ficco.FICCO_TILE_AUTO, A, W, M, N)
    want, _ = _run(gpu, make, ficco.FICCO_TILE_256x256, A, W, M, N)
    assert not torch.isnan(want.float()).any()
    assert torch.equal(got, want)
    assert tile[1] in (128, 256) and tile[0] <= 128, tile
    if (M, K, N) == (512, 1024, 1024):
        assert tile == (64, 128)
