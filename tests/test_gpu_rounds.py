"""How a resident launch hands out its tiles: by rank alone, with spare places that take what uneven lists have too many, by
rank and then by draws, and by draws from uneven lists. The shapes sit on either side of the lines (one round exactly, one
tile more, a last partial round, lists that differ by a row of tiles, the longest launch by rank, launches long enough to
draw); every run is repeated, since the counters are never
reset, and compared with the launch that has no lists (the serial schedule), bit for bit."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,tile", [
    (8192, 4096, ficco.FICCO_TILE_128x256),        # 1024 tiles: four rounds by rank
    (32 * 257, 256, ficco.FICCO_TILE_32x256),      # one round and one tile: lists of 33 and 32
    (32 * 300, 256, ficco.FICCO_TILE_32x256),      # a partial second round
    (32 * 9, 256 * 28, ficco.FICCO_TILE_32x256),   # 9 row tiles over 8 classes: uneven lists in one round
    (32 * 21, 256 * 24, ficco.FICCO_TILE_32x256),  # uneven lists, two rounds
    (2654, 3008, ficco.FICCO_TILE_128x128),        # the same in one round of two workgroups per CU
    (32 * 9, 256 * 455, ficco.FICCO_TILE_32x256),  # uneven lists, sixteen rounds: the longest launch by rank
    (32 * 9, 256 * 560, ficco.FICCO_TILE_32x256),  # uneven lists, twenty rounds: draws and stealing
    (32 * 1400, 256 * 5, ficco.FICCO_TILE_32x256), # 28 rounds: the last quarter is drawn
    (32 * 700, 256 * 5, ficco.FICCO_TILE_32x256),  # 14 rounds by rank
    (40, 24, ficco.FICCO_TILE_32x256),             # fewer tiles than lists
])
def test_every_tile_is_taken_once_in_every_run(gpu, M, N, tile):
    dev, K = gpu["dev"], 128
    g = torch.Generator(device=dev).manual_seed(M + N)
    A = torch.randn(M, K, generator=g, device=dev).bfloat16()
    W = torch.randn(K, N, generator=g, device=dev).bfloat16()

    def plan(schedule):
        p = ficco.ficco_plan(M, K, N, 1, 1, schedule)
        ficco.ficco_plan_set(p, ficco.FICCO_OPT_MODE, ficco.FICCO_MODE_GEMM_ONLY)
        ficco.ficco_plan_set(p, ficco.FICCO_OPT_TILE, tile)
        return p

    def run(p):
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=dev)
        torch.cuda.synchronize()
        print(f"rounds {M}x{K}x{N} tile {tile}", flush=True)
        ficco.ficco_run(p, None, A, W, C, None, gpu["cs"], gpu["xs"])
        ficco.ficco_query_stats(p)
        return C

    serial, resident = plan(ficco.FICCO_SERIAL), plan(ficco.FICCO_FINE_PERSISTENT)
    try:
        want = run(serial)
        assert not torch.isnan(want.float()).any()
        for _ in range(3):
            assert torch.equal(run(resident), want)
    finally:
        ficco.ficco_destroy(serial)
        ficco.ficco_destroy(resident)
