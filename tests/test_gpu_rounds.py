"""How a resident launch hands out its tiles: by rank alone, by rank and then by draws, and by draws from uneven lists.
The shapes sit on either side of the lines (one round exactly, one tile more, a last partial round, lists that differ
by a row of tiles, a launch long enough to draw its last quarter); every run is repeated, since the counters are never
reset, and compared with the launch that has no lists (the serial schedule), bit for bit."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,tile", [
    (8192, 4096, ficco.FICCO_TILE_128x256),        # 1024 tiles: four rounds by rank
    (32 * 257, 256, ficco.FICCO_TILE_32x256),      # one round and one tile: lists of 33 and 32
    (32 * 300, 256, ficco.FICCO_TILE_32x256),      # a partial second round
    (32 * 9, 256 * 28, ficco.FICCO_TILE_32x256),   # 9 row tiles over 8 classes: uneven lists, draws and stealing
    (32 * 700, 256 * 5, ficco.FICCO_TILE_32x256),  # 14 rounds: the last quarter is drawn
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
