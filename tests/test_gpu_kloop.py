"""The k loop at its shortest: k extents of one k-tile up to more than every ring holds, for every tile that can be asked for
(the 64x128 one has tests of its own), on a ragged product. Against an fp64 product rounded once, within one bf16 step of the result (the fp32 sums of at most 576
terms are off by less than 576 * 2^-24 of the sum of magnitudes, far below half a step, so only a rounding that falls the
other way is left), and bit for bit between the tile shapes."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILES = range(ficco.FICCO_TILE_256x256, ficco.FICCO_TILE_256x192 + 1)


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 576])
def test_short_k_for_every_tile_shape(gpu, K):
    dev, M, N = gpu["dev"], 300, 264
    g = torch.Generator(device=dev).manual_seed(K)
    A = torch.randn(M, K, generator=g, device=dev).bfloat16()
    W = (torch.randn(K, N, generator=g, device=dev) * K ** -0.5).bfloat16()
    exact = A.double() @ W.double()
    want = exact.to(torch.bfloat16).double()
    first = None
    for tile in TILES:
        p = ficco.ficco_plan(M, K, N, 1, 1, ficco.FICCO_FINE_PERSISTENT)
        ficco.ficco_plan_set(p, ficco.FICCO_OPT_MODE, ficco.FICCO_MODE_GEMM_ONLY)
        ficco.ficco_plan_set(p, ficco.FICCO_OPT_TILE, tile)
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=dev)
        torch.cuda.synchronize()
        print(f"k loop K={K} tile {tile}", flush=True)
        ficco.ficco_run(p, None, A, W, C, None, gpu["cs"], gpu["xs"])
        ficco.ficco_query_stats(p)
        ficco.ficco_destroy(p)
        assert ((C.double() - want).abs() <= 2.0 ** -7 * exact.abs() + 1e-5).all()
        first = C if first is None else first
        assert torch.equal(C, first)
