"""The 64x128 tile, which the library picks for launches that leave CUs idle with every larger one, in each kernel that has
it - row pieces, column pieces, one launch per step, output streaming and expert-parallel - at the edges of the tile (one
row, one column block, remainders of eight columns) and with fewer k-tiles than its ring of six stages, as many and more: bit for
bit what a forced 256x256 tile gives. And that it stays the library's own choice: the option refuses it as before."""
import os
import sys

import pytest

import paper_2512_10236_amd as ficco

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import internal

torch = pytest.importorskip("torch")

CASES = [
    ("rows", 504, 768, 2056, 8, 1), ("rows", 4112, 128, 264, 4, 4), ("rows", 8224, 64, 120, 8, 4), ("rows", 8224, 384, 120, 8, 4), ("rows", 10240, 1088, 72, 8, 4),
    ("rows", 1024, 1024, 2040, 8, 2), ("rows", 624, 256, 3088, 1, 1), ("rows", 624, 320, 3088, 1, 1),
    ("rows", 624, 384, 3088, 1, 1), ("rows", 624, 448, 3088, 1, 1),
    ("columns", 504, 1024, 2056, 8, 3), ("columns", 2056, 384, 776, 8, 3), ("columns", 624, 320, 3088, 2, 5),
    ("fused", 16, 1088, 2056, 8, 2), ("fused", 624, 320, 3088, 2, 1),
    ("scatter", 520, 1088, 1032, 8, 1), ("scatter", 624, 256, 3088, 2, 1),
    ("experts", 1000, 1024, 1032, 4, 2), ("experts", 3000, 320, 520, 4, 4), ("experts", 300, 768, 3088, 8, 4)]
SCHEDULE = dict(rows=ficco.FICCO_FINE_PERSISTENT, columns=ficco.FICCO_FINE_2D, fused=ficco.FICCO_FINE_FUSED, scatter=ficco.FICCO_FINE_PERSISTENT)


def _plan(kind, M, K, N, G, c):
    if kind == "experts":
        rows = [[M // (2 * G)] * 2 for _ in range(G)]
        rows[0][1] += M - sum(map(sum, rows))
        return ficco.ficco_plan_grouped(K, N, rows, c, ficco.FICCO_FINE_PERSISTENT)
    plan = ficco.ficco_plan(M, K, N, G, c, SCHEDULE[kind])
    if kind == "scatter":
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_DIRECTION, ficco.FICCO_DIR_GEMM_RS)
    return plan


def test_option_refuses_the_tile():
    plan = ficco.ficco_plan(64, 64, 64, 1, 1, ficco.FICCO_FINE_PERSISTENT)
    try:
        for value in (-1, ficco.FICCO_TILE_256x192 + 1):
            with pytest.raises(ficco.FiccoError):
                ficco.ficco_plan_set(plan, ficco.FICCO_OPT_TILE, value)
    finally:
        ficco.ficco_destroy(plan)


@pytest.mark.parametrize("kind,M,K,N,G,c", CASES)
def test_rule_picks_the_tile(kind, M, K, N, G, c):
    plan = _plan(kind, M, K, N, G, c)
    try:
        assert internal.choose_tile(plan)[0] == (64, 128)
    finally:
        ficco.ficco_destroy(plan)


def _run(gpu, case, tile, A, W):
    kind, M, K, N, G, c = case
    dev = gpu["dev"]
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=dev)
    rs = kind == "scatter"
    A_dev = A if rs else torch.full_like(A, float("nan"))
    peers = [torch.full((M // G, N), float("nan"), dtype=torch.bfloat16, device=dev) for _ in range(G)] if rs else None
    torch.cuda.synchronize()
    plan = _plan(*case)
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_TILE, tile)
        for _ in range(2):
            ficco.ficco_run(plan, None if rs else A, A_dev, W, C, peers, gpu["cs"], gpu["xs"])
            ficco.ficco_query_stats(plan)
        info = ficco.ficco_plan_info(plan)
    finally:
        ficco.ficco_destroy(plan)
    if rs:
        assert torch.equal(torch.cat(peers).view(torch.int16), C.view(torch.int16))
    return C, (info.tile_m, info.tile_n)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%dx%dx%d-%dx%d" % c)
def test_small_tile_has_the_bits_of_the_large_one(gpu, case):
    kind, M, K, N, G, c = case
    g = torch.Generator(device=gpu["dev"]).manual_seed(M + K + N)
    A = torch.randn((M, K), generator=g, device=gpu["dev"]).bfloat16()
    W = torch.randn((2 * K if kind == "experts" else K, N), generator=g, device=gpu["dev"]).bfloat16()
    print(f"small tile {kind} {M}x{K}x{N} {G}x{c}", flush=True)
    got, tile = _run(gpu, case, ficco.FICCO_TILE_AUTO, A, W)
    want, _ = _run(gpu, case, ficco.FICCO_TILE_256x256, A, W)
    assert not torch.isnan(want.float()).any()
    assert torch.equal(got, want)
    assert tile == (64, 128)
