"""The parts that tiles are cut into, 64x64 and 32x64, in each kernel that has them - row pieces, column pieces, one launch per step
and per shard, output streaming, expert-parallel - at their edges (few rows, one column block, remainders of rows and columns),
and over one to more than two rounds of their rings, odd and even k-tiles: bit for bit what a forced 256x256 tile gives. And a
plan tells the tile that was launched."""
import os
import sys

import pytest

import paper_2512_10236_amd as ficco

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import internal
import test_gpu_small_tile as small

torch = pytest.importorskip("torch")

T64x64, T32x64 = (64, 64), (32, 64)
SHARD = dict(small.SCHEDULE, shard=ficco.FICCO_SHARD)
CASES = [
    ("rows", 512, 1024, 1024, 4, 1, T64x64), ("rows", 1024, 1024, 1000, 8, 1, T64x64), ("rows", 1000, 576, 1000, 8, 1, T64x64),
    ("rows", 8, 64, 72, 8, 1, T32x64), ("rows", 132, 832, 136, 4, 1, T32x64), ("rows", 66, 4096, 520, 2, 1, T32x64),
    ("columns", 280, 1088, 776, 2, 2, T32x64), ("columns", 1000, 1088, 1000, 2, 3, T64x64),
    ("fused", 520, 1088, 1032, 4, 1, T64x64), ("fused", 264, 704, 264, 8, 1, T32x64),
    ("shard", 264, 1088, 520, 8, 1, T32x64), ("shard", 8000, 704, 1000, 8, 1, T64x64),
    ("scatter", 264, 704, 200, 8, 1, T32x64), ("scatter", 1024, 704, 1000, 8, 1, T64x64),
    ("experts", 665, 1024, 520, 4, 2, T32x64), ("experts", 1000, 704, 1000, 4, 1, T64x64)]


def _tile(case):
    plan = small._plan(*case[:6])
    try:
        return internal.choose_tile(plan)[0]
    finally:
        ficco.ficco_destroy(plan)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%dx%dx%d-%dx%d" % c[:6])
def test_rule_picks_the_part(case, monkeypatch):
    monkeypatch.setattr(small, "SCHEDULE", SHARD)
    assert _tile(case) == case[6]


@pytest.mark.parametrize("kind,M,K,N,G,c", [
    ("alone", 10240, 1600, 192, 1, 1), ("alone", 20224, 1472, 64, 1, 1), ("alone", 25600, 448, 64, 4, 2), ("columns", 8560, 12032, 168, 4, 2),
    ("scatter", 10344, 1024, 136, 4, 1), ("scatter", 23040, 2432, 64, 8, 1), ("fused", 9680, 5760, 184, 8, 1)])
def test_rule_picks_whole_tiles_where_they_fill_the_chip(kind, M, K, N, G, c):
    """Launches of more 64x128 tiles than CUs, each of which some whole tile does 2-18 % faster than 64x64."""
    assert -(-M // 64) * -(-N // 128) > internal.CUS
    plan = small._plan("rows" if kind == "alone" else kind, M, K, N, G, c)
    try:
        if kind == "alone":
            ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, ficco.FICCO_MODE_GEMM_ONLY)
        assert internal.choose_tile(plan)[0] not in (T64x64, T32x64)
    finally:
        ficco.ficco_destroy(plan)


@pytest.mark.parametrize("case", [("rows", 6144, 2816, 320, 8, 4), ("experts", 6144, 2240, 320, 8, 1)], ids=lambda c: c[0])
def test_rule_picks_parts_where_tiles_follow_their_pieces(case):
    """As many tiles, but those of the last step count, and they are few: 150 us against 161, 140 against 148 (sixteen peers)."""
    assert _tile(case) == T64x64


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%dx%dx%d-%dx%d" % c[:6])
def test_parts_have_the_bits_of_the_large_tile(gpu, case, monkeypatch):
    monkeypatch.setattr(small, "SCHEDULE", SHARD)
    kind, M, K, N = case[:4]
    g = torch.Generator(device=gpu["dev"]).manual_seed(M + K + N)
    A = torch.randn((M, K), generator=g, device=gpu["dev"]).bfloat16()
    W = torch.randn((2 * K if kind == "experts" else K, N), generator=g, device=gpu["dev"]).bfloat16()
    print(f"tile part {case}", flush=True)
    got, tile = small._run(gpu, case[:6], ficco.FICCO_TILE_AUTO, A, W)
    want, _ = small._run(gpu, case[:6], ficco.FICCO_TILE_256x256, A, W)
    assert not torch.isnan(want.float()).any()
    assert torch.equal(got, want)
    assert tile == case[6]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,part,ring", [(40, 72, T32x64, 12), (1000, 1000, T64x64, 8)])
def test_parts_over_their_rings(gpu, M, N, part, ring):
    g = torch.Generator(device=gpu["dev"]).manual_seed(M)
    for k_tiles in range(1, 2 * ring + 4):
        K = 64 * k_tiles
        A = torch.randn((M, K), generator=g, device=gpu["dev"]).bfloat16()
        W = torch.randn((K, N), generator=g, device=gpu["dev"]).bfloat16()
        out = []
        for tile in (ficco.FICCO_TILE_AUTO, ficco.FICCO_TILE_256x256):
            out.append(torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=gpu["dev"]))
            print(f"ring {M}x{K}x{N} tile {tile}", flush=True)
            torch.cuda.synchronize()
            plan = ficco.ficco_plan(M, K, N, 1, 1, ficco.FICCO_FINE_PERSISTENT)
            try:
                ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, ficco.FICCO_MODE_GEMM_ONLY)
                ficco.ficco_plan_set(plan, ficco.FICCO_OPT_TILE, tile)
                assert tile or internal.choose_tile(plan)[0] == part
                ficco.ficco_run(plan, None, A, W, out[-1], None, gpu["cs"], gpu["xs"])
                ficco.ficco_query_stats(plan)
            finally:
                ficco.ficco_destroy(plan)
        assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16)), K
