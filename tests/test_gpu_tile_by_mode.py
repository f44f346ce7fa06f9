"""The tile of a run follows from the plan and the run's mode, whatever ran before: each mode on a fresh plan, then on one
plan in both orders and behind the loss profiler, at a shape whose pair and whose GEMM alone get different tiles, with the
same result bit for bit (the counters of the tile lists go on from run to run)."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M, K, N, G, C = 8192, 4096, 768, 8, 2
PAIR, ALONE, BOTH = ficco.FICCO_MODE_PAIR, ficco.FICCO_MODE_GEMM_ONLY, ficco.FICCO_MODE_INDEPENDENT


@pytest.fixture(scope="module")
def operands(gpu):
    g = torch.Generator(device=gpu["dev"]).manual_seed(5)
    A = torch.randn((M, K), generator=g, device=gpu["dev"]).bfloat16()
    W = torch.randn((K, N), generator=g, device=gpu["dev"]).bfloat16()
    torch.cuda.synchronize()
    return A, W, A.clone(), torch.empty((M, N), dtype=torch.bfloat16, device=gpu["dev"])


def _run(gpu, plan, mode, ops):
    A, W, A_dev, out = ops
    print(f"mode {mode}", flush=True)
    ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, mode)
    out.fill_(7.0)
    torch.cuda.synchronize()
    ficco.ficco_run(plan, None if mode == ALONE else A, A_dev, W, out, None, gpu["cs"], gpu["xs"])
    ficco.ficco_query_stats(plan)
    info = ficco.ficco_plan_info(plan)
    return (info.tile_m, info.tile_n, info.resident_grid), out.view(torch.int16).clone()


def _fresh(gpu, mode, ops):
    plan = ficco.ficco_plan(M, K, N, G, C, ficco.FICCO_FINE_PERSISTENT)
    try:
        return _run(gpu, plan, mode, ops)
    finally:
        ficco.ficco_destroy(plan)


def test_tile_does_not_depend_on_what_ran_before(gpu, operands):
    tile, bits = {}, {}
    for mode in (PAIR, ALONE, BOTH):
        tile[mode], bits[mode] = _fresh(gpu, mode, operands)
        assert torch.equal(bits[mode], bits[PAIR])
    assert tile[PAIR] != tile[ALONE], "the shape no longer tells the two apart: take another one"
    for order in ((PAIR, ALONE, PAIR, BOTH, PAIR), (ALONE, PAIR, ALONE), (BOTH, PAIR)):
        plan = ficco.ficco_plan(M, K, N, G, C, ficco.FICCO_FINE_PERSISTENT)
        try:
            for mode in order:
                got, out = _run(gpu, plan, mode, operands)
                assert got == tile[mode], (order, mode)
                assert torch.equal(out, bits[PAIR]), (order, mode)
        finally:
            ficco.ficco_destroy(plan)


def test_loss_profile_leaves_the_pair_its_tile(gpu, operands):
    A, W, A_dev, out = operands
    pair = _fresh(gpu, PAIR, operands)[0]
    plan = ficco.ficco_plan(M, K, N, G, C, ficco.FICCO_FINE_PERSISTENT)
    try:
        ficco.ficco_profile_losses(plan, A, A_dev, W, out, gpu["cs"], gpu["xs"], 1, 2)
        info = ficco.ficco_plan_info(plan)
        assert (info.tile_m, info.tile_n, info.resident_grid) == pair, "the losses are those of the pair's launches"
        assert _run(gpu, plan, PAIR, operands)[0] == pair
    finally:
        ficco.ficco_destroy(plan)


@pytest.mark.parametrize("m,k,n,c,lists", [(4096, 256, 256, 1, 2), (32768, 512, 512, 1, 4), (1024, 1024, 1536, 4, 8)])
def test_column_lists_are_taken_wherever_a_tile_fits_them(gpu, m, k, n, c, lists):
    """Shapes whose own tile is too wide for the lists: they are taken all the same, before the first run and after it, and
    more lists than columns of the narrowest whole tile are refused, also where the rule would cut the launch into parts."""
    g = torch.Generator(device=gpu["dev"]).manual_seed(7)
    ops = (torch.randn((m, k), generator=g, device=gpu["dev"]).bfloat16(), torch.randn((k, n), generator=g, device=gpu["dev"]).bfloat16())
    ops += (torch.empty_like(ops[0]), torch.empty((m, n), dtype=torch.bfloat16, device=gpu["dev"]))
    plans = [ficco.ficco_plan(m, k, n, 8, c, ficco.FICCO_FINE_PERSISTENT) for _ in range(2)]
    try:
        own, want = _run(gpu, plans[0], PAIR, ops)
        assert -(-n // own[1]) < lists, "the shape's own tile fits the lists: take another one"
        for plan in plans:
            ficco.ficco_plan_set(plan, ficco.FICCO_OPT_TILE_COLUMN_LISTS, lists)
            tile, out = _run(gpu, plan, PAIR, ops)
            assert -(-n // tile[1]) >= lists
            assert torch.equal(out, want)
        ficco.ficco_plan_set(plans[0], ficco.FICCO_OPT_TILE_COLUMN_LISTS, 0)
        assert _run(gpu, plans[0], PAIR, ops)[0] == own
        if n == 256:
            ficco.ficco_plan_set(plans[0], ficco.FICCO_OPT_TILE_COLUMN_LISTS, 4)
            with pytest.raises(ficco.FiccoError):
                _run(gpu, plans[0], PAIR, ops)
    finally:
        for plan in plans:
            ficco.ficco_destroy(plan)


def test_streamed_output_when_the_tile_changes_between_runs(gpu):
    """GEMM -> reduce-scatter: the kernel counts a piece's tiles to release its transfer, and the count starts again where a
    run has another tile than the one before it. A block that left early would bring the poison its rows were filled with."""
    m, k, n, shards = 8192, 8192, 1160, 2
    g = torch.Generator(device=gpu["dev"]).manual_seed(11)
    A = torch.randn((m, k), generator=g, device=gpu["dev"]).bfloat16()
    W = torch.randn((k, n), generator=g, device=gpu["dev"]).bfloat16()
    out = torch.empty((m, n), dtype=torch.bfloat16, device=gpu["dev"])
    peers = [torch.empty((m // shards, n), dtype=torch.bfloat16, device=gpu["dev"]) for _ in range(shards)]
    tiles = []
    plan = ficco.ficco_plan(m, k, n, shards, 1, ficco.FICCO_FINE_PERSISTENT)
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_DIRECTION, ficco.FICCO_DIR_GEMM_RS)
        for lists in (8, 0, 0, 8, 0):
            ficco.ficco_plan_set(plan, ficco.FICCO_OPT_TILE_COLUMN_LISTS, lists)
            for t in peers + [out]:
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            print(f"{lists} column lists", flush=True)
            ficco.ficco_run(plan, None, A, W, out, peers, gpu["cs"], gpu["xs"])
            ficco.ficco_query_stats(plan)
            torch.cuda.synchronize()
            info = ficco.ficco_plan_info(plan)
            tiles.append((info.tile_m, info.tile_n))
            assert not torch.isnan(out.float()).any()
            assert torch.equal(torch.cat(peers).view(torch.int16), out.view(torch.int16)), tiles
    finally:
        ficco.ficco_destroy(plan)
    assert tiles[0] != tiles[1], "the shape no longer tells the two apart: take another one"
