"""The result in the place of the activation, bit for bit what a result of its own gets. A workgroup stores its tile while
others read, so this holds only where one workgroup reads a row of A whole: a tile as wide as the output. Square weights of
one narrow column block (64) to four (256) and of one and two blocks of the 128 columns that the smaller tiles have, from
less than a row block to more rows than a launch multiplies in one round, and one small product whose rows move."""
import pytest

import paper_2512_10236_amd as ficco

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _operands(dev, M, K, N):
    g = torch.Generator(device=dev).manual_seed(M * 7 + K)
    A = torch.randn((M, K), generator=g, device=dev).bfloat16()
    W = (torch.randn((K, N), generator=g, device=dev) * K ** -0.5).bfloat16()
    return A, W


@pytest.mark.parametrize("M", [1, 33, 1000, 10000, 16384, 32768, 65536])
@pytest.mark.parametrize("K", [64, 128, 192, 256])
def test_static_in_place(gpu, M, K):
    A, W = _operands(gpu["dev"], M, K, K)
    want = torch.empty_like(A)
    print(f"in place {M}x{K}", flush=True)
    torch.cuda.synchronize()
    ficco.ficco_gemm_static(M, K, K, A, W, want, gpu["cs"])
    ficco.ficco_gemm_static(M, K, K, A, W, A, gpu["cs"])
    torch.cuda.synchronize()
    assert torch.equal(A.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("M,K,N,lead", [(32, 512, 256, 64), (17, 2048, 200, 0), (32, 4096, 136, 8 * 4096)])
def test_static_result_over_a_part_of_the_activation(gpu, M, K, N, lead):
    A, W = _operands(gpu["dev"], M, K, N)
    want = torch.empty((M, N), dtype=torch.bfloat16, device=gpu["dev"])
    C = A.view(-1)[lead:lead + M * N].view(M, N)
    print(f"over a part {M}x{K}x{N}", flush=True)
    torch.cuda.synchronize()
    ficco.ficco_gemm_static(M, K, N, A, W, want, gpu["cs"])
    ficco.ficco_gemm_static(M, K, N, A, W, C, gpu["cs"])
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("schedule,G,c,mode", [
    (ficco.FICCO_FINE_PERSISTENT, 1, 1, ficco.FICCO_MODE_GEMM_ONLY), (ficco.FICCO_SERIAL, 1, 1, ficco.FICCO_MODE_GEMM_ONLY),
    (ficco.FICCO_FINE_PERSISTENT, 8, 2, ficco.FICCO_MODE_PAIR), (ficco.FICCO_FINE_FUSED, 8, 2, ficco.FICCO_MODE_PAIR)])
@pytest.mark.parametrize("M,K", [(16 * 100, 256), (65536, 192), (65536, 256)])
def test_run_in_place(gpu, schedule, G, c, mode, M, K):
    """One plan, first with a result of its own, then in place, then with its own again."""
    A, W = _operands(gpu["dev"], M, K, K)
    own = [torch.empty_like(A) for _ in range(2)]
    landing = A.clone()
    plan = ficco.ficco_plan(M, K, K, G, c, schedule)
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, mode)
        print(f"plan in place {M}x{K} schedule {schedule} {G}x{c}", flush=True)
        for C in (own[0], landing, own[1]):
            if mode == ficco.FICCO_MODE_GEMM_ONLY and C is not landing:
                landing.copy_(A)
            torch.cuda.synchronize()
            ficco.ficco_run(plan, None if mode == ficco.FICCO_MODE_GEMM_ONLY else A, landing, W, C, None, gpu["cs"], gpu["xs"])
            ficco.ficco_query_stats(plan)
            if C is landing:
                placed = landing.clone()
    finally:
        ficco.ficco_destroy(plan)
    for got in (placed, own[1]):
        assert torch.equal(got.view(torch.int16), own[0].view(torch.int16))


def test_experts_in_place(gpu):
    G, E, K, rows = 4, 2, 192, 8192
    g = torch.Generator(device=gpu["dev"]).manual_seed(3)
    A = torch.randn((G * E * rows, K), generator=g, device=gpu["dev"]).bfloat16()
    W = (torch.randn((E * K, K), generator=g, device=gpu["dev"]) * K ** -0.5).bfloat16()
    landing, own = torch.empty_like(A), torch.empty_like(A)
    plan = ficco.ficco_plan_grouped(K, K, [[rows] * E] * G, 1, ficco.FICCO_FINE_PERSISTENT)
    try:
        print("experts in place", flush=True)
        torch.cuda.synchronize()
        for C in (own, landing):
            ficco.ficco_run(plan, A, landing, W, C, None, gpu["cs"], gpu["xs"])
            ficco.ficco_query_stats(plan)
    finally:
        ficco.ficco_destroy(plan)
    assert torch.equal(landing.view(torch.int16), own.view(torch.int16))
