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
