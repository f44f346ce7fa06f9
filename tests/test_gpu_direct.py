"""The GEMM straight from a row-major weight (small products of ficco_gemm_static) and the weight packing kernels, bit for
bit against the plan path: the same MFMAs in the same k order. Sizes: one row and one column block, remainders of rows,
columns and of the 128-value stage, shapes on both sides of where the rule changes the row blocks, each with the route that
it is there for, and what the direct kernel does not take. And the kernel by itself with 1, 2 and 4 row blocks, over fewer
stages of 128 values than its ring holds (7, 6 and 4), as many, and more than two times round."""
import os
import sys

import pytest

import paper_2512_10236_amd as ficco
from paper_2512_10236_amd import _build

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import internal

torch = pytest.importorskip("torch")


def _operands(dev, M, K, N, lead=0):
    g = torch.Generator(device=dev).manual_seed(M * 7 + K * 3 + N)
    A = torch.randn((M, K), generator=g, device=dev).bfloat16()
    W = torch.empty(lead + K * N, dtype=torch.bfloat16, device=dev)[lead:].view(K, N)
    W.copy_(torch.randn((K, N), generator=g, device=dev) * K ** -0.5)
    return A, W


def _by_plan(gpu, A, W, M, K, N):
    C = torch.full((M, N), 7.0, dtype=torch.bfloat16, device=gpu["dev"])
    plan = ficco.ficco_plan(M, K, N, 1, 1, ficco.FICCO_FINE_PERSISTENT)
    try:
        ficco.ficco_plan_set(plan, ficco.FICCO_OPT_MODE, ficco.FICCO_MODE_GEMM_ONLY)
        torch.cuda.synchronize()
        ficco.ficco_run(plan, None, A, W, C, None, gpu["cs"], gpu["xs"])
        ficco.ficco_query_stats(plan)
    finally:
        ficco.ficco_destroy(plan)
    return C.view(torch.int16)


SHAPES = [(1, 64, 8), (16, 128, 64), (17, 192, 72), (5, 768, 136), (48, 896, 1160), (64, 1024, 56), (20, 896, 96), (16, 1024, 40), (64, 4096, 768), (130, 2880, 1448),
          (256, 512, 1024), (257, 512, 1024), (512, 576, 1000), (513, 576, 1032), (1024, 512, 1024), (1025, 640, 1032), (4096, 128, 64),
          (400, 1088, 1024), (512, 4096, 1024), (16384, 64, 128), (1024, 1088, 1024), (900, 2048, 1024), (2048, 4096, 1024), (4096, 1024, 1024)]
ROW_BLOCKS = [1] * 11 + [2, 2, 4, 4, 4, 1] + [2, 2, 4, 4, 4, 0, 0]


def test_shapes_take_the_route_they_are_there_for():
    assert [internal.direct_row_blocks(*s) for s in SHAPES] == ROW_BLOCKS


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_direct_gemm_has_the_plan_paths_bits(gpu, M, K, N):
    A, W = _operands(gpu["dev"], M, K, N)
    C = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=gpu["dev"])
    print(f"direct {M}x{K}x{N}", flush=True)
    torch.cuda.synchronize()
    ficco.ficco_gemm_static(M, K, N, A, W, C, gpu["cs"])
    torch.cuda.synchronize()
    assert torch.equal(C[:M].view(torch.int16), _by_plan(gpu, A, W, M, K, N))
    assert bool((C[M] == 7.0).all()), "wrote past the last row"
    ref = A.double().cpu() @ W.double().cpu()
    assert float((C[:M].double().cpu() - ref).norm() / ref.norm()) <= 2.0 ** -8      # one rounding to bf16


@pytest.mark.gpu
@pytest.mark.parametrize("row_blocks,ring", [(1, 7), (2, 6), (4, 4)])
def test_direct_kernel_over_its_ring(gpu, row_blocks, ring):
    M, N = 2 * 16 * row_blocks + 3, 136
    for K in range(64, 128 * (2 * ring + 2) + 1, 64):
        A, W = _operands(gpu["dev"], M, K, N)
        C = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=gpu["dev"])
        print(f"direct kernel, {row_blocks} row blocks, {M}x{K}x{N}", flush=True)
        torch.cuda.synchronize()
        internal.launch_direct(row_blocks, A, W, C, gpu["cs"])
        torch.cuda.synchronize()
        assert torch.equal(C[:M].view(torch.int16), _by_plan(gpu, A, W, M, K, N)), (row_blocks, K)
        assert bool((C[M] == 7.0).all()), (row_blocks, K)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(17, 192, 72), (64, 1024, 256)])
def test_weight_off_its_alignment_and_result_over_the_weight(gpu, M, K, N):
    """A weight at an odd element is packed two bytes at a time; a result that overlaps the weight is written after the
    weight has been packed."""
    A, W = _operands(gpu["dev"], M, K, N)
    want = _by_plan(gpu, A, W, M, K, N)
    odd = _operands(gpu["dev"], M, K, N, lead=1)[1]
    assert odd.data_ptr() % 16
    C = torch.full((M, N), 7.0, dtype=torch.bfloat16, device=gpu["dev"])
    print(f"odd weight {M}x{K}x{N}", flush=True)
    torch.cuda.synchronize()
    ficco.ficco_gemm_static(M, K, N, A, odd, C, gpu["cs"])
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int16), want)
    over = W.clone()
    C = over.view(-1)[K * N - M * N:].view(M, N)
    torch.cuda.synchronize()
    ficco.ficco_gemm_static(M, K, N, A, over, C, gpu["cs"])
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int16), want)


def test_wait_states_of_the_direct_loads(tmp_path):
    """M0 and scalar bases in front of the direct-to-LDS loads, as for the other GEMM kernels (the MFMAs are builtins
    here, whose wait states the compiler sees to)."""
    import subprocess
    from test_asm_hazards import hazards
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = str(tmp_path / "direct.s")
    r = subprocess.run([hipcc] + _build.FLAGS + ["-S", "--cuda-device-only", os.path.join(_build.CSRC, "ficco_direct.hip"), "-o", out],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    bad, seen = hazards(open(out).read())
    assert seen > 0
    assert not [b for b in bad if not b[1].startswith("MFMA")]
