"""max |C| as a by-product of the GEMM costs little beside the product, also where the product is cut into thousands of small
tiles: atomics on the one result word are resolved one after the other, so one per wave of a 128 x 128 or 64 x 64 tile
would take longer than the product.  The value is the largest stored |C| (also checked with ragged tiles)."""
import pytest
import torch

from paper_2601_22813_amd import binding as qii

from gpu_util import median_us, ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(20000, 3000, 112), (25683, 304, 864), (11790, 2272, 304)])
def test_max_of_the_result_costs_little(M, N, K):
    g = torch.Generator(device="cuda").manual_seed(5)
    A, B = qii.NVFP4Tensor.empty(M, K), qii.NVFP4Tensor.empty(N, K)
    for t in (A, B):
        qii.qii_quantize_nvfp4(torch.randn((t.rows, K), device="cuda", generator=g), False, qii.RTN, 0, 0, 0, None, t, ws(256))
    C = torch.empty((M, N), device="cuda")
    amax = torch.full((1,), float("nan"), device="cuda")
    plain = median_us(lambda: qii.qii_gemm_nvfp4(A, B, C, None))
    emits = median_us(lambda: qii.qii_gemm_nvfp4_amax(A, B, C, amax, None))
    print(f"gemm {M}x{N}x{K}: {plain:.1f} us, with the maximum {emits:.1f}", flush=True)
    assert amax.item() == C.abs().max().item()
    # the clearing launch is 2 to 5 us of it; one atomic per wave made these products 1.5 to 3 times as long
    assert emits <= 1.25 * plain + 5.0
