"""Forward pass: X and W are measured by one launch (a word per block) and quantized by one launch.  Saved operands byte
for byte against the oracle where that can go wrong: the smallest tensors, rows longer than one row of blocks covers
(d_in > 4096), very unequal sizes of X and W in both directions (the blocks are shared out by size), f32 and bf16,
none, one or both maxima supplied, and an all-zero W next to a non-zero X."""
import numpy as np
import pytest
import torch

from paper_2601_22813_amd import binding as qii
from paper_2601_22813_amd import synth

from gpu_util import assert_nv_equal, median_us, to_dev, ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d_in,d_out", [(1, 16, 1), (5, 4112, 3), (3, 8448, 700), (9000, 48, 2), (2, 256, 9000), (1027, 1040, 333)] +
                         # tensors that every block measures for itself, and a row or a column group beyond that
                         [(256, 256, 256), (257, 256, 255), (512, 64, 512), (513, 64, 300), (31, 2064, 7), (64, 1040, 5)])
@pytest.mark.parametrize("f32", [False, True])
def test_forward_operands_from_two_launches(oracle, T, d_in, d_out, f32):
    Xb, Wb, _ = synth.linear_layer_bf16(T, d_in, d_out, seed=4)
    if f32:
        Xb, Wb = synth.bf16_bits_to_f32(Xb) * np.float32(1.0001), synth.bf16_bits_to_f32(Wb) * np.float32(0.9999)
    for mode in (qii.RTN, qii.RTN_46):
        for zero_w in (False, True):
            W_ = np.zeros_like(Wb) if zero_w else Wb
            oXq, oWq = oracle.linear_fwd(Xb, W_, mode)
            X, W = to_dev(Xb), to_dev(W_)
            ax, aw = X.abs().max().float().reshape(1), W.abs().max().float().reshape(1)
            for px, pw in ((None, None), (ax, None), (None, aw), (ax, aw)):
                print(f"forward {T}x{d_in}->{d_out} f32 {f32} mode {mode} zero_w {zero_w} maxima {px is not None} {pw is not None}", flush=True)
                Xq, Wq = qii.NVFP4Tensor.empty(T, d_in), qii.NVFP4Tensor.empty(d_out, d_in)
                for t in (Xq, Wq):
                    t.codes.fill_(0xAB); t.scales.fill_(0xCD)
                Y = torch.empty((T, d_out), dtype=torch.float32, device="cuda")
                w = ws(qii.qii_linear_fwd_workspace_bytes(T, d_in, d_out))
                w.fill_(0x7F)   # as floats 3e38: a word that no block wrote must not count
                qii.qii_linear_fwd_mode(X, W, mode, Y, Xq, Wq, w, amax_x=px, amax_w=pw)
                assert_nv_equal(Xq, oXq, "X")
                assert_nv_equal(Wq, oWq, "W")


@pytest.mark.parametrize("T,d_in,mode,f32", [(16384, 3072, qii.RTN_46, True), (16384, 4096, qii.RTN_46, False)])
def test_quantizing_in_the_forward_pass_costs_no_more_than_alone(T, d_in, mode, f32):
    """A layer of one group of outputs is its quantizer: the pass beside the quantizer's own call and the product.  A block that
    waits for its rows before it reduces the maximum's words makes the quantize launch a quarter to a third longer: the pass
    then took 1.13 and 1.17 times as long as the two calls, 0.99 times without that wait."""
    g = torch.Generator(device="cuda").manual_seed(6)
    X = torch.randn((T, d_in), device="cuda", generator=g)
    W = torch.randn((16, d_in), device="cuda", generator=g)
    if not f32:
        X, W = X.bfloat16(), W.bfloat16()
    Xq, Wq, Y = qii.NVFP4Tensor.empty(T, d_in), qii.NVFP4Tensor.empty(16, d_in), torch.empty((T, 16), device="cuda")
    w = ws(max(qii.qii_linear_fwd_workspace_bytes(T, d_in, 16), qii.qii_gemm_workspace_bytes(T, 16, d_in)))
    whole = median_us(lambda: qii.qii_linear_fwd_mode(X, W, mode, Y, Xq, Wq, w))
    alone = median_us(lambda: qii.qii_quantize_nvfp4(X, False, mode, 0, 0, 0, None, Xq, w))
    product = median_us(lambda: qii.qii_gemm_nvfp4(Xq, Wq, Y, w))
    print(f"{T}x{d_in} mode {mode} f32 {f32}: forward {whole:.1f} us, quantizer {alone:.1f}, product {product:.1f}", flush=True)
    assert whole <= 1.08 * (alone + product)
