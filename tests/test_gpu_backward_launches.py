"""Backward pass: W and X are re-quantized by shared launches where the workspace allows, one after the other where it
does not, and block maxima go to a word per block or to the spread words.  dX and dW against the oracle (tolerance as in
test_gpu_gemm_linear.py) at shapes on both sides of those lines: d_in small and large against T and d_out, ragged d_in,
f32 gradients (whose two quantizations take separate kernels), and a workspace full of stale bytes."""
import numpy as np
import pytest
import torch

from paper_2601_22813_amd import binding as qii
from paper_2601_22813_amd import synth

from gpu_util import bf16_to_f64, nv_to_dev, to_dev, ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d_in,d_out", [(128, 16, 128), (128, 2048, 128), (256, 208, 384), (640, 1040, 256), (1024, 128, 1280)])
@pytest.mark.parametrize("mode", [qii.MS_EDEN, qii.MS_EDEN_PH])
@pytest.mark.parametrize("f32", [False, True])
def test_backward_at_both_sides_of_the_launch_rules(oracle, T, d_in, d_out, mode, f32):
    Xb, Wb, Eb = synth.linear_layer_bf16(T, d_in, d_out, seed=6)
    if f32:
        Eb = synth.bf16_bits_to_f32(Eb) * np.float32(1.0001)
    oXq, oWq = oracle.linear_fwd(Xb, Wb)
    Eq, WTq, ETq, XTq = oracle.linear_bwd_operands(Eb, oXq, oWq, 9, mode)
    E, Xq, Wq = to_dev(Eb), nv_to_dev(oXq), nv_to_dev(oWq)
    for dtype in (torch.float32, torch.bfloat16):
        print(f"backward T={T} {d_in}->{d_out} mode {mode} f32 {f32} {dtype}", flush=True)
        dX = torch.full((T, d_in), float("nan"), dtype=dtype, device="cuda")
        dW = torch.full((d_out, d_in), float("nan"), dtype=dtype, device="cuda")
        w = ws(qii.qii_linear_bwd_mode_workspace_bytes(T, d_in, d_out, mode))
        w.fill_(0x7F)   # as floats 3e38: a maximum that no block wrote must not count
        qii.qii_linear_bwd_mode(E, Xq, Wq, 9, mode, dX, dW, w)
        torch.cuda.synchronize()
        for got, (a, b) in ((dX, (Eq, WTq)), (dW, (ETq, XTq))):
            ref, absum = oracle.gemm(a, b, with_abs=True)
            tol = 1e-5 * absum + (2.0 ** -8 * np.abs(ref) if dtype == torch.bfloat16 else 0.0) + 1e-30
            assert np.all(np.abs(bf16_to_f64(got) - ref) <= tol)
