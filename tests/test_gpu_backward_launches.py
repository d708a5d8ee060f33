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


# the library's names for its kernels (qii_gemm_route)
MAIN, T64, T128, T128_WIDE = 0, 2, 3, 4


@pytest.mark.parametrize("T,d_in,d_out,routes", [
    (2048, 2048, 2048, (T128_WIDE, T128_WIDE)),    # both products in one launch, 128 x 128 tiles in four K groups
    (1792, 2064, 1792, (T128_WIDE, T128_WIDE)),    # ragged d_in: tiled scales (post hoc form) of a last, partial row tile
    (1280, 4112, 1280, (T128, T128)),              # 128 x 128 tiles in two K groups, five K tiles
    (384, 16400, 384, (T128, T128)),               # K no multiple of 256; W and X re-quantized by blocks of two chunks, three chunks each
    (2048, 2048, 5632, (T128_WIDE, MAIN)),         # dX and dW by different kernels, so in two launches
    (3840, 1280, 1024, (T128, T64)),               # different kernels alone, one launch of 64 x 64 tiles together
])
@pytest.mark.parametrize("mode", [qii.MS_EDEN, qii.MS_EDEN_PH])
def test_backward_products_of_the_larger_tiles(oracle, T, d_in, d_out, routes, mode):
    for (M, K), route in zip(((T, d_out), (d_out, T)), routes):   # (both schemes hand over tiled scale bytes)
        assert qii.lib().qii_gemm_route(M, d_in, K, qii.qii_gemm_workspace_bytes(M, d_in, K), int(K % 256 == 0)) == route
    Xb, Wb, Eb = synth.linear_layer_bf16(T, d_in, d_out, seed=7)
    oXq, oWq = oracle.linear_fwd(Xb, Wb)
    Eq, WTq, ETq, XTq = oracle.linear_bwd_operands(Eb, oXq, oWq, 10, mode)
    E, Xq, Wq = to_dev(Eb), nv_to_dev(oXq), nv_to_dev(oWq)
    rng = np.random.default_rng(T + d_in)
    for dtype in (torch.float32, torch.bfloat16):
        print(f"backward T={T} {d_in}->{d_out} mode {mode} {dtype}", flush=True)
        dX = torch.full((T, d_in), float("nan"), dtype=dtype, device="cuda")
        dW = torch.full((d_out, d_in), float("nan"), dtype=dtype, device="cuda")
        w = ws(qii.qii_linear_bwd_mode_workspace_bytes(T, d_in, d_out, mode))
        w.fill_(0x7F)
        qii.qii_linear_bwd_mode(E, Xq, Wq, 10, mode, dX, dW, w)
        torch.cuda.synchronize()
        for got, (a, b) in ((dX, (Eq, WTq)), (dW, (ETq, XTq))):
            assert torch.isfinite(got).all()
            # random entries, and as many in the last columns (a partial tile where d_in is ragged), and the corners
            ms = np.concatenate([rng.integers(0, a.rows, 6000), [0, 0, a.rows - 1, a.rows - 1]])
            ns = np.concatenate([rng.integers(0, b.rows, 3000), rng.integers(b.rows - 100, b.rows, 3000), [0, b.rows - 1, 0, b.rows - 1]])
            ref, absum = oracle.gemm_sampled(a, b, ms, ns)
            tol = 1e-5 * absum + (2.0 ** -8 * np.abs(ref) if dtype == torch.bfloat16 else 0.0) + 1e-30
            assert np.all(np.abs(bf16_to_f64(got)[ms, ns] - ref) <= tol)


@pytest.mark.parametrize("T,d_in,d_out", [(512, 2176, 3584), (512, 2064, 3584)])
@pytest.mark.parametrize("mode", [qii.MS_EDEN, qii.MS_EDEN_PH])
def test_backward_products_of_two_k_tiles(oracle, T, d_in, d_out, mode):
    """Both products in one launch, one with K = 512: two K tiles.  (64 x 64 tiles: no product of fewer than three K tiles takes 128 x 128 tiles in
    four K groups, whose loads run four ahead.)"""
    size = max(qii.qii_gemm_workspace_bytes(T, d_in, d_out), qii.qii_gemm_workspace_bytes(d_out, d_in, T))
    assert qii.lib().qii_linear_bwd_gemm_route(T, d_in, d_out, size, 1) == T64
    Xb, Wb, Eb = synth.linear_layer_bf16(T, d_in, d_out, seed=8)
    oXq, oWq = oracle.linear_fwd(Xb, Wb)
    Eq, WTq, ETq, XTq = oracle.linear_bwd_operands(Eb, oXq, oWq, 11, mode)
    E, Xq, Wq = to_dev(Eb), nv_to_dev(oXq), nv_to_dev(oWq)
    rng = np.random.default_rng(T + d_in)
    for dtype in (torch.float32, torch.bfloat16):
        print(f"backward T={T} {d_in}->{d_out} mode {mode} {dtype}", flush=True)
        dX, dW = (torch.full((r, d_in), float("nan"), dtype=dtype, device="cuda") for r in (T, d_out))
        w = ws(qii.qii_linear_bwd_mode_workspace_bytes(T, d_in, d_out, mode))
        w.fill_(0x7F)
        qii.qii_linear_bwd_mode(E, Xq, Wq, 11, mode, dX, dW, w)
        torch.cuda.synchronize()
        for got, (a, b) in ((dX, (Eq, WTq)), (dW, (ETq, XTq))):
            assert torch.isfinite(got).all()
            ms = np.concatenate([rng.integers(0, a.rows, 6000), [0, 0, a.rows - 1, a.rows - 1]])
            ns = np.concatenate([rng.integers(0, b.rows, 3000), rng.integers(b.rows - 100, b.rows, 3000), [0, b.rows - 1, 0, b.rows - 1]])
            ref, absum = oracle.gemm_sampled(a, b, ms, ns)
            tol = 1e-5 * absum + (2.0 ** -8 * np.abs(ref) if dtype == torch.bfloat16 else 0.0) + 1e-30
            assert np.all(np.abs(bf16_to_f64(got)[ms, ns] - ref) <= tol)


@pytest.mark.parametrize("T,d_in,d_out", [(128, 128, 128), (512, 512, 512), (384, 208, 256), (1024, 2048, 2048), (4096, 2048, 4096)])
@pytest.mark.parametrize("mode", [qii.MS_EDEN, qii.MS_EDEN_PH])
@pytest.mark.parametrize("place", ["apart", "misaligned", "dX in dY", "dW in dY", "dX beside dW"])
def test_where_the_results_lie_makes_no_difference(T, d_in, d_out, mode, place):
    """The four quantizations of a pass run in one launch, whose buffers of W and X (post hoc scheme) the results' memory takes; results
    that are misaligned for it, or share bytes with the gradient that the launch reads, get the launches one after the other.  The
    same bits.  Algorithm 1 has no such buffers and looks at no place: its reference is the same gradient in f32, whose quantizations
    always take launches of their own and leave row-major scale bytes (the kernels of the products are the same either way)."""
    n_e, n_x, n_w = T * d_out, T * d_in, d_out * d_in
    if (place == "dX in dY" and n_x > n_e) or (place == "dW in dY" and n_w > n_e):
        pytest.skip("the result is larger than the gradient")
    Xb, Wb, Eb = synth.linear_layer_bf16(T, d_in, d_out, seed=8)
    Xq, Wq = qii.NVFP4Tensor.empty(T, d_in), qii.NVFP4Tensor.empty(d_out, d_in)
    for x, q in ((Xb, Xq), (Wb, Wq)):
        qii.qii_quantize_nvfp4(to_dev(x), False, qii.RTN, 0, 0, 0, None, q, ws(256))

    def run(E, dX, dW):
        E.copy_(to_dev(Eb))
        w = ws(qii.qii_linear_bwd_mode_workspace_bytes(T, d_in, d_out, mode))
        w.fill_(0x7F)
        qii.qii_linear_bwd_mode(E, Xq, Wq, 11, mode, dX, dW, w)
        torch.cuda.synchronize()
        return dX.clone(), dW.clone()

    def buf(n, shape, off=0):
        return torch.full((n + 16,), float("nan"), dtype=torch.bfloat16, device="cuda")[off:off + n].view(shape)

    print(f"backward T={T} {d_in}->{d_out} mode {mode} {place}", flush=True)
    if mode == qii.MS_EDEN:
        for M, K in ((T, d_out), (d_out, T)):
            size = qii.qii_gemm_workspace_bytes(M, d_in, K)
            assert qii.lib().qii_gemm_route(M, d_in, K, size, int(K % 256 == 0)) == qii.lib().qii_gemm_route(M, d_in, K, size, 0)
        eX, eW = run(torch.empty((T, d_out), device="cuda"), buf(n_x, (T, d_in), 1), buf(n_w, (d_out, d_in), 1))
    else:
        eX, eW = run(buf(n_e, (T, d_out)), buf(n_x, (T, d_in), 1), buf(n_w, (d_out, d_in), 1))
    E, dX, dW = buf(n_e, (T, d_out)), buf(n_x, (T, d_in)), buf(n_w, (d_out, d_in))
    if place == "misaligned":
        dW = buf(n_w, (d_out, d_in), 3)
    elif place == "dX in dY":
        dX = E.view(-1)[:n_x].view(T, d_in)
    elif place == "dW in dY":
        dW = E.view(-1)[n_e - n_w:].view(d_out, d_in)
    elif place == "dX beside dW":
        both = buf(n_x + n_w, (n_x + n_w,))
        dX, dW = both[:n_x].view(T, d_in), both[n_x:].view(d_out, d_in)
    gX, gW = run(E, dX, dW)
    assert torch.isfinite(gX).all() and torch.isfinite(gW).all()
    assert torch.equal(gX, eX) and torch.equal(gW, eW)
