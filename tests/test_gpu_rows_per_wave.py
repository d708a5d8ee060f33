"""Quantizers along rows on both sides of their size rules: one row per wave or a quad of rows, tensors that every block measures
for itself or an abs-max launch, 1, 2 or 4 waves of a block side by side.  Every byte against the oracle, at row counts that are
no multiple of 4, last chunks that are partial ones, and rows that lie apart."""
import numpy as np
import pytest
import torch

from paper_2601_22813_amd import binding as qii
from paper_2601_22813_amd import synth

from gpu_util import assert_nv_equal, nv_bytes, to_dev, ws

pytestmark = pytest.mark.gpu

PLAIN, ROTATED = [qii.RTN, qii.SR, qii.RTN_46], [qii.SR, qii.MS_EDEN, qii.MS_EDEN_PH]


def quantize(x, mode, rht, amax=None):
    R, C = x.shape
    out = qii.NVFP4Tensor.empty(R, C)
    out.codes.fill_(0xAB); out.scales.fill_(0xCD)
    w = ws(qii.qii_quantize_posthoc_workspace_bytes(R, C) if mode == qii.MS_EDEN_PH else 256)
    w.fill_(0x7F)   # as floats 3e38: a word that no block wrote must not count
    qii.qii_quantize_nvfp4(x, False, mode, rht, 21, 22, amax, out, w)
    return out


@pytest.mark.parametrize("R,C,rht", [
    (1, 16, 0), (6, 1040, 0), (511, 80, 0), (512, 128, 0), (513, 128, 0), (63, 1024, 0), (255, 272, 0),     # the first six: measured by each block
    (1021, 1024, 0), (4097, 1024, 0), (1023, 2064, 0), (4099, 1040, 0), (301, 4112, 0), (205, 5648, 0), (1025, 4096, 0),
    (1, 128, 128), (1021, 1024, 128), (4097, 1024, 128), (515, 1152, 128), (205, 5120, 128), (1026, 5632, 128), (131, 7168, 128),
    (3356, 1024, 128), (3357, 1024, 128), (836, 2304, 128), (837, 2304, 128),      # the line of the post hoc scheme
])
@pytest.mark.parametrize("f32", [False, True])
def test_rows_on_both_sides_of_the_rules(oracle, R, C, rht, f32):
    x = synth.student_t_bf16((R, C), 3, 0.1, seed=R + C)
    if f32:
        x = synth.bf16_bits_to_f32(x) * np.float32(1.0001)
    for mode in (ROTATED if rht else PLAIN):
        print(f"quantize {R}x{C} mode {mode} f32 {f32}", flush=True)
        assert_nv_equal(quantize(to_dev(x), mode, rht), oracle.quantize(x, mode, rht_group=rht, seed_rht=21, seed_sr=22), f"{R}x{C} mode {mode}")


@pytest.mark.parametrize("mode", PLAIN)
def test_rows_that_lie_apart(oracle, mode):
    x = synth.student_t_bf16((40, 80), 3, 0.1, seed=1)
    assert_nv_equal(quantize(to_dev(x)[:, :64], mode, 0), oracle.quantize(np.ascontiguousarray(x[:, :64]), mode, rht_group=0, seed_rht=21, seed_sr=22))


@pytest.mark.parametrize("mode", PLAIN)
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("odd", [float("nan"), float("inf"), float("-inf"), 0.0])
def test_a_measured_maximum_is_that_of_the_abs_max_pass(mode, dt, odd):
    """Infinities, NaN and nothing but zeros, in a tensor that every block measures: the bytes that the abs-max pass's word gives."""
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((60, 208), device="cuda", generator=g).to(dt)
    if odd == 0.0:
        x.zero_()
    else:
        x[7, 33] = odd
        x[59, 207] = odd
    amax = torch.empty(1, device="cuda")
    qii.qii_absmax(x, False, 0, 0, amax)
    for got, want in zip(nv_bytes(quantize(x, mode, 0)), nv_bytes(quantize(x, mode, 0, amax))):
        assert np.array_equal(got.view(np.uint8), want.view(np.uint8))
