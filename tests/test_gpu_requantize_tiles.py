"""Re-quantization of a saved NVFP4 tensor with transposition, at the edges of its tiles (128 stored columns, one or two
128-row chunks per block), byte for byte against the oracle: column counts that end inside a 16-byte piece of codes
(16, 208, 144 columns) or inside a tile, odd and even numbers of chunks, the smallest tensor, and one with enough tiles
for two chunks per block whose last block is half empty; with and without rotation."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2601_22813_amd import binding as qii

from gpu_util import assert_nv_equal, nv_to_dev, ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(128, 16), (256, 208), (384, 144), (640, 1040), (1152, 128), (8320, 2064)])
@pytest.mark.parametrize("rht_group", [128, 0])
def test_tiles_of_a_transposed_requantization(oracle, rows, cols, rht_group):
    rng = np.random.default_rng(rows + cols)
    # every code, every scale byte the library writes, a tensor scale that is no power of two
    saved = oracle.NVFP4(rng.integers(0, 256, (rows, cols // 2)).astype(np.uint8), rng.integers(0, 127, (rows, cols // 16)).astype(np.uint8),
                         np.array([0.0123], np.float32))
    dev = nv_to_dev(saved)
    for mode in (qii.RTN, qii.SR, qii.MS_EDEN, qii.RTN_46, qii.MS_EDEN_PH) if rows < 8000 else (qii.MS_EDEN, qii.MS_EDEN_PH):
        print(f"requantize {rows}x{cols} rotation {rht_group} mode {mode}", flush=True)
        out = qii.NVFP4Tensor.empty(cols, rows)
        out.codes.fill_(0xAB)
        out.scales.fill_(0xCD)
        qii.qii_requantize_nvfp4(dev, True, mode, rht_group, 71, 72, None, out, ws(qii.qii_quantize_posthoc_workspace_bytes(cols, rows)))
        ref = oracle.requantize(saved, mode, transpose=True, rht_group=rht_group, seed_rht=71, seed_sr=72)
        assert_nv_equal(out, ref, f"{rows}x{cols} rotation {rht_group} mode {mode}")


@pytest.mark.parametrize("rows,cols,zero", [(128, 16, False), (128, 384, False), (128, 8192, False), (128, 8320, False), (384, 384, True)])
def test_a_requantization_of_few_blocks_is_two_launches(oracle, rows, cols, zero):
    """At 64 blocks or fewer (128 x 8192 has 64) the abs-max pass leaves a word per block in the 256-byte workspace: nothing is
    cleared first, stale words must not count, and the call is two launches (three beyond)."""
    rng = np.random.default_rng(cols)
    codes = np.zeros((rows, cols // 2), np.uint8) if zero else rng.integers(0, 256, (rows, cols // 2)).astype(np.uint8)
    saved = oracle.NVFP4(codes, rng.integers(0, 127, (rows, cols // 16)).astype(np.uint8), np.array([0.0123], np.float32))
    dev, out, w = nv_to_dev(saved), qii.NVFP4Tensor.empty(cols, rows), torch.empty(256, dtype=torch.uint8, device="cuda")
    w.fill_(0x7F)   # as floats 3e38

    def call():
        qii.qii_requantize_nvfp4(dev, True, qii.MS_EDEN, 128, 71, 72, None, out, w)

    call()
    assert_nv_equal(out, oracle.requantize(saved, qii.MS_EDEN, transpose=True, rht_group=128, seed_rht=71, seed_sr=72), f"{rows}x{cols}")
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    nodes = ctypes.c_size_t()
    get = ctypes.CDLL("libamdhip64.so").hipGraphGetNodes
    get.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    assert get(graph.raw_cuda_graph(), None, ctypes.byref(nodes)) == 0
    assert nodes.value == (2 if cols <= 8192 else 3)
