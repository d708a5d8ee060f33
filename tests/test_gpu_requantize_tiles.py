"""Re-quantization of a saved NVFP4 tensor with transposition, at the edges of its tiles (128 stored columns, one or two
128-row chunks per block), byte for byte against the oracle: column counts that end inside a 16-byte piece of codes
(16, 208, 144 columns) or inside a tile, odd and even numbers of chunks, the smallest tensor, and one with enough tiles
for two chunks per block whose last block is half empty; with and without rotation."""
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
