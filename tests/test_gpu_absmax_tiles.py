"""Rotated abs-max by 128 x 128 tiles (along the columns, and along both orientations for Algorithm 1's pair): bit for
bit the oracle's maximum where the tile kernels can go wrong: one tile, fewer tiles than a block has wave groups, a
tile count that leaves some groups without a tile in the last of two rounds (4480 x 5248; at 1280 x 6656 and 4224 x 4352
qii_absmax takes the columns kernel), a leading dimension beyond the row whose extra columns are huge, and a maximum that
sits in the last tile."""
import numpy as np
import pytest
import torch

from paper_2601_22813_amd import binding as qii
from paper_2601_22813_amd import synth

from gpu_util import assert_nv_equal, to_dev, ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(128, 128), (128, 384), (640, 384), (256, 1152), (1280, 6656), (4224, 4352), (4480, 5248)])
def test_rotated_abs_max_by_tiles(oracle, rows, cols):
    x = synth.student_t_bf16((rows, cols), 3, 0.1, seed=rows + cols)
    x[rows - 128:, cols - 128:] = synth.normal_bf16((128, 128), 5.0, 3)   # the largest values in the last tile
    full = to_dev(np.concatenate([x, np.full((rows, 128), 0x7000, np.uint16)], axis=1))[:, :cols]   # 1.6e29 beyond the row
    amax = torch.full((1,), float("nan"), device="cuda")
    qii.qii_absmax(full, True, 128, 91, amax)
    _, want = oracle.rht(x, transpose=True, rht_group=128, seed_rht=91)
    assert amax.item() == want
    if rows * cols > 1 << 20:
        return
    out_r, out_c = qii.NVFP4Tensor.empty(rows, cols), qii.NVFP4Tensor.empty(cols, rows)
    qii.qii_quantize_pair_nvfp4(full, qii.MS_EDEN, 91, 92, 93, 94, out_r, out_c, ws(qii.qii_quantize_pair_workspace_bytes(rows, cols, qii.MS_EDEN)))
    assert_nv_equal(out_r, oracle.quantize(x, qii.MS_EDEN, seed_rht=91, seed_sr=92), "rows")
    assert_nv_equal(out_c, oracle.quantize(x, qii.MS_EDEN, transpose=True, seed_rht=93, seed_sr=94), "columns")


@pytest.mark.parametrize("rows,cols,where", [(4096, 2048, "first"), (4096, 2048, "last"), (3456, 2432, "first"), (3456, 2432, "last"),   # (513: block 0's second)
                                              (3200, 5248, "first"), (3200, 5248, "block 0's second"), (3200, 5248, "last")])
def test_both_maxima_of_a_pair(rows, cols, where):
    """512 tiles (one a block), 513 (one block has a second one) and 1025 (two or three each, the two LDS images in turn):
    Algorithm 1's pair equals the two separate quantizations, whose maxima come from other kernels; one tile holds the maximum."""
    tiles_x = cols // 128
    tile = {"first": 0, "last": rows // 128 * tiles_x - 1}.get(where, 512)
    x = synth.normal_bf16((rows, cols), 1.0, rows + cols)
    r, c = tile // tiles_x * 128, tile % tiles_x * 128
    x[r:r + 128, c:c + 128] = synth.normal_bf16((128, 128), 50.0, 3)
    x = to_dev(x)
    out_r, out_c = qii.NVFP4Tensor.empty(rows, cols), qii.NVFP4Tensor.empty(cols, rows)
    qii.qii_quantize_pair_nvfp4(x, qii.MS_EDEN, 91, 92, 93, 94, out_r, out_c, ws(qii.qii_quantize_pair_workspace_bytes(rows, cols, qii.MS_EDEN)))
    for out, transpose, rht, sr in ((out_r, False, 91, 92), (out_c, True, 93, 94)):
        one = qii.NVFP4Tensor.empty(out.rows, out.cols)
        qii.qii_quantize_nvfp4(x, transpose, qii.MS_EDEN, 128, rht, sr, None, one, ws(qii.qii_quantize_workspace_bytes()))
        assert torch.equal(out.tensor_scale, one.tensor_scale)
        assert torch.equal(out.scales, one.scales) and torch.equal(out.codes, one.codes)
