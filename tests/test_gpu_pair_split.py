"""Both orientations of a matrix from one read (four waves of a block take the rows, four the columns): byte for byte the two
separate quantizations, from one tile to more than the chip holds at once, with a leading dimension beyond the row and an
all-zero tensor."""
import numpy as np
import pytest
import torch

from paper_2601_22813_amd import binding as qii
from paper_2601_22813_amd import synth

from gpu_util import assert_nv_equal, to_dev, ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [qii.MS_EDEN, qii.MS_EDEN_PH])
@pytest.mark.parametrize("rows,cols", [(128, 128), (384, 640), (2048, 2048), (2176, 2048), (4096, 4096), (4096, 4224)])
def test_pair_equals_separate_calls(rows, cols, mode):
    for x in (synth.student_t_bf16((rows, cols), 3, 0.1, seed=rows + cols), np.zeros((rows, cols), np.uint16)):
        full = to_dev(np.concatenate([x, np.full((rows, 8), 0x7000, np.uint16)], axis=1))[:, :cols]   # huge beyond the row
        pair = qii.NVFP4Tensor.empty(rows, cols), qii.NVFP4Tensor.empty(cols, rows)
        qii.qii_quantize_pair_nvfp4(full, mode, 11, 12, 13, 14, *pair, ws(qii.qii_quantize_pair_workspace_bytes(rows, cols, mode)))
        alone = qii.NVFP4Tensor.empty(rows, cols), qii.NVFP4Tensor.empty(cols, rows)
        size = ws(qii.qii_quantize_posthoc_workspace_bytes(rows, cols))
        qii.qii_quantize_nvfp4(full, False, mode, 128, 11, 12, None, alone[0], size)
        qii.qii_quantize_nvfp4(full, True, mode, 128, 13, 14, None, alone[1], size)
        for a, b in zip(pair, alone):
            assert torch.equal(a.codes, b.codes) and torch.equal(a.scales, b.scales)
            assert torch.equal(a.tensor_scale, b.tensor_scale)


@pytest.mark.parametrize("rows,cols", [(4096, 4096), (4096, 4224), (8192, 8064), (8192, 8192), (8192, 8320)])
def test_every_block_word_counts(rows, cols):
    """1024 blocks of the heavy pass (one load of the scales pass holds their words), 1056, 4032, 4096 (as many words as the region has) and
    4160 (the spread running maximum): an outlier in the first, a middle and the last tile sets the maximum, the
    same as a call that is given it, along the rows, the columns and both; the workspace holds no zeros before."""
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = (0.1 * torch.randn((rows, cols), device="cuda", generator=g)).bfloat16()
    for tile in ((0, 0), (rows // 256, cols // 256), (rows // 128 - 1, cols // 128 - 1)):
        y = x.clone()
        y[tile[0] * 128 + 77, tile[1] * 128 + 99] = 400.0
        pair = qii.NVFP4Tensor.empty(rows, cols), qii.NVFP4Tensor.empty(cols, rows)
        w = ws(qii.qii_quantize_pair_workspace_bytes(rows, cols, qii.MS_EDEN_PH))
        w.fill_(0x7E)
        qii.qii_quantize_pair_nvfp4(y, qii.MS_EDEN_PH, 11, 12, 13, 14, *pair, w)
        for transpose, seed, both in ((False, 11, pair[0]), (True, 13, pair[1])):
            top = torch.empty(1, device="cuda")
            qii.qii_absmax(y, transpose, 128, seed, top)
            alone, given = (qii.NVFP4Tensor.empty(both.rows, both.cols) for _ in range(2))
            size = ws(qii.qii_quantize_posthoc_workspace_bytes(both.rows, both.cols))
            size.fill_(0x7E)
            qii.qii_quantize_nvfp4(y, transpose, qii.MS_EDEN_PH, 128, seed, seed + 1, None, alone, size)
            qii.qii_quantize_nvfp4(y, transpose, qii.MS_EDEN_PH, 128, seed, seed + 1, top, given, size)
            for t in (alone, both):
                assert torch.equal(t.codes, given.codes) and torch.equal(t.scales, given.scales) and torch.equal(t.tensor_scale, given.tensor_scale)


@pytest.mark.parametrize("rows,cols,rht", [(1, 128, 128), (2, 64, 0), (3, 128, 128), (6, 192, 0), (5, 48, 0), (1001, 1024, 128), (4096, 8192, 128), (4100, 8192, 128)])
def test_scale_bytes_by_one_group_and_by_four(oracle, rows, cols, rht):
    """Post hoc scheme: a thread of the scales pass takes four rows of one group (groups a multiple of four, up to 2 M of them: 4096 x 8192) or of
    four groups (48 columns, 4100 x 8192); rows that are no multiple of four, and fewer than four."""
    x = synth.student_t_bf16((rows, cols), 3, 0.1, seed=rows + cols)
    out = qii.NVFP4Tensor.empty(rows, cols)
    w = ws(qii.qii_quantize_posthoc_workspace_bytes(rows, cols))
    w.fill_(0x7E)
    qii.qii_quantize_nvfp4(to_dev(x), False, qii.MS_EDEN_PH, rht, 31, 32, None, out, w)
    if rows * cols > 1 << 22:   # the oracle on a part: the scale bytes of the last rows depend on the tensor's maximum only
        tail = rows // 4 * 4 - 8
        top = torch.empty(1, device="cuda")
        qii.qii_absmax(to_dev(x), False, rht, 31, top)
        given = qii.NVFP4Tensor.empty(rows, cols)
        qii.qii_quantize_nvfp4(to_dev(x), False, qii.MS_EDEN_PH, rht, 31, 32, top, given, w)
        part = qii.NVFP4Tensor.empty(tail, cols)   # (2 M groups and more less two rows of threads: the other form or the same)
        qii.qii_quantize_nvfp4(to_dev(x[:tail]), False, qii.MS_EDEN_PH, rht, 31, 32, top, part, w)
        assert torch.equal(out.scales, given.scales) and torch.equal(out.tensor_scale, given.tensor_scale)
        assert torch.equal(out.scales[:tail], part.scales) and torch.equal(out.codes[:tail], part.codes)
        return
    assert_nv_equal(out, oracle.quantize(x, qii.MS_EDEN_PH, rht_group=rht, seed_rht=31, seed_sr=32), "rows")
