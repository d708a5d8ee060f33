"""Both orientations of a matrix from one read (four waves of a block take the rows, four the columns): byte for byte the two
separate quantizations, from one tile to more than the chip holds at once, with a leading dimension beyond the row and an
all-zero tensor."""
import numpy as np
import pytest
import torch

from paper_2601_22813_amd import binding as qii
from paper_2601_22813_amd import synth

from gpu_util import to_dev, ws

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
