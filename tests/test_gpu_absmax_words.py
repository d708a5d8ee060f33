"""Algorithm 1 and the other one-pass modes on small tensors: the blocks of the abs-max pass leave a word each in a 256-byte slot
that nobody clears.  The largest entry in the first, a middle and the last tile, in a workspace of exactly that slot which held NaN before, gives
what a call gives that is told the maximum: at one block, where 64 words are just enough and where they no longer are (clearing and
atomics again), for each kernel that measures (rows; columns by tiles of one, two and four groups to a block; columns by
32-column blocks), and for both orientations of a pair."""
import pytest
import torch

from paper_2601_22813_amd import binding as qii

from gpu_util import ws

pytestmark = pytest.mark.gpu


def nan_slots(n):
    """n slots of 256 bytes that hold NaN, and a guard behind them."""
    return torch.full((256 * n + 256,), 0xFF, dtype=torch.uint8, device="cuda")


def spiked(rows, cols, dtype, r, c):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = 0.1 * torch.randn((rows, cols), device="cuda", generator=g)
    x[r, c] = 400.0
    return x.to(dtype)


def places(rows, cols):
    return (0, 0), (rows // 2, cols // 2), (rows - 1, cols - 1)


def same(a, b):
    assert torch.equal(a.tensor_scale, b.tensor_scale) and torch.equal(a.scales, b.scales) and torch.equal(a.codes, b.codes)


@pytest.mark.parametrize("rows,cols,transpose,mode,rht,dtype", [
    (1, 128, False, qii.MS_EDEN, 128, torch.bfloat16), (1021, 1024, False, qii.MS_EDEN, 128, torch.bfloat16),
    (1040, 1024, False, qii.SR, 128, torch.float32), (2048, 2048, False, qii.MS_EDEN, 128, torch.bfloat16),
    (2049, 2048, False, qii.MS_EDEN, 128, torch.bfloat16), (67, 9216, False, qii.SR, 128, torch.float32),
    # a wave's rounds at the lines of the rule: rotated 3, 4 in few blocks, 4 in 64, 5; unrotated bf16 19, 20; f32 6, 7 above 8 MiB, 10, 11 below it
    (3072, 128, False, qii.MS_EDEN, 128, torch.bfloat16), (3080, 128, False, qii.SR, 128, torch.float32), (4096, 128, False, qii.MS_EDEN, 128, torch.float32),
    (4100, 128, False, qii.MS_EDEN, 128, torch.bfloat16), (19456, 64, False, qii.RTN, 0, torch.bfloat16), (19460, 64, False, qii.RTN_46, 0, torch.bfloat16),
    (6144, 512, False, qii.RTN, 0, torch.float32), (6148, 512, False, qii.SR, 0, torch.float32),
    (10240, 128, False, qii.RTN, 0, torch.float32), (10244, 128, False, qii.RTN, 0, torch.float32),
    (2000, 1552, False, qii.RTN_46, 0, torch.float32), (1000, 1552, False, qii.RTN, 0, torch.bfloat16),
    (128, 128, True, qii.MS_EDEN, 128, torch.bfloat16), (1024, 1024, True, qii.MS_EDEN, 128, torch.bfloat16),
    (640, 1664, True, qii.MS_EDEN, 128, torch.bfloat16), (1024, 2048, True, qii.SR, 128, torch.bfloat16),
    (384, 5504, True, qii.MS_EDEN, 128, torch.bfloat16), (2048, 2048, True, qii.MS_EDEN, 128, torch.bfloat16),
    (512, 8192, True, qii.MS_EDEN, 128, torch.bfloat16), (1536, 2304, True, qii.SR, 128, torch.bfloat16),
    (1664, 1664, True, qii.MS_EDEN, 128, torch.bfloat16), (1792, 1280, True, qii.MS_EDEN, 128, torch.bfloat16), (1408, 1664, True, qii.MS_EDEN, 128, torch.bfloat16), (1024, 1000, True, qii.SR, 128, torch.float32),
    (1024, 1024, True, qii.MS_EDEN, 128, torch.float32), (1024, 1026, True, qii.MS_EDEN, 128, torch.float32),
    (1920, 520, True, qii.RTN, 0, torch.bfloat16)])
def test_words_of_one_tensor(rows, cols, transpose, mode, rht, dtype):
    R, C = (cols, rows) if transpose else (rows, cols)
    for r, c in places(rows, cols):
        x = spiked(rows, cols, dtype, r, c)
        out, given = qii.NVFP4Tensor.empty(R, C), qii.NVFP4Tensor.empty(R, C)
        w, top = nan_slots(1), torch.empty(1, device="cuda")
        qii.qii_quantize_nvfp4(x, transpose, mode, rht, 21, 22, None, out, w[:256])
        qii.qii_absmax(x, transpose, rht, 21, top)
        qii.qii_quantize_nvfp4(x, transpose, mode, rht, 21, 22, top, given, None)
        same(out, given)
        assert bool((w[256:] == 0xFF).all())


@pytest.mark.parametrize("rows,cols", [(128, 128), (1024, 1024), (640, 1664), (2048, 4096)])
def test_words_of_a_pair(rows, cols):
    for r, c in places(rows, cols):
        x = spiked(rows, cols, torch.bfloat16, r, c)
        pair = qii.NVFP4Tensor.empty(rows, cols), qii.NVFP4Tensor.empty(cols, rows)
        w = nan_slots(2)
        qii.qii_quantize_pair_nvfp4(x, qii.MS_EDEN, 21, 22, 23, 24, *pair, w[:512])
        for out, transpose, seed in ((pair[0], False, 21), (pair[1], True, 23)):
            given, top = qii.NVFP4Tensor.empty(out.rows, out.cols), torch.empty(1, device="cuda")
            qii.qii_absmax(x, transpose, 128, seed, top)
            qii.qii_quantize_nvfp4(x, transpose, qii.MS_EDEN, 128, seed, seed + 1, top, given, None)
            same(out, given)
        assert bool((w[512:] == 0xFF).all())


@pytest.mark.parametrize("T,d_in,d_out", [(640, 1248, 5376), (1408, 768, 256)])
def test_slots_that_one_launch_has_cleared_take_one_word(T, d_in, d_out):
    """A backward pass with an f32 gradient clears all four slots at once: its quantizers have no launch to save, and their abs-max
    passes run as many blocks as are fastest.  What lies behind the first word of each dense tensor's slot stays as it was."""
    assert qii.lib().qii_absmax_words(qii.F32, T, d_out, 0, 128) > 1   # (a call of its own would leave as many)
    g = torch.Generator(device="cuda").manual_seed(T)
    saved = []
    for rows in (T, d_out):
        saved.append(qii.NVFP4Tensor.empty(rows, d_in))
        qii.qii_quantize_nvfp4(torch.randn((rows, d_in), device="cuda", generator=g), False, qii.RTN, 0, 0, 0, None, saved[-1], ws(256))
    dX, dW = torch.empty((T, d_in), device="cuda"), torch.empty((d_out, d_in), device="cuda")
    w = ws(qii.qii_linear_bwd_mode_workspace_bytes(T, d_in, d_out, qii.MS_EDEN))
    w.fill_(0x7F)
    qii.qii_linear_bwd_mode(torch.randn((T, d_out), device="cuda", generator=g), *saved, 5, qii.MS_EDEN, dX, dW, w)
    for slot in (0, 2):   # along the rows and along the columns of the gradient
        maximum = w[256 * slot:256 * slot + 4].view(torch.float32).item()
        assert 3.0 < maximum < 8.0
        assert bool((w[256 * slot + 4:256 * slot + 256] == 0x7F).all())
    assert torch.isfinite(dX).all() and torch.isfinite(dW).all()
