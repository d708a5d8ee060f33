// The four quantizations of a layer's backward pass in one launch: Q(E) and Q(E^T) from one read of E
// (quantize_pair_block.h) by the first blocks, the re-quantizations of W and X (quantize_requant_block.h) by the others.
// None of the four needs another's result, and each alone leaves a small layer's GPU mostly idle: with tensors of
// 512 x 512 the two launches are 16 blocks of 9 us and 32 of 7, one after the other; with large ones the rounds of one
// fill the last, incomplete round of the other.  Whole backward passes, us, the launches one after the
// other -> this (with the four scales passes of the post hoc scheme in one launch as well): post hoc 128 x 128 -> 128 26.8 -> 16.7,
// 512 x 512 -> 512 28.4 -> 17.5, 1024 x 1024 -> 4096 58.4 -> 50.7, 2048 x 2048 -> 5632 130 -> 122.5, 16384 x 2048 -> 8192 951 -> 947;
// Algorithm 1 512 x 512 -> 512 31.0 -> 24.9, 4096 x 1024 -> 1024 65.5 -> 62.0, 16384 x 2048 -> 2048 339 -> 334.  Nothing is lost
// where the other form has blocks enough: an image takes the LDS that a compute unit's two blocks leave free anyway.
// Algorithm 1's scale bytes go out in the main GEMM kernel's layout where the product's inner dimension is a multiple of 256, with no
// re-tiling launch: 4096 x 4096 -> 4096 280.8 -> 270.8 us, 2048 x 2048 -> 5632 142.0 -> 136.6, 16384 x 2048 -> 2048 327.5 -> 321.2.
#include "quantize_pair_block.h"
#include "quantize_requant_block.h"

namespace qii {
namespace {

// Registers for three blocks per compute unit in the post hoc scheme, 80 (85 without a bound, two blocks: one spilled register more than
// pays for itself), and images of one chunk, which leave the LDS for three.  Kernel 16384 x 2048 -> 8192 172.5 -> 157.6 us, 2048 x 2048 -> 5632 29.1 ->
// 27.6; passes 892 -> 884, 118.1 -> 116.2, 4096 x 4096 -> 4096 234.3 -> 232.9.  (Either alone gains nothing; 55 registers, one column at a
// time, and four blocks lose what they gain.)  Algorithm 1's 94 registers would spill 22.
template <int kMode, int kChunks, bool kWords>
__global__ __launch_bounds__(512, kMode == QII_MS_EDEN_PH ? 6 : 4) void quantize_backward_kernel(PairArgs e, RequantArgs w, RequantArgs x, int n_e, int n_w)
{
    extern __shared__ __align__(16) uint8_t lds[];   // kChunks images of 32 KiB, the first of them a block's tile of E
    const int block = (int)blockIdx.x;               // (branches on it are uniform)
    if (block < n_e) {
        pair_block<kMode, true, kWords, false, const PairArgs &>(e, block, lds);   // (512 x 512 -> 512 17.5 us, with non-temporal stores 17.8)
        return;
    }
    if (kChunks == 1 && threadIdx.x >= 256) return;   // (a wave that has ended takes no part in barriers)
    const bool first = block < n_e + n_w;
    RequantArgs a = w;
    if (!first) a = x;
    requant_block<kMode, true, kChunks, true, const RequantArgs &>(a, block - n_e - (first ? 0 : n_w), lds);
}

template <int kMode, int kChunks, bool kWords>
hipError_t launch(const PairArgs &e, const QuantizeArgs q[2], hipStream_t s)
{
    const hipError_t err = allow_dynamic_lds<quantize_backward_kernel<kMode, kChunks, kWords>>(kChunks * kImage);
    if (err != hipSuccess) return err;
    const RequantArgs w = requant_args(q[0], kChunks), x = requant_args(q[1], kChunks);
    const int n_e = (int)((e.rows / 128) * (e.cols / 128));
    hipLaunchKernelGGL((quantize_backward_kernel<kMode, kChunks, kWords>), dim3((unsigned)(n_e + w.tiles + x.tiles)), dim3(512), kChunks * kImage, s,
                       e, w, x, n_e, w.tiles);
    return hipGetLastError();
}

}  // namespace

static_assert(kPairImage <= kImage, "a tile of E takes one image");

int backward_requant_blocks(int64_t R, int64_t C) { return (int)tiles_of(R, C, 1); }

hipError_t launch_quantize_backward(const PairQuantizeArgs &e, const QuantizeArgs q[2], hipStream_t s)
{
    const int64_t R[2] = {q[0].R, q[1].R}, C[2] = {q[0].C, q[1].C};
    const PairArgs p = pair_args(e);
    if (e.mode == QII_MS_EDEN_PH) return launch<QII_MS_EDEN_PH, 1, false>(p, q, s);
    if (chunks_per_block(R, C, 2) == 2) return p.words ? hipErrorInvalidValue : launch<QII_MS_EDEN, 2, false>(p, q, s);   // (words: small tensors only)
    return p.words ? launch<QII_MS_EDEN, 1, true>(p, q, s) : launch<QII_MS_EDEN, 1, false>(p, q, s);
}

}  // namespace qii
