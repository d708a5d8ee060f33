// Re-quantization of a saved NVFP4 tensor with transposition (quantize_requant_block.h) and its abs-max pass.
#include "quantize_requant_block.h"

namespace qii {
namespace {

// W and X of a backward pass go through one launch: the first n0 blocks take a0, the others a1 (a call for one
// tensor gives all blocks to a0)
template <int kMode, bool kRht, int kChunks>
__global__ __launch_bounds__(256 * kChunks) void requantize_cols_kernel(RequantArgs a0, RequantArgs a1, int n0)
{
    const bool first = (int)blockIdx.x < n0;   // uniform
    RequantArgs a = a0;
    if (!first) a = a1;
    extern __shared__ __align__(16) uint8_t image[];
    requant_block<kMode, kRht, kChunks>(a, (int)blockIdx.x - (first ? 0 : n0), image);
}

// Abs-max pass: at most 512 blocks (one atomic each: such atomics on one address are resolved one after the
// other) that stride over the tiles, the next tile's loads in flight.
template <bool kRht, int kChunks>
__global__ __launch_bounds__(256 * kChunks) void requantize_absmax_kernel(RequantArgs a0, RequantArgs a1, int n0)
{
    const bool first = (int)blockIdx.x < n0;   // uniform
    RequantArgs a = a0;
    if (!first) a = a1;
    const int block = (int)blockIdx.x - (first ? 0 : n0), blocks = first ? n0 : (int)gridDim.x - n0;
    extern __shared__ __align__(16) uint8_t image[];
    __shared__ float wave_m[4 * kChunks];
    const int lane = threadIdx.x & 63, q = lane & 3;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float m = 0.0f;
    RawTile raw;
    int64_t chunk0, col0;
    tile_origin<kChunks>(a, block, chunk0, col0);
    load_tile<kChunks>(raw, a, chunk0, col0);
    for (int id = block; id < a.tiles; id += blocks) {
        const bool live = (chunk0 + (wave >> 2)) * 128 < a.C;   // wave-uniform
        const int64_t j0 = col0 + 32 * (wave & 3) + 2 * (lane >> 2);
        store_image<kChunks>(raw, image);
        if (id + blocks < a.tiles) {
            tile_origin<kChunks>(a, id + blocks, chunk0, col0);
            load_tile<kChunks>(raw, a, chunk0, col0);
        }
        __syncthreads();
        if (live) {
            float v[2][32];
            read_columns<kRht>(v, a, image, wave, lane);
            if (kRht) {
                fwht128_quad<false>(v[0], q);
                fwht128_quad<false>(v[1], q);
            }
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (j0 + e < a.R) m = fmaxf(m, fmaxf(group_absmax(v[e]), group_absmax(v[e] + 16)));
        }
        __syncthreads();   // the image is free again
    }
    if (kRht) m = __builtin_fmaf(m, kInvSqrt128, 0.0f);   // the scaling the rotation left out
    m = wave_max(m);
    if (lane == 0) wave_m[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 1; i < 4 * kChunks; ++i) m = fmaxf(m, wave_m[i]);
        if (a.words) a.amax_out[block] = f2u(m);
        else max_to_global(m, a.amax_out);
    }
}

template <auto kKernel>
hipError_t launch(dim3 grid, dim3 block, int lds, hipStream_t s, const RequantArgs *a, int count, int n0)
{
    const hipError_t e = allow_dynamic_lds<kKernel>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kKernel, grid, block, lds, s, a[0], a[count - 1], n0);
    return hipGetLastError();
}

}  // namespace

// a transposed NVFP4 source whose stored rows are a multiple of 128 (offsets within a tile's rows stay below 2^31)
bool requant_kernels_apply(const Source &src, int64_t R, int64_t C)
{
    return src.kind == kSrcNVFP4 && src.transpose && C % 128 == 0 && src.ld <= (int64_t)1 << 21 &&
           ((R + 127) / 128) * (C / 128) < ((int64_t)1 << 31);
}

int requant_amax_words(const Source &src, int64_t R, int64_t C)
{
    if (!requant_kernels_apply(src, R, C)) return 0;
    const int n = requant_blocks(&R, &C, 1, 0);
    return n <= kSlotWords ? n : 0;
}

int requant_blocks(const int64_t *R, const int64_t *C, int count, int i)
{
    return (int)tiles_of(R[i], C[i], chunks_per_block(R, C, count));
}

hipError_t launch_absmax_requant(const Source *src, const int64_t *R, const int64_t *C, int rht, const uint64_t *seed_rht,
                                 float *const *amax, int count, hipStream_t s, int words)
{
    const int ch = chunks_per_block(R, C, count);
    RequantArgs a[2];
    int64_t all = 0;
    for (int i = 0; i < count; ++i) {
        a[i] = make_args(src[i], R[i], C[i], seed_rht[i], 0, ch);
        a[i].amax_out = reinterpret_cast<uint32_t *>(amax[i]);
        a[i].words = words ? a[i].tiles : 0;
        all += a[i].tiles;
    }
    // at most 512 blocks, shared out by size
    int n[2] = {0, 0};
    for (int i = 0; i < count; ++i) {
        n[i] = all <= 512 ? a[i].tiles : (int)(512 * (int64_t)a[i].tiles / all);
        if (n[i] < 1) n[i] = 1;
    }
    const dim3 grid((unsigned)(n[0] + n[1])), block(256 * ch);
    if (ch == 2)
        return rht ? launch<requantize_absmax_kernel<true, 2>>(grid, block, 2 * kImage, s, a, count, n[0])
                   : launch<requantize_absmax_kernel<false, 2>>(grid, block, 2 * kImage, s, a, count, n[0]);
    return rht ? launch<requantize_absmax_kernel<true, 1>>(grid, block, kImage, s, a, count, n[0])
               : launch<requantize_absmax_kernel<false, 1>>(grid, block, kImage, s, a, count, n[0]);
}

hipError_t launch_quantize_requant(const QuantizeArgs *q, int count, hipStream_t s)
{
    int64_t R[2], C[2];
    for (int i = 0; i < count; ++i) { R[i] = q[i].R; C[i] = q[i].C; }
    const int ch = chunks_per_block(R, C, count);
    RequantArgs a[2];
    int blocks = 0;
    for (int i = 0; i < count; ++i) {
        a[i] = requant_args(q[i], ch);
        blocks += a[i].tiles;
    }
    const dim3 grid((unsigned)blocks), block(256 * ch);
#define QII_REQ(MODE, RHT)                                                                                                      \
    return ch == 2 ? launch<requantize_cols_kernel<MODE, RHT, 2>>(grid, block, 2 * kImage, s, a, count, a[0].tiles)             \
                   : launch<requantize_cols_kernel<MODE, RHT, 1>>(grid, block, kImage, s, a, count, a[0].tiles)
#define QII_REQ_MODE(RHT)                                        \
    switch (q[0].mode) {                                         \
        case QII_RTN: QII_REQ(QII_RTN, RHT);                     \
        case QII_SR: QII_REQ(QII_SR, RHT);                       \
        case QII_RTN_46: QII_REQ(QII_RTN_46, RHT);               \
        case QII_MS_EDEN_PH: QII_REQ(QII_MS_EDEN_PH, RHT);       \
        default: QII_REQ(QII_MS_EDEN, RHT);                      \
    }
    if (q[0].rht) QII_REQ_MODE(true)
    else QII_REQ_MODE(false)
#undef QII_REQ_MODE
#undef QII_REQ
}

}  // namespace qii
