// Both MS-EDEN quantizations of a dense bf16 matrix from one read (quantize_pair_block.h), and the abs-max passes by
// 128 x 128 tiles.
#include "quantize_pair_block.h"

namespace qii {
namespace {

template <int kMode, bool kWords, bool kStream>
__global__ __launch_bounds__(512) void quantize_pair_kernel(PairArgs a)
{
    __shared__ __align__(16) uint8_t tile[kPairImage];
    pair_block<kMode, false, kWords, kStream>(a, (int)blockIdx.x, tile);
}

// Abs-max of a rotated matrix along its columns.  The result word takes one atomic per block, and such atomics on one
// address are resolved one after the other (about 10 ns each), so the pass runs as few blocks; to keep the memory busy
// all the same a block is 16 waves: groups of four waves, each group with an LDS image of its own (as above), that
// stride over the 128 x 128 tiles with the next tile's loads in flight.  Up to 512 tiles a block is one
// group and one tile: small tensors need every compute unit.
// 8192 x 8192 along the columns: 39 -> 30 us against a pass whose two waves per SIMD loaded 4 bytes
// per lane and row.
template <int kGroups>
__global__ __launch_bounds__(256 * kGroups) void absmax_tiles_kernel(PairArgs a, int tiles)
{
    extern __shared__ __align__(16) uint8_t images[];
    __shared__ float wave_m[4 * kGroups];
    const int t = threadIdx.x & 255, lane = t & 63;
    const int wave16 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave16 & 3, group = wave16 >> 2;
    uint8_t *tile = images + group * (128 * 256);
    const int stride = (int)gridDim.x * kGroups;
    // (consecutive tiles, which share rows, go to the groups of one block)
    int id = (int)blockIdx.x * kGroups + group;
    u32x4 w[8];
    auto load = [&](int n) {   // a tile beyond the last reads as zeros
        const int ty = n / a.tiles_x, tx = n - ty * a.tiles_x;
        const __amdgpu_buffer_rsrc_t src = region(a.x + (int64_t)ty * 128 * a.ld + (int64_t)tx * 128, n < tiles ? (127 * a.ld + 128) * 2 : 0);
        const uint32_t voff = (uint32_t)(((t >> 4) * a.ld + (t & 15) * 8) * 2);
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b128(src, voff, (int)(i * 16 * a.ld * 2), 0);
    };
    load(id);
    float m = 0.0f;
    const int rounds = (tiles + stride - 1) / stride;   // the same for every group: the barriers are the block's
    for (int k = 0; k < rounds; ++k) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = (t >> 4) + 16 * i, p = (t & 15) ^ (2 * (r >> 5));
            *reinterpret_cast<u32x4 *>(tile + r * 256 + p * 16) = w[i];
        }
        __syncthreads();
        id += stride;
        if (k + 1 < rounds) load(id);
        {
            const int q = lane & 3, jp = lane >> 2;
            const uint8_t *src = tile + (32 * q) * 256 + 4 * ((16 * wave + jp) ^ (8 * q));
            const uint32_t sw = q == 0 ? a.c.sign[0] : q == 1 ? a.c.sign[1] : q == 2 ? a.c.sign[2] : a.c.sign[3];
#pragma unroll
            for (int e = 0; e < 2; ++e) {   // one column after the other: 32 registers instead of 64
                float v[32];
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const uint32_t raw = *reinterpret_cast<const uint32_t *>(src + i * 256), flip = ((sw >> i) & 1u) << 31;
                    v[i] = u2f((e == 0 ? raw << 16 : raw & 0xFFFF0000u) ^ flip);
                }
                fwht128_quad<false>(v, q);
                m = fmaxf(m, fmaxf(group_absmax(v), group_absmax(v + 16)));
            }
        }
        __syncthreads();   // the images are free again
    }
    m = wave_max(__builtin_fmaf(m, kInvSqrt128, 0.0f));   // the scaling the rotation left out
    if (lane == 0) wave_m[wave16] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 1; i < 4 * kGroups; ++i) m = fmaxf(m, wave_m[i]);
        if (a.words) a.c.amax_out[blockIdx.x] = f2u(m);
        else max_to_global(m, a.c.amax_out);
    }
}

// Abs-max along the rows and the columns from one read: blocks as in the quantizer (waves 0..3 take the rows, 4..7 the columns).
// The result words take one atomic per block, and such atomics on one address are resolved one after the other (about 10 ns
// each), so the pass runs as few blocks as fill the chip: they stride over the tiles, the next tile's loads in flight and two
// LDS images in turn (one barrier a tile: a wave that fills an image has passed the barrier that the last readers of that image
// reach after their reads).  Instruction issue and the waits between a tile's steps bound it.  Before, groups of four waves did
// the rows and then the columns of a tile, 12 waves a block between common barriers.  Whole MS-EDEN pair calls, us, before :
// now: 8192 x 8192 115.7 : 101.8, 16384 x 2048 64.0 : 58.6, 4096 x 4096 42.3 : 32.3, 4096 x 2560 31.5 : 26.6, 2048 x 2176
// 23.6 : 21.3, 1024 x 1024 17.2 : 16.6; one image 115.5, 59.4, 33.4, 26.6, 21.4, 17.1 where these took 113.3, 58.6, 32.8,
// 26.6, 21.3, 17.1; three blocks per unit of 80 registers, one column at a time, no faster (4096 x 4096 34.2).
constexpr int kAbsmaxPairBlocks = 512;   // two per compute unit

__global__ __launch_bounds__(512, 4) void absmax_pair_kernel(PairArgs a, int tiles)
{
    extern __shared__ __align__(16) uint8_t images[];
    __shared__ float wave_m[8];
    const int t = threadIdx.x, lane = t & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(t >> 6), wave = wave_id & 3;
    const bool take_rows = wave_id < 4;   // (wave-uniform)
    u32x4 w[4];
    const uint32_t voff = (uint32_t)(((t >> 4) * a.ld + (t & 15) * 8) * 2);
    auto load = [&](int n) {
        const int ty = n / a.tiles_x, tx = n - ty * a.tiles_x;
        const __amdgpu_buffer_rsrc_t src = region(a.x + (int64_t)ty * 128 * a.ld + (int64_t)tx * 128, (127 * a.ld + 128) * 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b128(src, voff, (int)(i * 32 * a.ld * 2), 0);
    };
    int id = (int)blockIdx.x;
    load(id);
    const OctetLane L = octet_lane(lane, a.r.sign);
    const int q = lane & 3, jp = lane >> 2;
    const uint32_t sign_word = q == 0 ? a.c.sign[0] : q == 1 ? a.c.sign[1] : q == 2 ? a.c.sign[2] : a.c.sign[3];
    float m = 0.0f;
    for (int k = 0; id < tiles; ++k) {   // uniform
        uint8_t *tile = images + (k & 1) * kPairImage;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = (t >> 4) + 32 * i, p = (t & 15) ^ (2 * (r >> 5));
            *reinterpret_cast<u32x4 *>(tile + r * 256 + p * 16) = w[i];
        }
        id += (int)gridDim.x;
        if (id < tiles) load(id);
        __syncthreads();
        if (take_rows) {
            uint32_t mask[8], sign16 = L.sign16;
            asm("" : "+v"(sign16));
            make_masks<true>(sign16, mask);
            const int quad = 8 * wave + (lane >> 3);
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const uint8_t *src = tile + (4 * quad + it) * 256 + ((L.blk ^ wave) * 32);
                const u32x4 q0 = *reinterpret_cast<const u32x4 *>(src), q1 = *reinterpret_cast<const u32x4 *>(src + 16);
                const uint32_t w8[8] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3]};
                float v[16];
                unpack_bf16x16<true>(w8, v, mask);
                rht128_lane<false>(v, L);
                m = fmaxf(m, group_absmax(v));
            }
        } else {
            const uint8_t *src = tile + (32 * q) * 256 + 4 * ((16 * wave + jp) ^ (8 * q));
            uint32_t sw = sign_word;
            asm("" : "+v"(sw));   // (the 32 sign masks are formed again for each tile: kept, they would take 32 registers)
            float v[2][32];
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const uint32_t raw = *reinterpret_cast<const uint32_t *>(src + i * 256), flip = ((sw >> i) & 1u) << 31;
                v[0][i] = u2f((raw << 16) ^ flip);
                v[1][i] = u2f((raw & 0xFFFF0000u) ^ flip);
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                fwht128_quad<false>(v[e], q);
                m = fmaxf(m, fmaxf(group_absmax(v[e]), group_absmax(v[e] + 16)));
            }
        }
    }
    m = wave_max(__builtin_fmaf(m, kInvSqrt128, 0.0f));   // the scaling the rotation left out
    if (lane == 0) wave_m[wave_id] = m;
    __syncthreads();
    if (t < 2) {
        m = fmaxf(fmaxf(wave_m[4 * t], wave_m[4 * t + 1]), fmaxf(wave_m[4 * t + 2], wave_m[4 * t + 3]));
        uint32_t *out = t == 0 ? a.r.amax_out : a.c.amax_out;
        if (a.words) out[blockIdx.x] = f2u(m);
        else max_to_global(m, out);
    }
}

hipError_t launch_absmax_pair(const PairArgs &a, int tiles, hipStream_t s)
{
    const int lds = (tiles > kAbsmaxPairBlocks ? 2 : 1) * kPairImage;
    const hipError_t e = allow_dynamic_lds<absmax_pair_kernel>(2 * kPairImage);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(absmax_pair_kernel, dim3((unsigned)(tiles < kAbsmaxPairBlocks ? tiles : kAbsmaxPairBlocks)), dim3(512), lds, s, a, tiles);
    return hipGetLastError();
}

template <int kGroups>
hipError_t launch_absmax_columns(const PairArgs &a, int tiles, hipStream_t s)
{
    constexpr int lds = kGroups * 128 * 256, most = kGroups == 1 ? 512 : 256;
    const hipError_t e = allow_dynamic_lds<absmax_tiles_kernel<kGroups>>(lds);
    if (e != hipSuccess) return e;
    const int blocks = (tiles + kGroups - 1) / kGroups;
    hipLaunchKernelGGL((absmax_tiles_kernel<kGroups>), dim3((unsigned)(blocks < most ? blocks : most)), dim3(256 * kGroups), lds, s, a, tiles);
    return hipGetLastError();
}

}  // namespace

// dense bf16, no transposition, both dimensions multiples of 128, 16-byte aligned rows, and
// offsets inside a tile's rows that fit the 32-bit fields of a buffer descriptor
bool pair_kernel_applies(const Source &src, int64_t rows, int64_t cols)
{
    return src.kind == kSrcBF16 && !src.transpose && rows > 0 && cols > 0 && rows % 128 == 0 && cols % 128 == 0 &&
           src.ld % 8 == 0 && (reinterpret_cast<uintptr_t>(src.x) & 15) == 0 && src.ld <= ((int64_t)1 << 21) &&
           cols <= ((int64_t)1 << 23) && rows <= ((int64_t)1 << 23) && (rows / 128) * (cols / 128) < ((int64_t)1 << 31);
}

// Non-temporal stores of the codes get out of the loads' way, but a product that follows finds the codes in the caches only after
// ordinary ones.  us, ordinary : non-temporal, post hoc scheme (Algorithm 1 alike), the call alone, and with a product of each orientation behind it:
//    512 x  512  9.8 :  9.8   19.1 : 19.7       1024 x 1024 10.1 : 10.1   23.1 : 23.3       1024 x 2048 10.3 : 10.3   28.4 : 28.3
//   1536 x 1536 10.8 : 10.8   40.1 : 39.6       2048 x 4096 16.8 : 16.3   84.8 : 84.7       4096 x 4096 27.0 : 26.3    147 : 149
//   16384 x 2048 43.2 : 42.2   251 : 252        8192 x 8192 75.9 : 74.9    450 : 452
// From 2 M elements the call gains 1 to 3 %, and the three together lose at most 1 %, about as much; below there is nothing to gain.
constexpr int kStreamTiles = 128;
static_assert(kSlotWords < kStreamTiles, "a pair whose blocks leave words has fewer tiles");

hipError_t launch_quantize_pair(const PairQuantizeArgs &p, hipStream_t s)
{
    const PairArgs a = pair_args(p);
    const int tiles = (int)((p.rows / 128) * (p.cols / 128));
    const dim3 grid((unsigned)tiles), block(512);
#define QII_PAIR(MODE, WORDS)                                                                                               \
    do {                                                                                                                   \
        if (tiles >= kStreamTiles) hipLaunchKernelGGL((quantize_pair_kernel<MODE, WORDS, true>), grid, block, 0, s, a);     \
        else hipLaunchKernelGGL((quantize_pair_kernel<MODE, WORDS, false>), grid, block, 0, s, a);                          \
    } while (0)
    if (p.mode == QII_MS_EDEN_PH) QII_PAIR(QII_MS_EDEN_PH, false);
    else if (a.words) hipLaunchKernelGGL((quantize_pair_kernel<QII_MS_EDEN, true, false>), grid, block, 0, s, a);   // (small tensors only)
    else QII_PAIR(QII_MS_EDEN, false);
#undef QII_PAIR
    return hipGetLastError();
}

// Along the columns alone: the tile kernel or absmax_cols_kernel (quantize_cols.hip).  The tile kernel works in rounds of 1024
// tiles (four a block, a block per unit), so a round with few tiles costs as much as a full one; below one round it has fewer
// waves in flight than the other.  The other reads 64-byte pieces of a source row, and fetches a line twice unless
// neighbouring column blocks run on one die (`local`: the number of its row blocks is a multiple of 8, or its stripe order
// applies).  Whole MS-EDEN calls, us, columns kernel : tile kernel, both with a cleared word and atomics, on one box (a quantizer call whose blocks leave
// words goes by absmax_tiles_words; this is the rule of the others and of qii_absmax):
//   128 tiles  1024 x 2048 13.0 : 12.5            4096 x  512 (local) 13.0 : 12.5   128 x 16384 (local) 15.5 : 11.8
//   256 tiles  2048 x 2048 14.6 : 15.7            4096 x 1024 (local) 14.5 : 14.2   512 x  8192 (local) 14.6 : 15.0
//   512 tiles  4096 x 2048 (local) 17.0 : 18.8    1024 x 8192 (local) 17.3 : 17.5
//  1088 tiles  8704 x 2048 34.7 : 36.0            2176 x 8192 (local) 25.9 : 30.2
//  1280 tiles 10240 x 2048 38.0 : 36.0            4096 x 5120 (local) 27.5 : 32.6
//  1792 tiles  7168 x 4096 47.2 : 41.7           28672 x 1024 (local) 34.2 : 35.3
//  2048 tiles                                     4096 x 8192 (local) 41.1 : 37.5
//  2112 and 2176 tiles  8448 x 4096 52.8 : 49.1  2176 x 16384 (local) 42.8 : 44.6
//  2560 tiles 10240 x 4096 61.0 : 52.9            5120 x 8192 (local) 47.5 : 45.2
static bool columns_local(int64_t rows, int64_t cols) { return ((rows + 511) / 512) % 8 == 0 || (cols + 31) / 32 % 256 == 0; }

bool absmax_tiles_pay(int64_t rows, int64_t cols)
{
    const int64_t tiles = (rows / 128) * (cols / 128);
    if (tiles <= 128) return true;
    if (!columns_local(rows, cols)) return tiles >= 1280;
    return (tiles > 1792 && tiles <= 2048) || tiles >= 2560;
}

// A word per block, at most kSlotWords blocks, and no clearing launch.  Both orientations: a tile a block.  Along the columns alone a
// block has one, two or four groups and a tile each.  Whole MS-EDEN calls, us, clearing and atomics (the form above) : words: both 128 x 128
// 15.5 : 11.9, 1024 x 1024 16.0 : 12.9; columns 1024 x 1024 12.9 : 11.2, 2048 x 1024 13.5 : 12.5, 2048 x 2048 16.7 : 15.3, but 512 x 8192
// (local) 14.8 : 14.9; 128 tiles in blocks of four groups 13.6 : 14.0.  Beyond 128 tiles the columns kernel is the other way, in blocks of four
// waves below one another: 635 shapes of 129 to 256 tiles, medians, columns kernel : words: one such block high 15.0 : 14.3, more and a whole last
// one 14.1 : 13.3, three waves of the last at work 13.9 : 13.4; two of them 12.9 : 13.5, one 13.6 : 14.3 (5760 x 512 11.6 : 13.2).
int absmax_tiles_words(int64_t rows, int64_t cols, bool both)
{
    const int64_t tiles = (rows / 128) * (cols / 128);
    if (both) return tiles <= kSlotWords ? (int)tiles : 0;
    if (tiles > 4 * kSlotWords) return 0;
    const int64_t last = rows % 512;   // rows of the columns kernel's last block
    if (tiles > 2 * kSlotWords && (columns_local(rows, cols) || (rows > 512 && (last == 128 || last == 256)))) return 0;
    const int64_t groups = tiles <= kSlotWords ? 1 : tiles <= 2 * kSlotWords ? 2 : 4;
    return (int)((tiles + groups - 1) / groups);
}

// max |rotated| along the columns and, amax_r not null, along the rows of a matrix that pair_kernel_applies to; words:
// absmax_tiles_words of them at each, else (words == 0) one word that must hold 0
hipError_t launch_absmax_tiles(const Source &src, int64_t rows, int64_t cols, uint64_t seed_rht_r, float *amax_r, uint64_t seed_rht_c,
                               float *amax_c, hipStream_t s, int words)
{
    PairArgs a = {};
    a.words = words;
    a.x = reinterpret_cast<const uint16_t *>(src.x);
    a.ld = src.ld; a.rows = rows; a.cols = cols;
    a.tiles_x = (int)(cols / 128);
    const U4 wr = philox_seeded(seed_rht_r, 0, 0, 0, kStreamRht), wc = philox_seeded(seed_rht_c, 0, 0, 0, kStreamRht);
    a.r.sign[0] = wr.x; a.r.sign[1] = wr.y; a.r.sign[2] = wr.z; a.r.sign[3] = wr.w;
    a.c.sign[0] = wc.x; a.c.sign[1] = wc.y; a.c.sign[2] = wc.z; a.c.sign[3] = wc.w;
    a.r.amax_out = reinterpret_cast<uint32_t *>(amax_r);
    a.c.amax_out = reinterpret_cast<uint32_t *>(amax_c);
    const int tiles = (int)((rows / 128) * (cols / 128));
    if (amax_r) return launch_absmax_pair(a, tiles, s);
    if (tiles <= (words ? kSlotWords : 512)) return launch_absmax_columns<1>(a, tiles, s);
    return words && tiles <= 2 * kSlotWords ? launch_absmax_columns<2>(a, tiles, s) : launch_absmax_columns<4>(a, tiles, s);
}

}  // namespace qii
