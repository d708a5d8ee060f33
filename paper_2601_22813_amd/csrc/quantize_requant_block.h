// Re-quantization of a saved NVFP4 tensor with transposition (the backward pass's Q(W^T), Q(X^T)): source
// element (e2m1 * e4m3) * tensor_scale, scale groups and rotation chunks down the rows of the stored tensor.
//
// The source is 0.5625 bytes per element, so reading it column-wise element by element (one byte per row and
// column pair) would issue 64 load instructions per 64 elements and bind on address processing: 30.8 us for
// 16384 x 2048, four times its 44 MB at the copy rate.  Here a block takes a tile of 128 columns and one or two
// 128-row chunks: 16-byte pieces of code rows and their two scale bytes are loaded row-wise, the products
// e2m1 * e4m3 (at most 6 significant bits: exact in bf16) go to LDS as a bf16 image, and a lane quad then
// takes two columns of a chunk as in quantize_cols.hip (quad layout of quantize_lanes.h).  Two chunks
// per block where there are blocks enough: a column's codes then leave as 128 contiguous bytes.
//
// LDS image: row r (of 128 per chunk) keeps its 4-byte word w (two columns) at word
// w ^ 8 ((r / 32) ^ (r & 1)) ^ 4 (w / 32 & 1): the column reads of a wave (rows 32 q + i, q = 0..3, and
// 16 consecutive words) hit 32 different banks per half wave, and the 16-byte stores of 8 consecutive lanes
// (two rows of four pieces) 8 different bank groups.
#pragma once
#include "qii_device.h"
#include "qii_internal.h"
#include "quantize_core.h"
#include "quantize_lanes.h"

namespace qii {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct RequantArgs {
    const uint8_t *in_codes, *in_scales;
    const float *in_ts;
    int64_t ld;          // stored columns
    int64_t R, C;        // logical shape: R = stored columns (output rows), C = stored rows
    uint32_t sign[4];
    uint64_t seed_sr;
    const float *amax;   // the tensor maximum: see slot_max
    uint8_t *codes;
    uint8_t *scales;
    float *tensor_scale;
    uint32_t *amax_out;  // abs-max kernel (one running word), heavy pass of the post hoc scheme (nullable there): the spread
    int words;           // words; or, words != 0, one word per block
    float *tbuf;         // post hoc scheme: corrected pseudo-scales [R][C/16]
    int64_t ksn;         // 0, or the K tiles of the main GEMM kernel's layout, which the scale bytes then go out in (modes with scale bytes)
    int tiles_x;         // tiles along a stored row
    int tiles;
};

constexpr uint32_t kNoLoad = 0xFFFFFFF0u;   // an offset beyond every descriptor: reads 0
constexpr int kImage = 128 * 256;           // LDS bytes of one chunk's 128 x 128 bf16 products

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const void *base, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}

// one thread's two pieces of a tile: 32 codes and two scale bytes each
struct RawTile {
    u32x4 c[2];
    uint32_t s0[2], s1[2];
};

// tile id -> first chunk and first column.  Consecutive block ids go to different dies: each die takes a
// contiguous run of tiles, column tiles fastest, so the halves of a source line are fetched through one L2.
template <int kChunks>
__device__ __forceinline__ void tile_origin(const RequantArgs &a, int id, int64_t &chunk0, int64_t &col0)
{
    if ((a.tiles & 7) == 0) id = (id & 7) * (a.tiles >> 3) + (id >> 3);
    chunk0 = (int64_t)(id / a.tiles_x) * kChunks;
    col0 = (int64_t)(id % a.tiles_x) * 128;
}

template <int kChunks>
__device__ __forceinline__ void load_tile(RawTile &r, const RequantArgs &a, int64_t chunk0, int64_t col0)
{
    const int t = threadIdx.x;
    const int64_t row0 = chunk0 * 128, left = a.C - row0, rows = left < 128 * kChunks ? left : 128 * kChunks;
    const int64_t cp = a.ld / 2, sp = a.ld / 16;
    const __amdgpu_buffer_rsrc_t rc = rows_rsrc(a.in_codes + row0 * cp, rows * cp), rs = rows_rsrc(a.in_scales + row0 * sp, rows * sp);
    const int p = t & 3;
    const bool in0 = col0 + 32 * p < a.ld, in1 = col0 + 32 * p + 16 < a.ld;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (t >> 2) + 64 * kChunks * i;
        // (a piece whose second half lies beyond the row reads on into the next one; those columns are dropped later)
        r.c[i] = __builtin_amdgcn_raw_buffer_load_b128(rc, in0 ? (uint32_t)(row * cp + col0 / 2 + 16 * p) : kNoLoad, 0, 0);
        const uint32_t so = (uint32_t)(row * sp + col0 / 16 + 2 * p);
        r.s0[i] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rs, in0 ? so : kNoLoad, 0, 0);
        r.s1[i] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rs, in1 ? so + 1u : kNoLoad, 0, 0);
    }
}

// eight codes (a dword) times their scale -> 16 bytes of exact bf16 products
__device__ __forceinline__ u32x4 products(uint32_t codes, float x8)
{
    u32x4 w;
#define QII_PAIR(I)                                                                               \
    do {                                                                                          \
        const float2_t c = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, 1.0f, I);              \
        w[I] = __builtin_amdgcn_perm(f2u(c[1] * x8), f2u(c[0] * x8), 0x07060302u);                \
    } while (0)
    QII_PAIR(0); QII_PAIR(1); QII_PAIR(2); QII_PAIR(3);
#undef QII_PAIR
    return w;
}

template <int kChunks>
__device__ __forceinline__ void store_image(const RawTile &r, uint8_t *image)
{
    const int t = threadIdx.x, p = t & 3;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (t >> 2) + 64 * kChunks * i, r7 = row & 127;
        uint8_t *dst = image + (row >> 7) * kImage + r7 * 256;
        const int flip = 2 * ((r7 >> 5) ^ (r7 & 1)) ^ (p >> 1);   // in 16-byte slots; slot of dword k: 4 p + k
        const float x0 = e4m3_decode(r.s0[i]), x1 = e4m3_decode(r.s1[i]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<u32x4 *>(dst + ((4 * p + k) ^ flip) * 16) = products(r.c[i][k], k < 2 ? x0 : x1);
    }
}

// this lane's 32 rows (32 q .. 32 q + 31 of its wave's chunk) of its two columns, times the tensor scale, with
// the rotation signs: multiplying by +-x32 is the same rounding as multiplying by x32 and flipping
template <bool kRht>
__device__ __forceinline__ void read_columns(float v[2][32], const RequantArgs &a, const uint8_t *image, int wave, int lane)
{
    const int q = lane & 3, w = 16 * (wave & 3) + (lane >> 2);
    const uint8_t *base = image + (wave >> 2) * kImage + 32 * q * 256;
    const int ws = (w ^ (8 * q)) ^ (4 * ((w >> 5) & 1));
    const uint8_t *even = base + 4 * ws, *odd = base + 4 * (ws ^ 8);
    const uint32_t sw = q == 0 ? a.sign[0] : q == 1 ? a.sign[1] : q == 2 ? a.sign[2] : a.sign[3];
    const float x32 = *a.in_ts;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const uint32_t raw = *reinterpret_cast<const uint32_t *>(((i & 1) ? odd : even) + i * 256);
        const float x = kRht ? u2f(f2u(x32) ^ ((sw << (31 - i)) & 0x80000000u)) : x32;
        v[0][i] = u2f(raw << 16) * x;
        v[1][i] = u2f(raw & 0xFFFF0000u) * x;
    }
}

// the four scale groups of a lane (two per column), their stores
template <int kMode, int kFast, bool kMayTile>
__device__ __forceinline__ void finish_groups(const RequantArgs &a, float v[2][32], const TensorConsts &tc, const uint32_t draw[2][2],
                                              int64_t chunk, int64_t j0, int q, const float *inv_tab)
{
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        uint32_t codes[4], sc = 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            sc |= quantize_group16<kMode, kFast, true>(v[e] + 16 * h, tc, draw[e][h], a.seed_sr, j0 + e, chunk * 8 + 2 * q + h,
                                                       codes + 2 * h, inv_tab) << (8 * h);
        if (tc.zero) { codes[0] = codes[1] = codes[2] = codes[3] = 0u; sc = 0u; }   // uniform: an all-zero tensor is emitted as zero bytes
        const uint2 s8 = gather_quad_scales(sc, q);
        if (j0 + e < a.R) {
            store_codes16(a.codes + (j0 + e) * (a.C / 2) + chunk * 64 + 16 * q, codes[0], codes[1], codes[2], codes[3]);
            if (q == 0)
                *reinterpret_cast<uint2 *>(kMayTile && a.ksn ? tiled_scales(a.scales, a.ksn, j0 + e, chunk) : a.scales + (j0 + e) * (a.C / 16) + chunk * 8) = s8;
        }
    }
}

// 256 kChunks threads; image: kChunks * kImage bytes of LDS; kMayTile: heeds ksn; Args: as for pair_block
template <int kMode, bool kRht, int kChunks, bool kMayTile = false, class Args = const RequantArgs>
__device__ __forceinline__ void requant_block(Args a, int block, uint8_t *image)
{
    __shared__ float inv_tab[128], wave_m[4 * kChunks];
    const int lane = threadIdx.x & 63, q = lane & 3;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t chunk0, col0;
    tile_origin<kChunks>(a, block, chunk0, col0);
    const float word = kMode != QII_MS_EDEN_PH ? slot_word(a.amax, a.words) : 0.0f;
    RawTile raw;
    load_tile<kChunks>(raw, a, chunk0, col0);
    // (the heavy pass of the post hoc scheme knows no tensor maximum: tc stays unused there)
    TensorConsts tc = TensorConsts{};
    if (kMode != QII_MS_EDEN_PH) {
        tc = tensor_consts(kMode, slot_max(a.amax, a.words, word));
        if (block == 0 && threadIdx.x == 0) *a.tensor_scale = tc.x32;
        fill_inv_table(inv_tab, tc);
    }
    store_image<kChunks>(raw, image);
    __syncthreads();
    const int64_t chunk = chunk0 + (wave >> 2), j0 = col0 + 32 * (wave & 3) + 2 * (lane >> 2);
    const bool live = chunk * 128 < a.C;   // wave-uniform
    float v[2][32];
    float m = 0.0f;
    if (live) {
        read_columns<kRht>(v, a, image, wave, lane);
        if (kRht) {
            fwht128_quad(v[0], q);
            fwht128_quad(v[1], q);
        }
    }
    if (kMode == QII_MS_EDEN_PH) {
        if (live) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                uint32_t codes[4];
                float t[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float gmax;
                    t[h] = posthoc_group16(v[e] + 16 * h, codes + 2 * h, gmax);
                    if (j0 + e < a.R) m = fmaxf(m, gmax);
                }
                if (j0 + e < a.R) {
                    *reinterpret_cast<uint4 *>(a.codes + (j0 + e) * (a.C / 2) + chunk * 64 + 16 * q) =
                        make_uint4(codes[0], codes[1], codes[2], codes[3]);
                    *reinterpret_cast<float2 *>(a.tbuf + (j0 + e) * (a.C / 16) + chunk * 8 + 2 * q) = make_float2(t[0], t[1]);
                }
            }
        }
        if (a.amax_out) {   // uniform
            m = wave_max(m);
            if (lane == 0) wave_m[wave] = m;
            __syncthreads();
            if (threadIdx.x == 0) {
#pragma unroll
                for (int i = 1; i < 4 * kChunks; ++i) m = fmaxf(m, wave_m[i]);
                leave_block_max(m, a.amax_out, a.words, block);
            }
        }
        return;
    }
    if (!live) return;
    uint32_t draw[2][2] = {{0u, 0u}, {0u, 0u}};
    if (kMode == QII_MS_EDEN) octet_draws(draw, a.seed_sr, chunk, j0, q);
    if (tc.fast) finish_groups<kMode, 1, kMayTile>(a, v, tc, draw, chunk, j0, q, inv_tab);   // uniform
    else finish_groups<kMode, 0, kMayTile>(a, v, tc, draw, chunk, j0, q, inv_tab);
}

inline RequantArgs make_args(const Source &src, int64_t R, int64_t C, uint64_t seed_rht, uint64_t seed_sr, int chunks)
{
    RequantArgs a;
    a.in_codes = (const uint8_t *)src.x; a.in_scales = src.scales; a.in_ts = src.ts; a.ld = src.ld; a.R = R; a.C = C;
    const U4 w = philox_seeded(seed_rht, 0, 0, 0, kStreamRht);
    a.sign[0] = w.x; a.sign[1] = w.y; a.sign[2] = w.z; a.sign[3] = w.w;
    a.seed_sr = seed_sr;
    a.amax = nullptr; a.codes = nullptr; a.scales = nullptr; a.tensor_scale = nullptr; a.amax_out = nullptr; a.tbuf = nullptr; a.words = 0; a.ksn = 0;
    a.tiles_x = (int)((R + 127) / 128);
    a.tiles = (int)((C / 128 + chunks - 1) / chunks) * a.tiles_x;
    return a;
}

inline RequantArgs requant_args(const QuantizeArgs &q, int chunks)
{
    RequantArgs a = make_args(q.src, q.R, q.C, q.seed_rht, q.seed_sr, chunks);
    a.amax = q.amax; a.codes = q.codes; a.scales = q.scales; a.tensor_scale = q.tensor_scale;
    a.tbuf = q.tbuf; a.amax_out = q.amax_accum; a.words = q.amax_words;
    a.ksn = q.tiled ? q.C / 256 : 0;
    return a;
}

inline int64_t tiles_of(int64_t R, int64_t C, int chunks) { return (R + 127) / 128 * ((C / 128 + chunks - 1) / chunks); }

// two chunks per block when that still gives every compute unit two blocks
inline int chunks_per_block(const int64_t *R, const int64_t *C, int count)
{
    int64_t tiles2 = 0;
    for (int i = 0; i < count; ++i) tiles2 += tiles_of(R[i], C[i], 2);
    return tiles2 >= 512 ? 2 : 1;
}

}  // namespace
}  // namespace qii
