// One read of a dense bf16 matrix x producing BOTH of its MS-EDEN quantizations: Q(x), scale
// groups and rotation chunks along the rows of x, and Q(x^T), along its columns, each with its own
// rotation and rounding seeds.  The backward pass of a linear layer (paper Sec. 5) needs the output
// gradient E in both orientations (dX = Q(E) Q(W^T)^T over d_out, dW = Q(E^T) Q(X^T)^T over the
// tokens); Sec. 7 ("Fused Re-Quantization Kernel") describes the backward quantizers as fused
// kernels around a single load of their operand.  Bytes are identical to those of the two
// separate quantizer calls.
//
// A block takes one 128 x 128 tile: 16-byte loads along the rows (256 contiguous bytes per row)
// into an LDS image, then four waves run the row part in the octet layout (a lane = one 16-element group
// of a row, 4 rows per lane) and four the column part in the quad layout (a lane quad = one 128-chunk of
// two columns), both reading the image.  LDS image: row r keeps its 4-byte word w (two bf16
// columns) at word w ^ (8 (r / 32)): the column part's 64 lanes (rows 32 q + i for q = 0..3,
// 16 consecutive words) then hit 32 different banks per half wave, and the row part's 32-byte
// groups stay contiguous (the xor only permutes whole groups).
#pragma once
#include "qii_device.h"
#include "qii_internal.h"
#include "quantize_core.h"
#include "quantize_lanes.h"

namespace qii {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct PairSide {
    uint32_t sign[4];      // the 128 rotation signs (host-side Philox), bit j of word j / 32
    uint64_t seed_sr;
    const float *amax;     // QII_MS_EDEN: max |rotated tensor| (device scalar)
    uint8_t *codes;
    uint8_t *scales;
    float *tensor_scale;
    float *tbuf;           // QII_MS_EDEN_PH: corrected pseudo-scales, one f32 per group
    uint32_t *amax_out;    // QII_MS_EDEN_PH: spread running maximum, or one word per block (nullable)
    int ksn;               // QII_MS_EDEN: 0, or the K tiles of the main GEMM kernel's layout, which the scale bytes then go out in
};

struct PairArgs {
    const uint16_t *x;
    int64_t ld;            // elements
    int64_t rows, cols;    // of x; both multiples of 128
    int tiles_x;           // tiles along a row of x
    int words;             // QII_MS_EDEN_PH: the maxima go to one word per block; QII_MS_EDEN and abs-max pass: see slot_max
    PairSide r, c;         // r: Q(x), rows x cols;  c: Q(x^T), cols x rows
};

constexpr uint32_t kNoStore = 0xFFFFFFF0u;   // a lane offset beyond every buffer descriptor: the store is dropped

__device__ __forceinline__ __amdgpu_buffer_rsrc_t region(const void *base, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}

// Eight waves: 0..3 take the rows, 4..7 the columns.  (Four waves that did the rows and then the columns left small
// tensors bound by that chain and large ones with too few waves in flight: whole post hoc calls 512 x 512 13.2 -> 11.2 us,
// 2048 x 2048 16.0 -> 13.9, 4096 x 4096 29.9 -> 26.8, 8192 x 4096 50.8 -> 48.9; Algorithm 1 17.2 -> 15.5, 20.5 -> 19.0,
// 46.1 -> 43.2, 69.4 -> 65.3.)
constexpr int kPairImage = 128 * 256;   // LDS bytes of the tile

// tile: kPairImage bytes of LDS; kMayTile: heeds ksn (false costs nothing where nobody asks for it); kWords: Algorithm 1's maxima are those
// of a.words words each (as a run-time question 0.7 % of a backward pass); kStream: the codes leave by non-temporal stores
// (launch_quantize_pair).  Args: by value, or by reference
// in a kernel that holds other arguments too (the addresses are then formed otherwise: 0.1 us of a small pair's call by reference,
// but 1 to 2 % of a backward pass by value)
template <int kMode, bool kMayTile, bool kWords, bool kStream, class Args = const PairArgs>
__device__ __forceinline__ void pair_block(Args a, int block, uint8_t *tile)
{
    __shared__ float inv_r[128], inv_c[128];
    __shared__ float wave_m[2][4];
    const int t = threadIdx.x, lane = t & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(t >> 6), wave = wave_id & 3;
    const bool take_rows = wave_id < 4;   // (wave-uniform)
    const int ty = block / a.tiles_x, tx = block - ty * a.tiles_x;
    const int64_t row0 = (int64_t)ty * 128, col0 = (int64_t)tx * 128;

    const int words = kMode == QII_MS_EDEN && kWords ? a.words : 0;
    const float word_r = slot_word(a.r.amax, words), word_c = slot_word(a.c.amax, words);

    // ---- the tile's loads first: 4 pieces of 16 bytes per thread, 16 threads per row
    u32x4 w[4];
    {
        const __amdgpu_buffer_rsrc_t src = region(a.x + row0 * a.ld + col0, (127 * a.ld + 128) * 2);
        const uint32_t voff = (uint32_t)(((t >> 4) * a.ld + (t & 15) * 8) * 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b128(src, voff, (int)(i * 32 * a.ld * 2), 0);
    }

    // ---- tensor constants and reciprocal tables of the two sides while the loads are in flight
    TensorConsts tcr = TensorConsts{}, tcc = TensorConsts{};
    if (kMode == QII_MS_EDEN) {
        tcr = tensor_consts(QII_MS_EDEN, slot_max(a.r.amax, words, word_r));
        tcc = tensor_consts(QII_MS_EDEN, slot_max(a.c.amax, words, word_c));
        if (block == 0 && t == 0) {
            *a.r.tensor_scale = tcr.x32;
            *a.c.tensor_scale = tcc.x32;
        }
        const uint32_t b = t & 127;
        const float x32 = t < 128 ? tcr.x32 : tcc.x32;
        if (t < 256) (t < 128 ? inv_r : inv_c)[b] = b == 0u ? 0.0f : 1.0f / (e4m3_decode(b) * x32);
    }

    // ---- LDS image (swizzled, see the file header)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = (t >> 4) + 32 * i, p = (t & 15) ^ (2 * (r >> 5));
        *reinterpret_cast<u32x4 *>(tile + r * 256 + p * 16) = w[i];
    }
    __syncthreads();

    float m_r = 0.0f, m_c = 0.0f;

    // ---- row part: Q(x).  quad = 4 consecutive rows of the tile (one draw call serves them);
    // the 8 lanes of an octet own the 8 groups of those rows inside the tile
    if (take_rows) {
        const OctetLane L = octet_lane(lane, a.r.sign);
        uint32_t mask[8];
        make_masks<true>(L.sign16, mask);
        const int quad = 8 * wave + (lane >> 3);
        const int64_t G = a.cols / 16, cpitch = a.cols / 2;
        uint32_t draw[4] = {0u, 0u, 0u, 0u};
        if (kMode == QII_MS_EDEN) {
            const U4 d = philox_seeded(a.r.seed_sr, (uint32_t)(tx * 8 + L.blk), (uint32_t)(ty * 32 + quad), 0, kStreamScale);
            draw[0] = d.x >> 12; draw[1] = d.y >> 12; draw[2] = d.z >> 12; draw[3] = d.w >> 12;
        }
        // this tile's part of the outputs: 64 code bytes, 8 scale bytes (or 8 f32) per row
        const __amdgpu_buffer_rsrc_t rc = region(a.r.codes + row0 * cpitch + col0 / 2, 127 * cpitch + 64);
        const int64_t ksn = kMayTile ? a.r.ksn : 0, spitch = ksn ? 16 : G;   // (uniform; a tile's rows lie in one tile of 256 rows of the tiled layout)
        const __amdgpu_buffer_rsrc_t rs = region(ksn ? tiled_scales(a.r.scales, ksn, row0, tx) : a.r.scales + row0 * G + col0 / 16, 127 * spitch + 8);
        const bool zero = kMode == QII_MS_EDEN && tcr.zero;   // uniform: an all-zero tensor is emitted as zero bytes
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int r = 4 * quad + it;   // (r / 32 == wave)
            const uint8_t *src = tile + r * 256 + ((L.blk ^ wave) * 32);
            const u32x4 q0 = *reinterpret_cast<const u32x4 *>(src), q1 = *reinterpret_cast<const u32x4 *>(src + 16);
            const uint32_t w8[8] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3]};
            float v[16];
            unpack_bf16x16<true>(w8, v, mask);
            rht128_lane(v, L);
            uint32_t packed[2];
            const uint32_t vc = (uint32_t)(r * cpitch) + 8u * L.blk;
            if (kMode == QII_MS_EDEN_PH) {
                float gmax;
                const float tt = posthoc_group16(v, packed, gmax);
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{packed[0], packed[1]}, rc, vc, 0, kStream ? 2 /* nt */ : 0);
                a.r.tbuf[(row0 + r) * G + col0 / 16 + L.blk] = tt;
                m_r = fmaxf(m_r, gmax);
                continue;
            }
            uint32_t b = quantize_group16<QII_MS_EDEN, -1, true>(v, tcr, draw[it], a.r.seed_sr, row0 + r, tx * 8 + L.blk, packed, inv_r);
            if (zero) { packed[0] = 0u; packed[1] = 0u; b = 0u; }
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{packed[0], packed[1]}, rc, vc, 0, kStream ? 2 /* nt */ : 0);
            const uint2 sc = gather_scale_bytes(b, L.blk);
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{sc.x, sc.y}, rs, L.blk == 0 ? (uint32_t)(r * spitch) : kNoStore, 0, 0);
        }
    }

    auto put_codes = [](uint8_t *dst, const uint32_t c[4]) {
        if (kStream) store_codes16(dst, c[0], c[1], c[2], c[3]);
        else *reinterpret_cast<uint4 *>(dst) = make_uint4(c[0], c[1], c[2], c[3]);
    };

    // ---- column part: Q(x^T).  The tile is chunk `ty` of the columns' 128-chunks; wave w takes the
    // tile's columns 32 w .. 32 w + 31, a lane quad two of them, lane q of the quad rows 32 q .. 32 q + 31
    if (!take_rows) {
        const int q = lane & 3, jp = lane >> 2;
        const uint8_t *src = tile + (32 * q) * 256 + 4 * ((16 * wave + jp) ^ (8 * q));
        uint32_t raw[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) raw[i] = *reinterpret_cast<const uint32_t *>(src + i * 256);
        const uint32_t sw = q == 0 ? a.c.sign[0] : q == 1 ? a.c.sign[1] : q == 2 ? a.c.sign[2] : a.c.sign[3];
        float v[2][32];
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const uint32_t flip = ((sw >> i) & 1u) << 31;
            v[0][i] = u2f((raw[i] << 16) ^ flip);
            v[1][i] = u2f((raw[i] & 0xFFFF0000u) ^ flip);
        }
        fwht128_quad(v[0], q);
        fwht128_quad(v[1], q);
        const int64_t chunk = ty, j0 = col0 + 32 * wave + 2 * jp;
        const int64_t G = a.rows / 16, cpitch = a.rows / 2;
        uint32_t draw[2][2] = {{0u, 0u}, {0u, 0u}};
        if (kMode == QII_MS_EDEN) octet_draws(draw, a.c.seed_sr, chunk, j0, q);
        const bool zero = kMode == QII_MS_EDEN && tcc.zero;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            uint32_t codes[4];
            if (kMode == QII_MS_EDEN_PH) {
                float tt[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float gmax;
                    tt[h] = posthoc_group16(v[e] + 16 * h, codes + 2 * h, gmax);
                    m_c = fmaxf(m_c, gmax);
                }
                put_codes(a.c.codes + (j0 + e) * cpitch + chunk * 64 + 16 * q, codes);
                *reinterpret_cast<float2 *>(a.c.tbuf + (j0 + e) * G + chunk * 8 + 2 * q) = make_float2(tt[0], tt[1]);
                continue;
            }
            uint32_t sc = 0u;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t b = quantize_group16<QII_MS_EDEN, -1, true>(v[e] + 16 * h, tcc, draw[e][h], a.c.seed_sr, j0 + e,
                                                                           chunk * 8 + 2 * q + h, codes + 2 * h, inv_c);
                sc |= b << (8 * h);
            }
            if (zero) { codes[0] = codes[1] = codes[2] = codes[3] = 0u; sc = 0u; }
            const uint2 s8 = gather_quad_scales(sc, q);
            put_codes(a.c.codes + (j0 + e) * cpitch + chunk * 64 + 16 * q, codes);
            if (q == 0) *reinterpret_cast<uint2 *>(kMayTile && a.c.ksn ? tiled_scales(a.c.scales, a.c.ksn, j0 + e, chunk) : a.c.scales + (j0 + e) * G + chunk * 8) = s8;
        }
    }

    // ---- post hoc scheme: the block's two maxima into the spread running maxima
    if (kMode == QII_MS_EDEN_PH && (a.r.amax_out || a.c.amax_out)) {   // uniform
        m_r = wave_max(m_r);
        m_c = wave_max(m_c);
        if (lane == 0) wave_m[take_rows ? 0 : 1][wave] = take_rows ? m_r : m_c;
        __syncthreads();
        if (t < 2) {
            uint32_t *out = t == 0 ? a.r.amax_out : a.c.amax_out;
            if (out) leave_block_max(fmaxf(fmaxf(wave_m[t][0], wave_m[t][1]), fmaxf(wave_m[t][2], wave_m[t][3])), out, a.words, block);
        }
    }
}

inline PairArgs pair_args(const PairQuantizeArgs &p)
{
    PairArgs a;
    a.x = reinterpret_cast<const uint16_t *>(p.src.x);
    a.ld = p.src.ld; a.rows = p.rows; a.cols = p.cols;
    a.tiles_x = (int)(p.cols / 128);
    a.words = p.amax_words;
    const PairQuantizeArgs::Side *in[2] = {&p.r, &p.c};
    PairSide *out[2] = {&a.r, &a.c};
    for (int i = 0; i < 2; ++i) {
        const U4 w = philox_seeded(in[i]->seed_rht, 0, 0, 0, kStreamRht);
        out[i]->sign[0] = w.x; out[i]->sign[1] = w.y; out[i]->sign[2] = w.z; out[i]->sign[3] = w.w;
        out[i]->seed_sr = in[i]->seed_sr;
        out[i]->amax = in[i]->amax;
        out[i]->codes = in[i]->codes; out[i]->scales = in[i]->scales; out[i]->tensor_scale = in[i]->tensor_scale;
        out[i]->tbuf = in[i]->tbuf; out[i]->amax_out = in[i]->amax_accum;
        out[i]->ksn = in[i]->tiled ? (int)((i == 0 ? p.cols : p.rows) / 256) : 0;
    }
    return a;
}

}  // namespace
}  // namespace qii
