// Tuned quantizer / abs-max kernels for dense row-major sources quantized along their rows
// (the contiguous case: Q(E), and the forward-pass RTN of X and W).
//
// Layout of the work: a lane owns one 16-element scale group, 8 lanes one 128-chunk, a wave
// 8 consecutive chunks of a row (1024 elements, 2 KiB of bf16) of one quad of 4 rows (one
// scale-rounding draw call serves the 4 rows of a group), or of one row of a small tensor; a block 4
// waves, side by side on a row or below one another (rows_wpr).  A wave's rows are requested together
// (32 B per lane and row) before anything else happens in the kernel.
// The octet register layout and its rotation are in quantize_lanes.h.
#include "qii_device.h"
#include "qii_internal.h"
#include "quantize_core.h"
#include "quantize_lanes.h"

namespace qii {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct RowsArgs {
    const void *x;
    int64_t ld;          // elements
    int64_t R, C;
    uint32_t sign[4];    // the 128 rotation signs (host-side Philox), bit j of word j/32
    uint64_t seed_sr;
    const float *amax;
    int n_amax;          // words at amax whose maximum is the tensor's: 1, or one per block of the pass that measured it
    uint8_t *codes;
    uint8_t *scales;
    float *tensor_scale;
    uint32_t *amax_out;  // abs-max kernel (one word, or one per block), and the heavy pass of the post hoc scheme
                         // (nullable there: the spread words, or, words != 0, one per block)
    int words;
    float *tbuf;         // post hoc scheme: corrected pseudo-scales [R][C/16]
    uint8_t *tiled;      // nullable: a second copy of the scale bytes, [row / 256][C / 256][row % 256][16]
    int wpr;             // waves of a block that sit side by side on a row: 1, 2 or 4
    int gy;              // blocks side by side on a row; the grid is one-dimensional, columns fastest
};

struct LaneSetup : OctetLane {
    int unit;             // this wave's rows: kRows unit .. kRows unit + kRows - 1; wave-uniform
    int64_t g;            // scale group within the row
    bool col_ok;
};

__device__ __forceinline__ LaneSetup lane_setup(const RowsArgs &a, int64_t G, int block)
{
    LaneSetup L;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, kept in a scalar register
    static_cast<OctetLane &>(L) = octet_lane(lane, a.sign);
    // wpr waves side by side, 4 / wpr waves below one another
    const int wcol = wave & (a.wpr - 1), wq = wave / a.wpr, upb = 4 / a.wpr;
    // consecutive blocks walk along a row first, then down the rows: blocks that run at the same
    // time read one contiguous region of the tensor
    const int bx = block / a.gy, by = block - bx * a.gy;
    L.unit = bx * upb + wq;
    const int64_t chunk = ((int64_t)by * a.wpr + wcol) * 8 + (lane >> 3);
    L.g = chunk * 8 + L.blk;
    L.col_ok = L.g < G;
    return L;
}

// raw row data of one lane: 16 elements
template <bool kBf16>
struct Raw {
    u32x4 q[kBf16 ? 2 : 4];
};

// All row addressing is wave-uniform (a wave works on whole rows): the row's base address sits
// in scalar registers inside a buffer descriptor that covers exactly the row's C elements, and a
// lane only contributes a 32-bit byte offset that never changes.  A row beyond the tensor gets an
// empty descriptor, a lane beyond the last column an offset beyond the descriptor: such loads
// return 0 and such stores are dropped by the hardware, so neither needs a branch or a mask.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void *base, int64_t row_bytes_offset, bool row_ok, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(base) + row_bytes_offset), 0,
                                             row_ok ? bytes : 0, 0x00020000);
}

constexpr uint32_t kNoStore = 0xFFFFFFF0u;   // a lane offset beyond every descriptor
// Cache policy of the code stores.  With rotation (the backward pass's quantizers) they are
// non-temporal: the lines do not linger dirty in L2, where the next kernel's traffic would have to
// push them out (-1 % and -3 % on the two 8192 x 8192 kernels, and the kernel that follows starts
// on a clean cache).  Without rotation (the forward pass) the GEMM reads the codes right away and
// ran 1.2 % slower when they had to come back from memory, so those stores stay ordinary.
template <bool kRht>
constexpr int code_store_policy() { return kRht ? 2 : 0; }

template <bool kBf16>
__device__ __forceinline__ void load_raw(Raw<kBf16> &r, const RowsArgs &a, int row, uint32_t voff)
{
    constexpr int n = kBf16 ? 2 : 4, esz = kBf16 ? 2 : 4;
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(a.x, (int64_t)row * a.ld * esz, row < (int)a.R, (int)(a.C * esz));
#pragma unroll
    for (int i = 0; i < n; ++i) r.q[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 16u * i, 0, 0);
}

template <bool kBf16, int kRows>
__device__ __forceinline__ void load_rows(Raw<kBf16> raw[kRows], const RowsArgs &a, int unit, uint32_t voff)
{
#pragma unroll
    for (int it = 0; it < kRows; ++it) load_raw<kBf16>(raw[it], a, unit * kRows + it, voff);
}

// widen to f32 and apply the rotation signs (sign masks are lane constants)
template <bool kBf16, bool kRht>
__device__ __forceinline__ void unpack_signed(const Raw<kBf16> &r, float v[16], const uint32_t mask[kBf16 ? 8 : 16])
{
    if (kBf16) {
        const uint32_t w[8] = {r.q[0][0], r.q[0][1], r.q[0][2], r.q[0][3], r.q[1][0], r.q[1][1], r.q[1][2], r.q[1][3]};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t s = kRht ? (w[i] ^ mask[i]) : w[i];
            v[2 * i] = bf16_lo(s);
            v[2 * i + 1] = bf16_hi(s);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * i + j] = u2f(kRht ? (r.q[i][j] ^ mask[4 * i + j]) : r.q[i][j]);
    }
}

// per-lane store offsets (bytes within a row of the output)
struct StoreOffsets {
    uint32_t codes;    // 8 bytes of codes per group
    uint32_t scale8;   // the gathered 8 scale bytes of a chunk: the lane holding block 0 stores them
    uint32_t scale1;   // one scale byte per lane (rows whose group count is not a multiple of 8)
    uint32_t t4;       // post hoc scheme: one f32 per group
    uint32_t tiled8;   // the chunk's 8 scale bytes within the tiled copy, relative to (row tile, row)
};

// A wave's rows (a quad or one) for one lane: their raw words are in registers (requested at the very
// start of the kernel).
template <bool kBf16, int kMode, bool kRht, int kFast, int kRows>
__device__ __forceinline__ void quantize_rows(const RowsArgs &a, const LaneSetup &L, const TensorConsts &tc,
                                              const uint32_t *mask, Raw<kBf16> raw[kRows], int64_t G,
                                              const StoreOffsets &so, float &m, const float *inv_tab)
{
    uint32_t draw[4] = {0u, 0u, 0u, 0u};
    if (kMode == QII_MS_EDEN) {
        const U4 w = philox_seeded(a.seed_sr, (uint32_t)L.g, (uint32_t)(L.unit * kRows / 4), 0, kStreamScale);
        draw[0] = w.x >> 12; draw[1] = w.y >> 12; draw[2] = w.z >> 12; draw[3] = w.w >> 12;
        if (kRows == 1) draw[0] = draw[L.unit & 3];   // (wave-uniform)
    }
#pragma unroll
    for (int it = 0; it < kRows; ++it) {
        const int row = L.unit * kRows + it;   // wave-uniform
        float v[16];
        unpack_signed<kBf16, kRht>(raw[it], v, mask);
        if (kRht) rht128_lane(v, L);
        const bool row_ok = row < (int)a.R;
        const __amdgpu_buffer_rsrc_t rc = row_rsrc(a.codes, (int64_t)row * (a.C / 2), row_ok, (int)(a.C / 2));
        uint32_t packed[2];
        if (kMode == QII_MS_EDEN_PH) {
            // heavy pass of the post hoc scheme: codes, corrected pseudo-scale, running maximum
            float gmax;
            const float t = posthoc_group16(v, packed, gmax);
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{packed[0], packed[1]}, rc, so.codes, 0, code_store_policy<kRht>());
            __builtin_amdgcn_raw_buffer_store_b32(f2u(t), row_rsrc(a.tbuf, (int64_t)row * G * 4, row_ok, (int)(G * 4)), so.t4, 0, 0);
            if (L.col_ok && row_ok) m = fmaxf(m, gmax);
            continue;
        }
        const uint32_t b = quantize_group16<kMode, kFast, true>(v, tc, draw[it], a.seed_sr, row, L.g, packed, inv_tab);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{packed[0], packed[1]}, rc, so.codes, 0, code_store_policy<kRht>());
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(a.scales, (int64_t)row * G, row_ok, (int)G);
        if (kRht || G % 8 == 0) {   // whole octets (always so with rotation): one 8-byte store per chunk
            const uint2 sc = gather_scale_bytes(b, L.blk);
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{sc.x, sc.y}, rs, so.scale8, 0, 0);
            if (!kRht && a.tiled) {   // uniform: the forward pass's copy for the GEMM (C a multiple of 256)
                const int64_t ksn = a.C / 256;
                const __amdgpu_buffer_rsrc_t rt = row_rsrc(a.tiled, ((int64_t)(row >> 8) * ksn * 256 + (row & 255)) * 16, row_ok,
                                                           (int)(ksn * 4096 - (row & 255) * 16));
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{sc.x, sc.y}, rt, so.tiled8, 0, 0);
            }
        } else {
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)b, rs, so.scale1, 0, 0);
        }
    }
}

// The tensor's maximum: one word, or (forward pass) the maximum of the words that the blocks of the abs-max
// pass left, reduced by every block.  The words are requested before the block's rows, so that the reduction
// does not wait for those (loads return in order: requested after the rows, 16384 x 3072 f32 with 4/6 took 50.6 us
// instead of 38.4, 16384 x 2048 and 8192 x 2048 bf16 32.7 instead of 28.5).  All threads of the block must call both.
static_assert(kForwardMaxWords <= 1024, "four words per thread");

__device__ __forceinline__ void request_words(const RowsArgs &a, float w[4])
{
    if (a.n_amax > 1) {   // uniform; (a thread beyond the last word takes that one again)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = (int)threadIdx.x + 256 * k;
            w[k] = a.amax[i < a.n_amax ? i : a.n_amax - 1];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ float reduce_words(const RowsArgs &a, const float w[4], float *wave_m)
{
    if (a.n_amax == 1) return *a.amax;   // uniform
    const float m = wave_max(fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3])));
    if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = m;
    __syncthreads();
    return fmaxf(fmaxf(wave_m[0], wave_m[1]), fmaxf(wave_m[2], wave_m[3]));
}

constexpr int kMeasuringWaves = 16;   // of a block that measures its tensor

// A small dense tensor's maximum, measured by every block of kMeasuringWaves waves for itself: contiguous 16-byte pieces, eight
// in flight per thread (beyond the tensor they read as zeros).
template <bool kBf16>
__device__ __forceinline__ float measure_tensor(const RowsArgs &a, float *wave_m)
{
    constexpr int kAtOnce = 8, kStep = kMeasuringWaves * 64 * 16;
    const int bytes = (int)(a.R * a.C * (kBf16 ? 2 : 4));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, bytes, 0x00020000);
    float m = 0.0f;
    for (int base = 0; base < bytes; base += kAtOnce * kStep) {
        u32x4 w[kAtOnce];
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, base + i * kStep + (int)threadIdx.x * 16, 0, 0);
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (kBf16) m = fmaxf(fmaxf(m, fabsf(bf16_lo(w[i][j]))), fabsf(bf16_hi(w[i][j])));
                else m = fmaxf(m, fabsf(u2f(w[i][j])));
            }
    }
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = m;
    __syncthreads();
    m = wave_m[0];
#pragma unroll
    for (int i = 1; i < kMeasuringWaves; ++i) m = fmaxf(m, wave_m[i]);
    return m;
}

// One wave = a quad of rows, or one row of a small tensor (kRows), x 1024 columns; one block = 4 such pieces (a measuring block
// has 12 waves more, without rows); the grid covers the tensor.
// Blocks are short-lived on purpose: many independent blocks that start and finish at different
// times keep the memory traffic of the chip smooth, where long-lived waves marching in step (a
// grid-stride loop with prefetch was measured) load and compute in bursts and ran 10 % slower.
// kMax: the tensor's maximum is one word, or may be that of several, or every block measures it (a small tensor).
enum MaxFrom { kOneWord, kWords, kMeasured };

template <bool kBf16, int kMode, bool kRht, MaxFrom kMax, int kRows>
__device__ __forceinline__ void quantize_rows_body(const RowsArgs &a, int block)
{
    __shared__ float inv_tab[128];
    __shared__ float wave_m[kMax == kMeasured ? kMeasuringWaves : 4];
    constexpr int esz = kBf16 ? 2 : 4;
    const int64_t G = a.C / 16;
    // (the waves beyond the fourth of a measuring block have no rows: they load nothing and end once the maximum is known)
    const bool has_rows = kMax != kMeasured || threadIdx.x < 256;   // wave-uniform
    LaneSetup L = lane_setup(a, G, block);
    if (!has_rows) L.unit = (int)(a.R + 1);
    // the rows are requested before anything else: the loads do not depend on the tensor
    // constants, whose set-up (a dependent load, divisions, the table) then overlaps them
    const uint32_t voff = (uint32_t)L.g * (16u * esz);   // (beyond the row for lanes beyond the last column)
    float words[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (kMax == kWords) request_words(a, words);
    else if (kMax == kOneWord && kMode != QII_MS_EDEN_PH) words[0] = slot_word(a.amax, a.words);
    Raw<kBf16> raw[kRows];
    load_rows<kBf16, kRows>(raw, a, L.unit, voff);
    // (the heavy pass of the post hoc scheme knows no tensor maximum: tc stays unused there)
    const TensorConsts tc = kMode == QII_MS_EDEN_PH ? TensorConsts{}
                                                    : tensor_consts(kMode, kMax == kMeasured ? measure_tensor<kBf16>(a, wave_m)
                                                                           : kMax == kWords  ? reduce_words(a, words, wave_m) : slot_max(a.amax, a.words, words[0]));
    if (!has_rows) return;   // (a wave that has ended takes no part in barriers)
    if (kMode != QII_MS_EDEN_PH && block == 0 && threadIdx.x == 0) *a.tensor_scale = tc.x32;
    StoreOffsets so;
    so.codes = L.col_ok ? (uint32_t)L.g * 8u : kNoStore;
    so.scale8 = (L.col_ok && L.blk == 0) ? (uint32_t)L.g : kNoStore;
    so.scale1 = L.col_ok ? (uint32_t)L.g : kNoStore;
    so.t4 = L.col_ok ? (uint32_t)L.g * 4u : kNoStore;
    so.tiled8 = (L.col_ok && L.blk == 0) ? (uint32_t)(L.g >> 4) * 4096u + (uint32_t)((L.g >> 3) & 1) * 8u : kNoStore;
    if (tc.zero) {  // uniform: an all-zero tensor is emitted as zero bytes
        for (int it = 0; it < kRows; ++it) {
            const int64_t row = (int64_t)L.unit * kRows + it;
            if (L.col_ok && row < a.R) {
                *reinterpret_cast<uint2 *>(a.codes + (row * a.C + L.g * 16) / 2) = make_uint2(0u, 0u);
                a.scales[row * G + L.g] = 0;
                if (!kRht && a.tiled) a.tiled[(((row >> 8) * (a.C / 256) + (L.g >> 4)) * 256 + (row & 255)) * 16 + (L.g & 15)] = 0;
            }
        }
        return;
    }
    if (kMode != QII_MS_EDEN_PH) fill_inv_table(inv_tab, tc);
    uint32_t mask[kBf16 ? 8 : 16];
    make_masks<kBf16>(L.sign16, mask);
    float m = 0.0f;
    if (kMode == QII_MS_EDEN_PH || tc.fast)   // uniform: one branch for the whole kernel
        quantize_rows<kBf16, kMode, kRht, 1, kRows>(a, L, tc, mask, raw, G, so, m, inv_tab);
    else
        quantize_rows<kBf16, kMode, kRht, 0, kRows>(a, L, tc, mask, raw, G, so, m, inv_tab);
    if (kMode == QII_MS_EDEN_PH && a.amax_out) {   // uniform: one update per block, spread over the slot's words
        m = wave_max(m);
        if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = m;
        __syncthreads();
        if (threadIdx.x == 0)
            leave_block_max(fmaxf(fmaxf(wave_m[0], wave_m[1]), fmaxf(wave_m[2], wave_m[3])), a.amax_out, a.words, block);
    }
}

template <bool kBf16, int kMode, bool kRht, int kRows>
__global__ __launch_bounds__(256) void quantize_rows_kernel(RowsArgs a)
{
    quantize_rows_body<kBf16, kMode, kRht, kOneWord, kRows>(a, (int)blockIdx.x);
}

// X and W of a forward pass in one launch: the first n0 blocks take a0
template <bool kBf16, int kMode, int kRows>
__global__ __launch_bounds__(256) void quantize_rows2_kernel(RowsArgs a0, RowsArgs a1, int n0)
{
    const bool first = (int)blockIdx.x < n0;   // uniform
    RowsArgs a = a0;
    if (!first) a = a1;
    quantize_rows_body<kBf16, kMode, false, kWords, kRows>(a, (int)blockIdx.x - (first ? 0 : n0));
}

// The same for small tensors whose maxima are not supplied, one or two of them: every block measures its tensor.
template <bool kBf16, int kMode>
__global__ __launch_bounds__(64 * kMeasuringWaves) void quantize_small_rows_kernel(RowsArgs a0, RowsArgs a1, int n0)
{
    const bool first = (int)blockIdx.x < n0;   // uniform
    RowsArgs a = a0;
    if (!first) a = a1;
    quantize_rows_body<kBf16, kMode, false, kMeasured, 1>(a, (int)blockIdx.x - (first ? 0 : n0));
}

// Abs-max pass.  Its result is one word that every block has to fold its maximum into, and such
// device-wide atomics on one address are resolved one after the other (about 10 ns each), so this
// kernel runs as few, long-lived blocks (two per compute unit) that stride over the row quads with
// the next quad's loads in flight, and issue one atomic each at the very end.
template <bool kBf16, bool kRht>
__device__ __forceinline__ float absmax_rows_body(const RowsArgs &a, int block, int blocks)
{
    constexpr int esz = kBf16 ? 2 : 4;
    __shared__ float wave_m[4];
    const int64_t G = a.C / 16;
    const LaneSetup L = lane_setup(a, G, block);
    const int quads = (int)((a.R + 3) / 4);
    const int step = (blocks / a.gy) * (4 / a.wpr);
    const uint32_t voff = (uint32_t)L.g * (16u * esz);
    uint32_t mask[kBf16 ? 8 : 16];
    make_masks<kBf16>(L.sign16, mask);
    float m = 0.0f;
    Raw<kBf16> raw[4];
    load_rows<kBf16, 4>(raw, a, L.unit, voff);   // (rows and columns beyond the tensor read as 0 and cannot change the maximum)
    for (int quad = L.unit; quad < quads; quad += step) {
        Raw<kBf16> nxt[4];
        load_rows<kBf16, 4>(nxt, a, quad + step, voff);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            float v[16];
            unpack_signed<kBf16, kRht>(raw[it], v, mask);
            if (kRht) rht128_lane<false>(v, L);
            m = fmaxf(m, group_absmax(v));
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) raw[it] = nxt[it];
    }
    if (kRht) m = __builtin_fmaf(m, kInvSqrt128, 0.0f);   // the scaling the rotation left out
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = m;
    __syncthreads();
    return fmaxf(fmaxf(wave_m[0], wave_m[1]), fmaxf(wave_m[2], wave_m[3]));
}

template <bool kBf16, bool kRht>
__global__ __launch_bounds__(256) void absmax_rows_kernel(RowsArgs a)
{
    const float m = absmax_rows_body<kBf16, kRht>(a, (int)blockIdx.x, (int)gridDim.x);
    if (threadIdx.x == 0) {
        if (a.words) a.amax_out[blockIdx.x] = f2u(m);
        else max_to_global(m, a.amax_out);
    }
}

// X and W of a forward pass in one launch: the first n0 blocks take a0.  The result stays inside the
// library, so every block leaves its maximum in a word of its own and the quantizer's blocks reduce
// the words: no clearing launch before, no atomics.
template <bool kBf16>
__global__ __launch_bounds__(256) void absmax_rows2_kernel(RowsArgs a0, RowsArgs a1, int n0)
{
    const bool first = (int)blockIdx.x < n0;   // uniform
    RowsArgs a = a0;
    if (!first) a = a1;
    const int block = (int)blockIdx.x - (first ? 0 : n0), blocks = first ? n0 : (int)gridDim.x - n0;
    const float m = absmax_rows_body<kBf16, false>(a, block, blocks);
    if (threadIdx.x == 0) a.amax_out[block] = f2u(m);
}


// Waves of a block side by side on a row (a wave takes 8 chunks of 128).  Those beyond the row's end run the arithmetic
// all the same, so a block's waves are as many as divide the row's: 4, 2 or 1.  Measured, whole calls, us, waves of a block
// 1 : 2 : 4 (abs-max pass as below):
//   5 waves   8192 x 4112 f32 SR 65.1 : 68.1 : 76.7, bf16 RTN 32.7 : 31.6 : 35.0; 2048 x 5120 f32 SR 26.3 : 25.8 : 28.7
//   6 waves   8192 x 5632 f32 SR 79.5 : 78.0 : 89.2, bf16 MS-EDEN 46.3 : 46.1 : 52.1; 2048 x 5632 f32 SR 26.5 : 26.8 : 29.2
//   7 waves   8192 x 7168 f32 SR 93.2 : 96.6 : 97.1, bf16 MS-EDEN 54.2 : 55.9 : 56.1
//   4, 8      8192 x 8192 bf16 MS-EDEN 61.7 : 60.1 : 59.4, 1024 x 4096 bf16 forward pass 29.3 : 28.5 : 28.1
//   3 waves   8192 x 2560 f32 SR 42.3 : 47.8 : 46.6, bf16 MS-EDEN 29.8 : 32.6 : 31.6; but in fours where the last chunk is a partial
//             one (8192 x 2064 bf16 RTN 20.2 : 21.8 : 19.3) or rows are few (2048 x 3072 bf16 forward pass 32.7 : 32.2 : 32.0)
int rows_waves(int64_t C) { return (int)(((C / 16 + 7) / 8 + 7) / 8); }

int rows_wpr(int64_t R, int64_t C)
{
    const int waves = rows_waves(C);
    if (waves == 3 && (C % 128 != 0 || R < 4096)) return 4;
    return waves % 4 == 0 ? 4 : waves % 2 == 0 ? 2 : 1;
}

// blocks side by side on a row
int64_t rows_gy(int64_t C, int wpr) { return ((C / 16 + 7) / 8 + 8 * wpr - 1) / (8 * wpr); }

// The abs-max passes: as many as the row needs, at most 4, but 2 where fours would leave some beyond the end of 5 waves or
// more (2 : 4, quantizer as above: 8192 x 4112 bf16 RTN 32.7 : 35.2, 8192 x 5632 bf16 MS-EDEN 46.1 : 47.1, f32 SR 78.0 : 80.0; one
// wave a block would leave every other one of a 1040-wide tensor's idle, and with it half of the dies).
int absmax_wpr(int64_t C)
{
    const int waves = rows_waves(C);
    return waves >= 5 && waves % 4 != 0 ? 2 : waves >= 3 ? 4 : waves;
}

// one wave per `rows` rows (4, or 1: rows_per_wave) x 1024 columns; max_block_rows > 0 caps the number of blocks below one
// another (the abs-max pass then strides over the rest)
dim3 rows_grid(int64_t R, int64_t C, int wpr, int64_t max_block_rows, int rows = 4)
{
    const int64_t gy = rows_gy(C, wpr);
    const int64_t units = (R + rows - 1) / rows, upb = 4 / wpr;
    int64_t gx = (units + upb - 1) / upb;
    if (max_block_rows > 0 && gx > max_block_rows) {
        const int64_t iters = (gx + max_block_rows - 1) / max_block_rows;
        gx = (gx + iters - 1) / iters;   // even split
    }
    return dim3((unsigned)((gx < 1 ? 1 : gx) * gy), 1u);
}

RowsArgs make_args(const Source &src, int64_t R, int64_t C, uint64_t seed_rht, uint64_t seed_sr, int wpr)
{
    RowsArgs a;
    a.x = src.x; a.ld = src.ld; a.R = R; a.C = C;
    const U4 w = philox_seeded(seed_rht, 0, 0, 0, kStreamRht);
    a.sign[0] = w.x; a.sign[1] = w.y; a.sign[2] = w.z; a.sign[3] = w.w;
    a.seed_sr = seed_sr;
    a.amax = nullptr; a.n_amax = 1; a.codes = nullptr; a.scales = nullptr; a.tensor_scale = nullptr; a.amax_out = nullptr;
    a.tbuf = nullptr;
    a.words = 0;
    a.tiled = nullptr;
    a.wpr = wpr;
    a.gy = (int)rows_gy(C, wpr);
    return a;
}

}  // namespace

// Rows of a quantizer's wave: a quad, whose rows share a scale-rounding draw call, or one where quads leave the GPU's 1024
// vector units short of waves, each of which then works its four rows off one after the other.  Whole calls, us, quads : rows
// (`waves`: those that quads make):
//   64 waves     256 x  256 f32 RTN 8.6 : 7.6, 4/6 9.7 : 7.9, SR 10.6 : 8.2, MS-EDEN 11.0 : 9.0, post hoc 9.9 : 7.8
//   256 waves   1024 x 1024 bf16 RTN 8.5 : 7.6, 4/6 9.7 : 8.1, SR 10.7 : 8.3, MS-EDEN 10.9 : 9.1, post hoc 10.4 : 8.4
//   512 waves   2048 x 1024 bf16 RTN 9.3 : 8.5, MS-EDEN 11.7 : 10.3, post hoc 10.5 : 9.2; f32 RTN 10.1 : 10.2
//   1024 waves  2048 x 2048 bf16 RTN 10.8 : 11.3, MS-EDEN 13.0 : 14.0, post hoc 11.0 : 11.3; f32 12.1 : 12.8, 15.2 : 15.0
//   2048 waves  4096 x 2048 f32 RTN 18.1 : 20.0, bf16 post hoc 13.7 : 14.5
// 4/6 has twice the arithmetic per row and gains a little longer (forward passes, both tensors' waves: 1280 26.8 : 25.2,
// 2048 31.8 : 31.4, 4096 46.2 : 46.1).  The post hoc scheme's heavy pass gains less long (no abs-max pass before it leaves the tensor
// in cache, and its blocks each leave a word for the scales pass), and what counts are the waves launched, with those beyond
// the row's end (rows of three waves go in fours).  bf16, by launched waves:
//   680 511 x 2304 10.2 : 9.6, 768 3071 x 1024 10.5 : 10.0, 852 851 x 2304 10.3 : 10.5, 896 3583 x 1024 10.6 : 10.8,
//   1192 1191 x 2560 12.0 : 12.5 (where blocks of single rows are too many for a word each)
int rows_per_wave(int64_t R, int64_t C, int mode)
{
    const int64_t quads = (R + 3) / 4;
    if (mode == QII_MS_EDEN_PH) {
        const int wpr = rows_wpr(R, C);
        return quads * rows_gy(C, wpr) * wpr < 840 ? 1 : 4;
    }
    return quads * rows_waves(C) < (mode == QII_RTN_46 ? 2048 : 1024) ? 1 : 4;
}

// (a row of the source and of every output is addressed through a 32-bit buffer descriptor)
bool rows_kernels_apply(const Source &src, int64_t R, int64_t C)
{
    return !src.transpose && (src.kind == kSrcBF16 || src.kind == kSrcF32) && C <= ((int64_t)1 << 28) &&
           R < ((int64_t)1 << 31) - 8;   // row indices are 32-bit in the kernels
}

// A tensor so small that the blocks of its quantizer had better measure it themselves (from L2, all of it, each) than
// wait for an abs-max launch, and in a call of its own for a clearing launch too.  Whole calls, us, abs-max launch : measured by
// every block (one row per wave in both): 128 x 128 f32 RTN 7.5 : 4.4, SR 8.0 : 5.0; 256 x 256 f32 RTN 7.6 : 5.4, forward pass
// 10.6 : 9.8, bf16 10.3 : 8.8; 256 x 512 bf16 RTN 7.2 : 5.5, forward pass 11.0 : 10.6, f32 7.7 : 7.2, forward pass 11.4 : 12.4;
// 512 x 512 bf16 RTN 7.4 : 7.6.  Rows add blocks, each of which reads everything: 2048 x 128 bf16 RTN 8.4 : 14.6.
constexpr int64_t kMeasuredBytes = 256 * 1024, kMeasuredRows = 512;

bool measures_itself(const QuantizeArgs &q)
{
    return q.rht == 0 && (q.mode == QII_RTN || q.mode == QII_RTN_46 || q.mode == QII_SR) && q.src.ld == q.C && rows_kernels_apply(q.src, q.R, q.C) &&
           q.R <= kMeasuredRows &&
           q.R * q.C * (q.src.kind == kSrcBF16 ? 2 : 4) <= kMeasuredBytes;
}

// a: make_args and the outputs of q, one or two tensors of one mode and type
static hipError_t launch_small_rows(const RowsArgs *a, const QuantizeArgs *q, int count, hipStream_t s)
{
    int n[2] = {0, 0};
    for (int i = 0; i < count; ++i) n[i] = (int)rows_grid(q[i].R, q[i].C, a[i].wpr, 0, 1).x;
    const dim3 grid((unsigned)(n[0] + n[1])), block(64 * kMeasuringWaves);
    const bool bf = q[0].src.kind == kSrcBF16;
#define QII_SMALL(MODE)                                                                                                              \
    do {                                                                                                                             \
        if (bf) hipLaunchKernelGGL((quantize_small_rows_kernel<true, MODE>), grid, block, 0, s, a[0], a[count - 1], n[0]);            \
        else hipLaunchKernelGGL((quantize_small_rows_kernel<false, MODE>), grid, block, 0, s, a[0], a[count - 1], n[0]);              \
    } while (0)
    if (q[0].mode == QII_RTN) QII_SMALL(QII_RTN);
    else if (q[0].mode == QII_SR) QII_SMALL(QII_SR);
    else QII_SMALL(QII_RTN_46);
#undef QII_SMALL
    return hipGetLastError();
}

// the launch below: at most two blocks per compute unit
static dim3 absmax_rows_grid(int64_t R, int64_t C, int words)
{
    const int wpr = absmax_wpr(C);
    const int64_t gy = rows_gy(C, wpr), most = (words ? kSlotWords : 512) / gy;
    return rows_grid(R, C, wpr, most > 0 ? most : 1);
}

// A word per block, at most kSlotWords blocks, and no clearing launch, where the few blocks' longer way through the tensor costs less:
// what counts are the rounds, row quads that a wave takes one after the other, whose loads and rotation wait for one another (narrow
// rows fill their waves with as many quads as wide ones).  Whole calls, us, clearing and atomics : words, medians over 3500 tensors of up to 4 M
// elements.  Rotated, by rounds: 1 9.0 : 7.3, 2 10.1 : 9.0, 3 11.5 : 11.2, 4 in 56 blocks and more 13.4 : 13.3, in fewer 12.6 : 13.0, 5 15.4 :
// 15.9, 6 17.0 : 18.4; 20480 x 128 bf16 MS-EDEN 22.4 : 37.7, 16384 x 256 f32 20.0 : 31.2.  (f32 rows of 7 or 15 waves: four or eight blocks side by
// side, so that the idle waves of the last are all on the same dies: the fourth round costs 1.3 more.)  Unrotated bf16: 4 10.5 : 8.3, 8 14.4 : 11.6,
// 14 19.0 : 18.3, 21 20.6 : 21.3, 24 23.2 : 25.7; f32, whose bytes count as well: 5 and 6 up to 8 MiB 13.4 : 10.5, above 13.1 : 12.2, 7 to 10 up to 8 MiB
// 14.5 : 12.4, above 13.5 : 13.9, 13 up to 2 MiB 16.6 : 15.8, above 15.6 : 17.7.
int absmax_rows_words(const Source &src, int64_t R, int64_t C, int rht)
{
    const int wpr = absmax_wpr(C);
    const int64_t gy = rows_gy(C, wpr), elements = R * C;
    if (elements > (int64_t)4 << 20 || gy > kSlotWords) return 0;
    const int64_t block_rows = rows_grid(R, C, wpr, 0).x / gy, most = kSlotWords / gy, rounds = (block_rows + most - 1) / most;
    const int blocks = (int)absmax_rows_grid(R, C, 1).x;
    const bool bf16 = src.kind == kSrcBF16;
    const bool pays = rht    ? rounds <= 3 || (rounds == 4 && blocks >= 56 && (bf16 || rows_waves(C) % 8 != 7))
                      : bf16 ? rounds <= 19
                             : rounds <= 6 || (rounds <= 10 && elements <= (int64_t)2 << 20) || (rounds <= 13 && elements <= (int64_t)1 << 19);
    return pays ? blocks : 0;
}

hipError_t launch_absmax_rows(const Source &src, int64_t R, int64_t C, int rht, uint64_t seed_rht,
                              float *amax, hipStream_t s, int words)
{
    RowsArgs a = make_args(src, R, C, seed_rht, 0, absmax_wpr(C));
    a.amax_out = reinterpret_cast<uint32_t *>(amax);
    a.words = words;
    const dim3 grid = absmax_rows_grid(R, C, words), block(256);
    const bool bf = src.kind == kSrcBF16;
    if (bf) { if (rht) hipLaunchKernelGGL((absmax_rows_kernel<true, true>), grid, block, 0, s, a); else hipLaunchKernelGGL((absmax_rows_kernel<true, false>), grid, block, 0, s, a); }
    else { if (rht) hipLaunchKernelGGL((absmax_rows_kernel<false, true>), grid, block, 0, s, a); else hipLaunchKernelGGL((absmax_rows_kernel<false, false>), grid, block, 0, s, a); }
    return hipGetLastError();
}

hipError_t launch_quantize_rows(const QuantizeArgs &q, hipStream_t s)
{
    RowsArgs a = make_args(q.src, q.R, q.C, q.seed_rht, q.seed_sr, rows_wpr(q.R, q.C));
    a.amax = q.amax; a.codes = q.codes; a.scales = q.scales; a.tensor_scale = q.tensor_scale;
    a.tbuf = q.tbuf; a.amax_out = q.amax_accum; a.words = q.amax_words;
    if (q.scales_tiled) {
        if (q.rht || q.C % 256 != 0 || q.mode == QII_MS_EDEN_PH) return hipErrorInvalidValue;
        a.tiled = q.scales_tiled;
    }
    const int rows = rows_per_wave(q.R, q.C, q.mode);
    const dim3 grid = rows_grid(q.R, q.C, a.wpr, 0, rows), block(256);
    const bool bf = q.src.kind == kSrcBF16;
#define QII_ROWS(BF, MODE, RHT)                                                                          \
    do {                                                                                                 \
        if (rows == 1) hipLaunchKernelGGL((quantize_rows_kernel<BF, MODE, RHT, 1>), grid, block, 0, s, a); \
        else hipLaunchKernelGGL((quantize_rows_kernel<BF, MODE, RHT, 4>), grid, block, 0, s, a);          \
    } while (0)
#define QII_ROWS_MODE(BF, RHT)                                   \
    do {                                                         \
        if (q.mode == QII_RTN) QII_ROWS(BF, QII_RTN, RHT);       \
        else if (q.mode == QII_SR) QII_ROWS(BF, QII_SR, RHT);    \
        else if (q.mode == QII_RTN_46) QII_ROWS(BF, QII_RTN_46, RHT); \
        else if (q.mode == QII_MS_EDEN_PH) QII_ROWS(BF, QII_MS_EDEN_PH, RHT); \
        else QII_ROWS(BF, QII_MS_EDEN, RHT);                     \
    } while (0)
    if (bf) { if (q.rht) QII_ROWS_MODE(true, true); else QII_ROWS_MODE(true, false); }
    else { if (q.rht) QII_ROWS_MODE(false, true); else QII_ROWS_MODE(false, false); }
#undef QII_ROWS_MODE
#undef QII_ROWS
    return hipGetLastError();
}

hipError_t launch_quantize_small(const QuantizeArgs &q, hipStream_t s)
{
    RowsArgs a = make_args(q.src, q.R, q.C, 0, q.seed_sr, rows_wpr(q.R, q.C));
    a.codes = q.codes; a.scales = q.scales; a.tensor_scale = q.tensor_scale; a.tiled = q.scales_tiled;
    if (a.tiled && q.C % 256 != 0) return hipErrorInvalidValue;
    return launch_small_rows(&a, &q, 1, s);
}

int rows_blocks(int64_t R, int64_t C) { return (int)rows_grid(R, C, rows_wpr(R, C), 0, rows_per_wave(R, C, QII_MS_EDEN_PH)).x; }

// Forward pass: Q(X) and Q(W), no rotation, RTN or RTN with 4/6.  Where a maximum is not supplied it is measured
// first: about kForwardMaxWords blocks in all, shared out by the tensors' sizes, leave one word each (rows longer than 4096
// elements take whole rows of blocks, so that both tensors together can have more; each has at most kForwardMaxWords).
hipError_t launch_forward_quantize(const QuantizeArgs q[2], float *words, hipStream_t s)
{
    RowsArgs a[2], m[2];   // of the quantize and of the abs-max launch
    int64_t size[2];
    for (int i = 0; i < 2; ++i) {
        a[i] = make_args(q[i].src, q[i].R, q[i].C, 0, 0, rows_wpr(q[i].R, q[i].C));
        m[i] = make_args(q[i].src, q[i].R, q[i].C, 0, 0, absmax_wpr(q[i].C));
        a[i].amax = q[i].amax;
        a[i].codes = q[i].codes; a[i].scales = q[i].scales; a[i].tensor_scale = q[i].tensor_scale;
        a[i].tiled = q[i].scales_tiled;
        if (a[i].tiled && q[i].C % 256 != 0) return hipErrorInvalidValue;
        size[i] = q[i].amax ? 0 : q[i].R * q[i].C;
    }
    const bool bf = q[0].src.kind == kSrcBF16;
    const dim3 block(256);
    if (!q[0].amax && !q[1].amax && measures_itself(q[0]) && measures_itself(q[1])) return launch_small_rows(a, q, 2, s);
    if (size[0] + size[1] > 0) {
        int n[2] = {0, 0};
        for (int i = 0; i < 2; ++i) {
            if (size[i] == 0) continue;
            int64_t share = (int64_t)((double)kForwardMaxWords * (double)size[i] / (double)(size[0] + size[1])) / m[i].gy;
            if (share * m[i].gy > kForwardMaxWords - 64) share = (kForwardMaxWords - 64) / m[i].gy;   // (the other tensor has room)
            if (share < 1) share = 1;
            n[i] = (int)rows_grid(q[i].R, q[i].C, m[i].wpr, share).x;
            if (n[i] > kForwardMaxWords) return hipErrorInvalidValue;   // (see forward_quantize_applies)
            m[i].amax_out = reinterpret_cast<uint32_t *>(words + i * kForwardMaxWords);
            a[i].amax = words + i * kForwardMaxWords;
            a[i].n_amax = n[i];
        }
        const dim3 grid((unsigned)(n[0] + n[1]));
        if (bf) hipLaunchKernelGGL((absmax_rows2_kernel<true>), grid, block, 0, s, m[0], m[1], n[0]);
        else hipLaunchKernelGGL((absmax_rows2_kernel<false>), grid, block, 0, s, m[0], m[1], n[0]);
    }
    const int rows = rows_per_wave(q[0].R + q[1].R, q[0].C, q[0].mode);
    const int n0 = (int)rows_grid(q[0].R, q[0].C, a[0].wpr, 0, rows).x;
    const dim3 grid((unsigned)n0 + rows_grid(q[1].R, q[1].C, a[1].wpr, 0, rows).x);
#define QII_FWD(BF, MODE)                                                                                          \
    do {                                                                                                           \
        if (rows == 1) hipLaunchKernelGGL((quantize_rows2_kernel<BF, MODE, 1>), grid, block, 0, s, a[0], a[1], n0); \
        else hipLaunchKernelGGL((quantize_rows2_kernel<BF, MODE, 4>), grid, block, 0, s, a[0], a[1], n0);           \
    } while (0)
    if (q[0].mode == QII_RTN) { if (bf) QII_FWD(true, QII_RTN); else QII_FWD(false, QII_RTN); }
    else { if (bf) QII_FWD(true, QII_RTN_46); else QII_FWD(false, QII_RTN_46); }
#undef QII_FWD
    return hipGetLastError();
}

// both tensors by the rows kernels, a row within what one row of abs-max blocks covers, grids that fit
bool forward_quantize_applies(const Source &x, int64_t T, const Source &w, int64_t d_out, int64_t d_in)
{
    return T > 0 && d_out > 0 && d_in > 0 && rows_kernels_apply(x, T, d_in) && rows_kernels_apply(w, d_out, d_in) &&
           d_in <= (int64_t)4096 * (kForwardMaxWords / 2) && ((T + d_out) / 4 + 2) * ((d_in + 4095) / 4096) < ((int64_t)1 << 30);
}

}  // namespace qii
