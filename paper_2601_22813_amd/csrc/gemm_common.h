// Pieces shared by the GEMM kernels of libqii: vector types, the in-register dequantization of a
// fragment, and the epilogue that stages a wave's accumulator tile through LDS and stores full rows
// (optionally emitting max |C|).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qii_device.h"

namespace qii {
namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Launch position -> tile coordinates.  XCD-aware order: consecutive block ids land on different XCDs (8
// of them, each with its own L2), so every XCD gets a contiguous run of tiles; within the run, tiles are
// walked in groups of 4 tile rows, column by column, so that the tiles an XCD works on at once share
// few operand panels.
__device__ __forceinline__ void tile_coords(int pos, int tiles_m, int tiles_n, int &tm, int &tn)
{
    int tile = pos;
    const int ntiles = tiles_m * tiles_n;
    if ((ntiles & 7) == 0) tile = (tile & 7) * (ntiles >> 3) + (tile >> 3);
    constexpr int kGroupM = 4;
    const int width = kGroupM * tiles_n, first_m = (tile / width) * kGroupM;
    const int gm = tiles_m - first_m < kGroupM ? tiles_m - first_m : kGroupM;
    tm = first_m + (tile % width) % gm;
    tn = (tile % width) / gm;
}

// Optional by-product of the epilogue: max |C| over the stored values, for a consumer that
// quantizes C next and would otherwise have to read it once more just for its abs-max (the
// paper's layer timings assume the abs-max comes from the producing kernel, App. D).  Atomics on
// one word are resolved one after the other, so a block combines its waves first and leaves
// the word alone where it already holds as much (20000 x 3000 x 112 in 128 x 128 tiles: 90 us without
// the maximum, 97 with it; one atomic per wave 196).  All threads of the block must call it.
__device__ __forceinline__ void emit_tile_max(float cmax, uint32_t *amax_out)
{
    if (!amax_out) return;   // uniform
    __shared__ float wave_m[8];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, off));
    if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = cmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < (int)(blockDim.x >> 6); ++i) cmax = fmaxf(cmax, wave_m[i]);
        max_to_global(cmax, amax_out);
    }
}

// The two scale bytes of a lane's 32 elements of K, as two f16 numbers in one register: byte b in
// f16 position (b << 7) is e4m3 * 2^-8, subnormals included.  v_perm_b32 spreads the bytes to the
// two halves, one shift moves them to f16 position.
constexpr uint32_t kScalesLow = 0x0C010C00u, kScalesHigh = 0x0C030C02u;   // of the two in the low or the high half of a word
__device__ __forceinline__ uint32_t scale_halves(uint32_t bytes, uint32_t selector = kScalesLow)
{
    return __builtin_amdgcn_perm(0u, bytes, selector) << 7;
}

// half of one fragment (4 of its 8 values): two conversions and two packed multiplies by the f16
// scale in the low (kHi = 0) or high half of `scales`, taken for both lanes of the packed multiply
// through the instruction's operand selectors
template <int H, int kHi>
__device__ __forceinline__ void dequant_half(half8_t &dst, uint32_t codes, uint32_t scales)
{
    const half2_t c0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes, 256.0f, 2 * H);
    const half2_t c1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes, 256.0f, 2 * H + 1);
    half2_t h0, h1;
    if (kHi) {
        asm("v_pk_mul_f16 %0, %1, %2 op_sel:[0,1] op_sel_hi:[1,1]" : "=v"(h0) : "v"(c0), "v"(scales));
        asm("v_pk_mul_f16 %0, %1, %2 op_sel:[0,1] op_sel_hi:[1,1]" : "=v"(h1) : "v"(c1), "v"(scales));
    } else {
        asm("v_pk_mul_f16 %0, %1, %2 op_sel_hi:[1,0]" : "=v"(h0) : "v"(c0), "v"(scales));
        asm("v_pk_mul_f16 %0, %1, %2 op_sel_hi:[1,0]" : "=v"(h1) : "v"(c1), "v"(scales));
    }
    dst[4 * H] = h0[0]; dst[4 * H + 1] = h0[1]; dst[4 * H + 2] = h1[0]; dst[4 * H + 3] = h1[1];
}

// The lanes of a wave exchange data through LDS: its LDS operations run in order, so nothing has to be waited
// for; the compiler only must not move accesses across this point.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Epilogue: C = acc * ts for a wave's tile of 32 MT x 32 NT entries at (row0, col0).  The matrix instructions take B's
// fragment as their first operand and A's as their second, so entry r of accumulator (i, j) is row 32 i + lane % 32,
// column 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4: a lane holds four neighbouring entries of a row, which go into
// the wave's staging area as 8 (bf16) or 16 bytes at once (row pitch padded by 16 bytes: no bank conflicts for the
// 16-byte accesses).  kGroup bands of 32 rows are staged, then stored as 16-byte pieces of full rows while the next group
// is converted; the area holds kRoom bands.  (One band at a time, two bytes per LDS write, with the wave waiting for
// each: 6.1 us for the main kernel's 256 x 256 bf16 tile and 9.3 for f32; now 3.6 and 7.3; the
// 128 x 128 form of the small-tile kernels, reduction included, 5.4 -> 2.7.)
// A tile that lies inside C with 16-byte aligned rows takes the loop without checks; where the rows are aligned only the
// pieces that N cuts go entry by entry; other rows: consecutive lanes store consecutive entries (store_entries).
// kStreaming: C is written once and not read again here, so the stores are non-temporal (false: a partial tile that
// the next kernel reads back).  kPaced: a pause before each store of a whole tile.  All threads of the block must call it if
// amax_out is given.
template <bool kBf16Out, int NT>
constexpr int staging_pitch() { return 32 * NT * (kBf16Out ? 2 : 4) + 16; }

// `rows` staged rows whose places in C are aligned for one entry only, or (kEach = 2, bf16) for two: consecutive lanes store
// consecutive entries, the reads of eight rows not waiting for the stores of those before.  A column is checked once, a row
// only beside the last ones, and the maximum taken only where it is wanted (uniform): with all three at each store, bf16
// 9420 x 2177 x 256 took 30.7 us instead of 27.5, f32 922 x 12753 x 256 22.4 instead of 21.3.
template <bool kBf16Out, int NT, int kEach, int kRows>
__device__ __forceinline__ void store_entries(const uint8_t *staged, uint8_t *out, int64_t rb, int live_rows, int live_cols, int lane, bool want_max,
                                              float &cmax)
{
    constexpr int esz = kBf16Out ? 2 : 4, cols = 32 * NT, pitch = staging_pitch<kBf16Out, NT>(), kAtOnce = 8;
    constexpr int lanes = cols / kEach < 64 ? cols / kEach : 64, rows_at_once = 64 / lanes;
    static_assert(kRows % (kAtOnce * rows_at_once) == 0, "whole steps");
    const int rl = lane / lanes;
#pragma unroll 1
    for (int c0 = 0; c0 < cols; c0 += lanes * kEach) {
        const int col = c0 + lane % lanes * kEach;
        const uint8_t *src = staged + rl * pitch + col * esz;
        uint8_t *dst = out + rl * rb + col * esz;
        if (col >= live_cols) continue;
        const bool both = kEach == 2 && col + 1 < live_cols;
#pragma unroll 1
        for (int r0 = 0; r0 < kRows && r0 < live_rows; r0 += kAtOnce * rows_at_once) {
            uint32_t v[kAtOnce];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) {
                const uint8_t *e = src + (r0 + i * rows_at_once) * pitch;
                v[i] = esz * kEach == 4 ? *reinterpret_cast<const uint32_t *>(e) : (uint32_t)*reinterpret_cast<const uint16_t *>(e);
            }
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) {
                const int row = r0 + i * rows_at_once;
                if (row + rl >= live_rows) continue;
                uint8_t *d = dst + row * rb;
                if (esz * kEach == 4 && (kEach == 1 || both)) *reinterpret_cast<uint32_t *>(d) = v[i];
                else *reinterpret_cast<uint16_t *>(d) = (uint16_t)v[i];
            }
            if (want_max)
#pragma unroll
                for (int i = 0; i < kAtOnce; ++i) {
                    if (r0 + i * rows_at_once + rl >= live_rows) continue;
                    cmax = fmaxf(cmax, fabsf(u2f(kBf16Out ? v[i] << 16 : v[i])));
                    if (both) cmax = fmaxf(cmax, fabsf(u2f(v[i] & 0xFFFF0000u)));
                }
        }
    }
}

template <bool kBf16Out, bool kStreaming, int MT, int NT, int kGroup, int kRoom, bool kPaced = false>
__device__ __forceinline__ void store_tile(const floatx16 (&acc)[MT][NT], uint8_t *area, float ts, void *Cout, int64_t ldc, int64_t M,
                                           int64_t N, int64_t row0, int64_t col0, int lane, uint32_t *amax_out)
{
    constexpr int esz = kBf16Out ? 2 : 4, cols = 32 * NT, pitch = staging_pitch<kBf16Out, NT>(), entries = 16 / esz;
    constexpr int per_row = cols / entries, rows_per_pass = 64 / per_row, kPasses = 32 * kGroup / rows_per_pass;
    static_assert(MT % kGroup == 0 && kRoom % kGroup == 0, "whole groups");
    const int64_t rb = ldc * esz;   // bytes from row to row of C
    uint8_t *out = reinterpret_cast<uint8_t *>(Cout) + row0 * rb + col0 * esz;
    const int live_rows = (int)(M - row0 < 32 * MT ? M - row0 : 32 * MT), live_cols = (int)(N - col0 < cols ? N - col0 : cols);   // (may be negative)
    const bool aligned = ((reinterpret_cast<uintptr_t>(Cout) | (uintptr_t)rb) & 15) == 0;   // (col0: a multiple of 32)
    const bool pairs = ((reinterpret_cast<uintptr_t>(Cout) | (uintptr_t)rb) & 3) == 0;
    const bool whole = aligned && live_rows == 32 * MT && live_cols == cols && rb < (1 << 26);
    const int piece = lane % per_row, row_l = lane / per_row;
    uint8_t *lane_write = area + (lane & 31) * pitch + (lane >> 5) * 4 * esz;
    const uint8_t *lane_read = area + row_l * pitch + piece * 16;
    float cmax = 0.0f;
    auto fold = [&](const u32x4 &v) {
#pragma unroll
        for (int e = 0; e < entries; ++e)
            cmax = fmaxf(cmax, fabsf(kBf16Out ? u2f((e & 1) ? (v[e >> 1] & 0xFFFF0000u) : (v[e >> 1] << 16)) : u2f(v[e & 3])));
    };
    auto put = [&](uint8_t *dst, const u32x4 &v) {
        if (kStreaming) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
        else *reinterpret_cast<u32x4 *>(dst) = v;
    };
    auto put_entry = [&](int row, int col, const uint8_t *src) {
        uint8_t *dst = out + row * rb + col * esz;
        uint32_t v;
        if (kBf16Out) *reinterpret_cast<uint16_t *>(dst) = (uint16_t)(v = *reinterpret_cast<const uint16_t *>(src));
        else *reinterpret_cast<uint32_t *>(dst) = v = *reinterpret_cast<const uint32_t *>(src);
        cmax = fmaxf(cmax, fabsf(u2f(kBf16Out ? v << 16 : v)));
    };
#pragma unroll
    for (int g = 0; g < MT; g += kGroup) {
        constexpr int kBand = 32 * pitch;
        const int band0 = g % kRoom;   // (a compile-time constant)
#pragma unroll
        for (int b = 0; b < kGroup; ++b)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const floatx16 &a = acc[g + b][j];
                    const float v0 = a[4 * q] * ts, v1 = a[4 * q + 1] * ts, v2 = a[4 * q + 2] * ts, v3 = a[4 * q + 3] * ts;
                    uint8_t *dst = lane_write + (band0 + b) * kBand + (32 * j + 8 * q) * esz;
                    if (kBf16Out) {   // (two packed conversions, round to nearest even)
                        const uint32_t lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(float2_t{v0, v1}, bf16x2_t));
                        const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(float2_t{v2, v3}, bf16x2_t));
                        *reinterpret_cast<uint2 *>(dst) = make_uint2(lo, hi);
                    } else {
                        *reinterpret_cast<float4 *>(dst) = make_float4(v0, v1, v2, v3);
                    }
                }
        wave_lds_fence();
        const uint8_t *src = lane_read + band0 * kBand;
        uint8_t *row_out = out + 32 * g * rb;   // (uniform)
        if (whole) {   // uniform
            const uint32_t voff = (uint32_t)row_l * (uint32_t)rb + (uint32_t)piece * 16u;
            constexpr int kMost = kPaced ? 2 : 8, kAtOnce = kPasses < kMost ? kPasses : kMost;
#pragma unroll
            for (int p0 = 0; p0 < kPasses; p0 += kAtOnce) {
                u32x4 v[kAtOnce];
#pragma unroll
                for (int p = 0; p < kAtOnce; ++p) v[p] = *reinterpret_cast<const u32x4 *>(src + (p0 + p) * rows_per_pass * pitch);
#pragma unroll
                for (int p = 0; p < kAtOnce; ++p) {
                    if (kPaced) __builtin_amdgcn_s_sleep(3);   // (192 cycles)
                    put(row_out + (p0 + p) * rows_per_pass * rb + voff, v[p]);
                }
                if (amax_out)   // uniform
#pragma unroll
                    for (int p = 0; p < kAtOnce; ++p) fold(v[p]);
            }
        } else if (aligned) {
#pragma unroll 1
            for (int p = 0; p < kPasses; ++p) {
                const int row = 32 * g + p * rows_per_pass + row_l;
                if (row < live_rows && (piece + 1) * entries <= live_cols) {
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(src + p * rows_per_pass * pitch);
                    put(out + row * rb + piece * 16, v);
                    if (amax_out) fold(v);
                }
            }
            if (live_cols > 0 && live_cols % entries != 0 && lane < 32)   // the rows' last, partial piece
#pragma unroll 1
                for (int b = 0; b < kGroup; ++b)
                    if (32 * (g + b) + lane < live_rows)
#pragma unroll 1
                        for (int col = live_cols / entries * entries; col < live_cols; ++col)
                            put_entry(32 * (g + b) + lane, col, area + ((band0 + b) * 32 + lane) * pitch + col * esz);
        } else {
            const uint8_t *group = area + band0 * kBand;
            if (kBf16Out && pairs) store_entries<kBf16Out, NT, 2, 32 * kGroup>(group, row_out, rb, live_rows - 32 * g, live_cols, lane, amax_out != nullptr, cmax);   // uniform
            else store_entries<kBf16Out, NT, 1, 32 * kGroup>(group, row_out, rb, live_rows - 32 * g, live_cols, lane, amax_out != nullptr, cmax);
        }
        wave_lds_fence();   // the reads come before the writes of a group that takes the same room
    }
    emit_tile_max(cmax, amax_out);
}

}  // namespace
}  // namespace qii
