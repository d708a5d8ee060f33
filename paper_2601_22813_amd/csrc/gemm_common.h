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
__device__ __forceinline__ uint32_t scale_halves(uint32_t two_bytes)
{
    return __builtin_amdgcn_perm(0u, two_bytes, 0x0C010C00u) << 7;
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

// epilogue: C = acc * (x32_A * x32_B).  acc[r] of a 32x32 tile is row
// 8*(r/4) + 4*(lane/32) + r%4, column lane%32.  One 32-row band of the wave's 32 MT x 32 NT tile
// at a time goes through a per-wave LDS tile (row pitch padded by 16 bytes) and leaves as
// 16-byte pieces of full rows.  The caller guarantees that nobody reads the stages any more.
template <bool kBf16Out, bool kStreaming = true, int MT = 4, int NT = 4>
__device__ __forceinline__ void store_tile_through_lds(floatx16 (&acc)[MT][NT], uint8_t *smem, float ts,
                                                       void *Cout, int64_t ldc, int64_t M, int64_t N,
                                                       int64_t m0, int64_t n0, int wave, int wm, int wn,
                                                       int lane, int li, int kb, uint32_t *amax_out)
{
    float cmax = 0.0f;
    constexpr int esz = kBf16Out ? 2 : 4;
    constexpr int pitch = 32 * NT * esz + 16;
    uint8_t *wtile = smem + wave * (32 * pitch);
    constexpr int per_row = 32 * NT * esz / 16;          // 16-byte pieces per row
    constexpr int rows_per_pass = 64 / per_row;      // rows covered by one wave-wide store
#pragma unroll
    for (int ti = 0; ti < MT; ++ti) {
#pragma unroll
        for (int tj = 0; tj < NT; ++tj)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                // two consecutive rows of one column: one packed conversion (round to nearest even)
                const int row = 8 * (r >> 2) + 4 * kb + (r & 3), col = tj * 32 + li;
                const float v0 = acc[ti][tj][r] * ts, v1 = acc[ti][tj][r + 1] * ts;
                if (kBf16Out) {
                    const bf16x2_t pk = __builtin_convertvector(float2_t{v0, v1}, bf16x2_t);
                    const uint32_t bits = __builtin_bit_cast(uint32_t, pk);
                    *reinterpret_cast<uint16_t *>(wtile + row * pitch + col * 2) = (uint16_t)bits;
                    *reinterpret_cast<uint16_t *>(wtile + (row + 1) * pitch + col * 2) = (uint16_t)(bits >> 16);
                } else {
                    *reinterpret_cast<float *>(wtile + row * pitch + col * 4) = v0;
                    *reinterpret_cast<float *>(wtile + (row + 1) * pitch + col * 4) = v1;
                }
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // wave-local: same wave reads below
#pragma unroll
        for (int pass = 0; pass < 32 / rows_per_pass; ++pass) {
            const int row = pass * rows_per_pass + lane / per_row, piece = lane % per_row;
            const uint4 v = *reinterpret_cast<const uint4 *>(wtile + row * pitch + piece * 16);
            const int64_t grow = m0 + wm * (32 * MT) + ti * 32 + row;
            const int64_t gcol = n0 + wn * (32 * NT) + piece * (16 / esz);
            if (grow < M) {
                if (amax_out) {   // uniform: max |C| over the entries of this piece that lie inside the matrix
                    const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 16 / esz; ++e)
                        if (gcol + e < N)
                            cmax = fmaxf(cmax, fabsf(kBf16Out ? u2f((e & 1) ? (w4[e >> 1] & 0xFFFF0000u) : (w4[e >> 1] << 16)) : u2f(w4[e])));
                }
                uint8_t *dst = reinterpret_cast<uint8_t *>(Cout) + (grow * ldc + gcol) * esz;
                if (gcol + 16 / esz <= N && ((reinterpret_cast<uintptr_t>(dst) & 15) == 0)) {
                    // C is written once and not read again here: a streaming (non-temporal) store
                    // (kStreaming = false: a partial tile that the next kernel reads back)
                    if (kStreaming) __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(dst));
                    else *reinterpret_cast<u32x4 *>(dst) = u32x4{v.x, v.y, v.z, v.w};
                } else {
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 16 / esz; ++e)
                        if (gcol + e < N) {
                            if (kBf16Out) reinterpret_cast<uint16_t *>(dst)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                            else reinterpret_cast<uint32_t *>(dst)[e] = w[e];
                        }
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // reads done before the next band overwrites
    }
    emit_tile_max(cmax, amax_out);
}

}  // namespace
}  // namespace qii
