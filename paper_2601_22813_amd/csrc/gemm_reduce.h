// Sum of the K groups' accumulators through LDS, at the end of a block of the small-tile GEMM kernels (gemm_small.hip).
// Uses floatx16 and wave_lds_fence of gemm_common.h; a header of its own so that a CPU can run it, lane by lane.
#pragma once
#include <stdint.h>

namespace qii {
namespace {

// Unit u of a wave of group kg (of KG, N units a wave) is the wave's 32 x 32 tile u ^ reduce_flip: the groups hold their tiles
// in different orders, so that every group keeps the first half of its units in each round and gives away the second, and no wave
// has code of its own.  (Chosen by value, which half is kept cost a select per accumulator and round, 1.2 us of the 128 x 128 form's
// 5.5 from the last product to the last store; chosen by a branch, barriers and the registers of both halves
// are in the way: 68 bytes of scratch memory in the 4 x 4 form.)
template <int KG, int N>
__device__ __forceinline__ constexpr int reduce_flip(int kg) { return kg * (N / KG); }

// One round: partners exchange halves.  A wave writes the area `own` and reads its partner's, `other`, which nobody else
// reads: after a round that area is the wave's own, for the next round or the epilogue, in any lane layout (the fence),
// with no barrier between.
template <int N>
__device__ __forceinline__ void reduce_round(const floatx16 (&u)[N], floatx16 (&out)[N / 2], uint8_t *own, const uint8_t *other, int lane)
{
    float4 *give_to = reinterpret_cast<float4 *>(own) + lane;
    const float4 *take_from = reinterpret_cast<const float4 *>(other) + lane;
#pragma unroll
    for (int k = 0; k < N / 2; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const floatx16 &give = u[N / 2 + k];
            give_to[(k * 4 + r) * 64] = make_float4(give[4 * r], give[4 * r + 1], give[4 * r + 2], give[4 * r + 3]);
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N / 2; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float4 v = take_from[(k * 4 + r) * 64];
            out[k][4 * r] = u[k][4 * r] + v.x;
            out[k][4 * r + 1] = u[k][4 * r + 1] + v.y;
            out[k][4 * r + 2] = u[k][4 * r + 2] + v.z;
            out[k][4 * r + 3] = u[k][4 * r + 3] + v.w;
        }
    wave_lds_fence();
}

// The whole sum of a block of KG groups of WM waves, an area of kArea bytes per wave: out[k] of wave wm of group kg is tile
// reduce_flip(kg) + k.  Returns the area that is this wave's own from then on.  All threads of the block call
// it, behind a barrier after their last other use of smem.
template <int WM, int KG, int kArea, int N>
__device__ __forceinline__ uint8_t *reduce_groups(const floatx16 (&acc)[N], floatx16 (&out)[N / KG], uint8_t *smem, int kg, int wm, int lane)
{
    static_assert(KG == 2 || KG == 4, "one or two rounds");
    uint8_t *const wave0 = smem + wm * kArea;   // (partners have the same wm)
    constexpr int kGroup = WM * kArea;
    if constexpr (KG == 2) {
        reduce_round(acc, out, wave0 + kg * kGroup, wave0 + (kg ^ 1) * kGroup, lane);
        return wave0 + (kg ^ 1) * kGroup;
    } else {
        floatx16 h[N / 2];
        reduce_round(acc, h, wave0 + kg * kGroup, wave0 + (kg ^ 2) * kGroup, lane);
        reduce_round(h, out, wave0 + (kg ^ 2) * kGroup, wave0 + (kg ^ 3) * kGroup, lane);
        return wave0 + (kg ^ 3) * kGroup;
    }
}

}  // namespace
}  // namespace qii
