// Small-tile kernels of the block-scaled NVFP4 GEMM (same scheme as gemm.hip: raw codes and scale
// bytes in LDS, fragments dequantized to exact f16 products in registers, f16 matrix instruction):
// for products whose 256 x 256 tiles leave most compute units idle, and for any K that is a multiple
// of 16 (NVFP4's own rule).
//
// A wave dequantizes MT + NT fragments per MT * NT matrix instructions (2 conversions + 2 packed products
// each per matrix instruction at 4 x 4, the main kernel's tile; 3 + 3 at 2 x 4, 4 + 4 at 2 x 2, 8 + 8 at
// 1 x 1, against 32 cycles of the matrix pipe), so a wave's tile must stay as large as its registers
// allow even where the block's tile is small.  The waves of a block therefore share K, not M and N: the
// four 64-wide slices of a 256-wide K tile go to KG groups of waves, and the groups' accumulators are added
// through LDS at the end, in a fixed order.
//   128 x 128 block tile: 2 waves of 64 x 128 (MT, NT = 2, 4) per group, 2 groups (two blocks per compute unit);
//                         or one wave of 128 x 128 (4, 4) per group, 4 groups (one block per unit);
//   64 x 64 block tile:   one wave of 64 x 64 (2, 2) per group, 4 groups.
//
// Operands are staged through registers (global -> VGPR -> LDS) but for the 4 x 4 form where gemm_wide_applies (gemm_wide_kernel): a tile is
// small enough for that (at most 36 registers), the next tile's loads then stay in flight for a whole tile's time, and a ragged K
// needs no padding of the operands: codes and scales beyond K are staged as zeros.  The scale bytes are
// read row-major or in the tiled layout, whichever the operand has: no re-tiling launch, no workspace.
#include <utility>

#include "gemm_common.h"
#include "gemm_reduce.h"
#include "gemm_tail.h"
#include "qii_device.h"
#include "qii_internal.h"

namespace qii {
namespace {

constexpr int BK = 256;

// where an operand's scale bytes are: 16 bytes per row and K tile at s + row_term(row) + kt * kt_stride
struct ScaleView {
    const uint8_t *s;
    int64_t row_pitch;    // row-major: bytes per row; tiled: bytes per 256 rows
    int64_t kt_stride;    // row-major: 16; tiled: 4096
    int tiled;
};

struct SmallArgs {
    const uint8_t *a_codes, *b_codes;
    ScaleView as, bs;
    const float *a_ts, *b_ts;
    int64_t M, N, K;
    void *C;
    int64_t ldc;
    int tiles_m, tiles_n;
    uint32_t *amax_out;
};

__device__ __forceinline__ const uint8_t *scale_row(const ScaleView &v, int64_t row)
{
    return v.tiled ? v.s + (row >> 8) * v.row_pitch + (row & 255) * 16 : v.s + row * v.row_pitch;
}

// Block of WM * KG waves: tile BM x BN, wave tile 32 MT x 32 NT (the waves of a group sit below one another)
template <int MT_, int NT_, int WM_, int KG_>
struct Geo {
    static constexpr int MT = MT_, NT = NT_, WM = WM_, KG = KG_;
    static constexpr int BM = 32 * MT * WM, BN = 32 * NT, kThreads = 64 * WM * KG;
    static constexpr int kRowsPerPass = kThreads / 8;         // 8 pieces of 16 bytes per code row
    static constexpr int kPassA = BM / kRowsPerPass, kPassB = BN / kRowsPerPass;
    static constexpr bool kNarrow = MT < 4;                   // see Sources
    static constexpr int kBlocksPerUnit = MT == 4 ? 1 : NT == 4 ? 2 : 3;   // (registers: 512, 256, 168)
    static constexpr int kSlices = 4 / KG;                    // of a K tile per group
    static constexpr int kStage = (BM + BN) * (128 + 16);     // LDS bytes of one K tile
    static constexpr int kUnits = MT * NT;                    // 32 x 32 accumulator tiles of a wave
    // what a wave finishes once the groups' accumulators are added up
    static constexpr int FM = KG == 2 ? MT / 2 : 1, FN = KG == 2 || MT == 4 ? NT : NT / 2;
    static_assert(FM * FN * KG == kUnits, "the groups share the tile");
    // a wave's fragments of A and B are in the order that reduce_groups asks of its group: unit i NT + j is tile (i ^ row_flip, j ^ col_flip)
    __device__ static constexpr int row_flip(int kg) { return reduce_flip<KG, kUnits>(kg) / NT; }
    __device__ static constexpr int col_flip(int kg) { return reduce_flip<KG, kUnits>(kg) % NT; }
    // LDS: two stages; then, per wave, half of its accumulators (the reduction's first round) or the rows it stores
    static constexpr int kStaged = FM * 32 * staging_pitch<false, FN>();
    static constexpr int kArea = (kUnits / 2) * 4096 > kStaged ? (kUnits / 2) * 4096 : kStaged;
    static constexpr int kLds = 2 * kStage > WM * KG * kArea ? 2 * kStage : WM * KG * kArea;
};

// One thread's share of a K tile on its way to LDS: 16-byte pieces of code rows and, for threads below
// the row count, one row's 16 scale bytes
template <class G>
struct Staged {
    uint4 a[G::kPassA], b[G::kPassB], s;
};

// This thread's source addresses (K tile 0), rows beyond the matrix replaced by its last row (their results land in
// accumulator rows or columns that are never stored).  kNarrow (the forms whose registers are short: 256 for two blocks per unit,
// 168 for three): 32-bit offsets from the tile's first row, which is in scalar registers; a block tile's rows are then below 4 GiB
// (kMaxNarrowK).  With 64-bit addresses the two-group form keeps the scale bytes on their way to LDS in scratch memory, and
// every K tile waits for its successor's loads: 2048 x 2048 x 1024 14.4 us instead of 12.8, 2816 x 2048 x 4096 62.4 instead of 56.5.
template <class G>
struct Sources {
    const uint8_t *a0, *b0, *s0;   // uniform (kNarrow)
    const uint8_t *a[G::kNarrow ? 1 : G::kPassA], *b[G::kNarrow ? 1 : G::kPassB], *s;
    uint32_t a_off[G::kPassA], b_off[G::kPassB], s_off;
    int64_t kt_stride;
};

// piece p of A's (or B's) rows in the tile that o stands for
template <class G, bool kA>
__device__ __forceinline__ const uint8_t *codes_at(const Sources<G> &src, int p, const TileOffsets &o)
{
    if constexpr (G::kNarrow) return piece_at(kA ? src.a0 : src.b0, kA ? src.a_off[p] : src.b_off[p], o);
    else return piece_at(kA ? src.a[p] : src.b[p], o);
}

template <class G, bool kAnyK, bool kA>
__device__ __forceinline__ uint4 load_codes16(const Sources<G> &src, int p, const TileOffsets &o)
{
    const uint8_t *c = codes_at<G, kA>(src, p, o);
    if (!kAnyK) return *reinterpret_cast<const uint4 *>(c);
    const uint2 l = *reinterpret_cast<const uint2 *>(c), h = *reinterpret_cast<const uint2 *>(c + 8);
    return make_uint4(l.x, l.y, h.x, h.y);
}

template <bool kAnyK>
__device__ __forceinline__ uint4 load_scales16(const uint8_t *p)
{
    if (kAnyK) {
        uint4 v;
        __builtin_memcpy(&v, p, 16);
        return v;
    }
    const uint2 lo = *reinterpret_cast<const uint2 *>(p), hi = *reinterpret_cast<const uint2 *>(p + 8);   // (8-byte aligned)
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}

// rows of fewer than 16 scale bytes (K < 256)
__device__ __forceinline__ uint4 load_scales_short(const uint8_t *p, int groups)
{
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i >> 2] |= (i < groups ? (uint32_t)p[i < groups ? i : 0] : 0u) << (8 * (i & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

template <class G>
__device__ __forceinline__ const uint8_t *scales_at(const Sources<G> &src, int64_t offset)
{
    if constexpr (G::kNarrow) return src.s0 + offset + src.s_off;
    else return src.s + offset;
}

template <class G, bool kAnyK, bool kFirst>
__device__ __forceinline__ void load_tile(Staged<G> &st, const Sources<G> &src, int kt, int64_t K)
{
    const TileOffsets o = tile_offsets<kAnyK>(kt, src.kt_stride, K, threadIdx.x & 7);
    if (kAnyK && kFirst && K < 32) {   // uniform: 8 bytes a row
#pragma unroll
        for (int p = 0; p < G::kPassA + G::kPassB; ++p) {
            const uint2 c = *reinterpret_cast<const uint2 *>(p < G::kPassA ? codes_at<G, true>(src, p, o) : codes_at<G, false>(src, p - G::kPassA, o));
            (p < G::kPassA ? st.a[p] : st.b[p - G::kPassA]) = make_uint4(0u, 0u, c.x, c.y);
        }
    } else {
#pragma unroll
        for (int p = 0; p < G::kPassA; ++p) st.a[p] = load_codes16<G, kAnyK, true>(src, p, o);
#pragma unroll
        for (int p = 0; p < G::kPassB; ++p) st.b[p] = load_codes16<G, kAnyK, false>(src, p, o);
    }
    if ((int)threadIdx.x < G::BM + G::BN) {
        if (kAnyK && kFirst && K < BK) st.s = load_scales_short(scales_at(src, 0), (int)K / 16);   // uniform
        else st.s = load_scales16<kAnyK>(scales_at(src, o.s));
    }
}

// The last, partial tile: what came from the end of the row to its place, zeros beyond K.
template <class G>
__device__ __forceinline__ void finish_tail(Staged<G> &st, int kt, int64_t K)
{
    const int tail = (int)(K - (int64_t)kt * BK), left = tail - 32 * (int)(threadIdx.x & 7);
#pragma unroll
    for (int p = 0; p < G::kPassA; ++p) finish_piece(st.a[p], left);
#pragma unroll
    for (int p = 0; p < G::kPassB; ++p) finish_piece(st.b[p], left);
    if (kt > 0) finish_scales(st.s, tail);   // (rows of 16 bytes or more)
}

// LDS stage: A codes, B codes (128 bytes per row; row r keeps its 16-byte piece s in slot s ^ (r & 7), so
// that the 128-bit reads of 8 consecutive rows hit different banks), then the rows' 16 scale bytes
template <class G>
__device__ __forceinline__ void store_tile(const Staged<G> &st, uint8_t *stage)
{
    const int t = threadIdx.x, slot = ((t & 7) ^ ((t >> 3) & 7)) * 16;   // (rows of a thread differ by multiples of 8)
    uint8_t *dst = stage + (t >> 3) * 128 + slot;
#pragma unroll
    for (int p = 0; p < G::kPassA; ++p) *reinterpret_cast<uint4 *>(dst + p * G::kRowsPerPass * 128) = st.a[p];
#pragma unroll
    for (int p = 0; p < G::kPassB; ++p) *reinterpret_cast<uint4 *>(dst + (G::BM + p * G::kRowsPerPass) * 128) = st.b[p];
    if (t < G::BM + G::BN) *reinterpret_cast<uint4 *>(stage + (G::BM + G::BN) * 128 + t * 16) = st.s;
}

// raw fragments of one 64-wide K slice: 32 codes and two scale bytes per lane and 32-row block
template <class G>
struct RawFrags {
    u32x4 a[G::MT], b[G::NT];
    uint32_t sa[G::MT], sb[G::NT];
};

template <class G>
__device__ __forceinline__ void read_slice(RawFrags<G> &f, const uint8_t *stage, int j, int wm, int kg, int li, int kb)
{
    const int slot = ((2 * j + kb) ^ (li & 7)) * 16, sc = 4 * j + 2 * kb;
    const uint8_t *codes = stage, *scales = stage + (G::BM + G::BN) * 128;
#pragma unroll
    for (int t = 0; t < G::MT; ++t) {
        const int row = (wm * G::MT + (t ^ G::row_flip(kg))) * 32 + li;
        f.a[t] = *reinterpret_cast<const u32x4 *>(codes + row * 128 + slot);
        f.sa[t] = *reinterpret_cast<const uint16_t *>(scales + row * 16 + sc);
    }
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
        const int row = G::BM + (t ^ G::col_flip(kg)) * 32 + li;
        f.b[t] = *reinterpret_cast<const u32x4 *>(codes + row * 128 + slot);
        f.sb[t] = *reinterpret_cast<const uint16_t *>(scales + row * 16 + sc);
    }
}

// Dword D of a fragment's codes -> 8 exact f16 values.  The products are written in plain C++ (they compile
// to one packed multiply with operand selectors each), not as the inline assembly of dequant_half: here a
// matrix instruction may follow at once, and only the compiler knows how far it must stay behind.
template <int D>
__device__ __forceinline__ half8_t dequant_dword(const u32x4 &codes, uint32_t scales)
{
    const half2_t both = __builtin_bit_cast(half2_t, scales), s = {both[D >> 1], both[D >> 1]};
    const half2_t h0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes[D], 256.0f, 0) * s;
    const half2_t h1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes[D], 256.0f, 1) * s;
    const half2_t h2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes[D], 256.0f, 2) * s;
    const half2_t h3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes[D], 256.0f, 3) * s;
    half8_t r;
    r[0] = h0[0]; r[1] = h0[1]; r[2] = h1[0]; r[3] = h1[1];
    r[4] = h2[0]; r[5] = h2[1]; r[6] = h3[0]; r[7] = h3[1];
    return r;
}

template <class G, int D>
__device__ __forceinline__ void mma_dword(floatx16 (&acc)[G::kUnits], const RawFrags<G> &f)
{
    half8_t fa[G::MT], fb[G::NT];
#pragma unroll
    for (int t = 0; t < G::MT; ++t) fa[t] = dequant_dword<D>(f.a[t], f.sa[t]);
#pragma unroll
    for (int t = 0; t < G::NT; ++t) fb[t] = dequant_dword<D>(f.b[t], f.sb[t]);
    // (2 x 2: rows outside, 2857 x 123 x 20992 64.7 us, 1024 x 1024 x 2048 10.1; columns outside 67.0 and 10.3.  2 x 4: columns
    // outside, 2048 x 2048 x 512 9.9, 4096 x 2048 x 1024 21.2; rows outside 10.5 and 22.6)
#pragma unroll
    for (int k = 0; k < G::kUnits; ++k) {
        const int i = G::NT == 2 ? k / G::NT : k % G::MT, j = G::NT == 2 ? k % G::NT : k / G::MT;
        acc[i * G::NT + j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[j], fa[i], acc[i * G::NT + j], 0, 0, 0);   // (B first: store_tile)
    }
}

// first and second half of the 64-wide K slice held in f
template <class G>
__device__ __forceinline__ void mma_first(floatx16 (&acc)[G::kUnits], RawFrags<G> &f)
{
#pragma unroll
    for (int t = 0; t < G::MT; ++t) f.sa[t] = scale_halves(f.sa[t]);
#pragma unroll
    for (int t = 0; t < G::NT; ++t) f.sb[t] = scale_halves(f.sb[t]);
    mma_dword<G, 0>(acc, f);
    mma_dword<G, 1>(acc, f);
}

template <class G>
__device__ __forceinline__ void mma_second(floatx16 (&acc)[G::kUnits], const RawFrags<G> &f)
{
    mma_dword<G, 2>(acc, f);
    mma_dword<G, 3>(acc, f);
}

// ---- explicit pipeline of the one-wave-per-SIMD form (4 x 4 tiles) -----------------------------
// While a step's 16 matrix instructions run on the fragments in cu, the next step's fragments (dword D of
// f) are dequantized into nx, half a fragment after each matrix instruction; the scheduling barriers keep
// that order.  A fragment is complete several matrix instructions before the first one that reads it.
template <class G>
struct Frags {
    half8_t a[G::MT], b[G::NT];
};

template <class G, int D>
__device__ __forceinline__ void dequant_chunk(Frags<G> &nx, RawFrags<G> &f, int i)
{
    const int t = (i >> 1) & 3;
    if (i < 8) {
        if (D == 0 && (i & 1) == 0) f.sa[t] = scale_halves(f.sa[t]);
        if ((i & 1) == 0) dequant_half<0, (D >> 1)>(nx.a[t], f.a[t][D], f.sa[t]);
        else dequant_half<1, (D >> 1)>(nx.a[t], f.a[t][D], f.sa[t]);
    } else {
        if (D == 0 && (i & 1) == 0) f.sb[t] = scale_halves(f.sb[t]);
        if ((i & 1) == 0) dequant_half<0, (D >> 1)>(nx.b[t], f.b[t][D], f.sb[t]);
        else dequant_half<1, (D >> 1)>(nx.b[t], f.b[t][D], f.sb[t]);
    }
}

// side(i): further work of the caller after matrix instruction i (memory operations, spread out)
template <class G, int D, class Side>
__device__ __forceinline__ void mma_step(floatx16 (&acc)[G::kUnits], const Frags<G> &cu, Frags<G> &nx, RawFrags<G> &f, Side &&side)
{
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = i >> 2, col = i & 3;
        acc[row * G::NT + col] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cu.b[col], cu.a[row], acc[row * G::NT + col], 0, 0, 0);
        side(i);
        dequant_chunk<G, D>(nx, f, i);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// stores what the wave has finished: FM x FN tiles
template <bool kBf16Out, class G>
__device__ __forceinline__ void finish(const floatx16 (&u)[G::FM * G::FN], uint8_t *area, float ts, const SmallArgs &g, int64_t row0, int64_t col0, int lane)
{
    floatx16 c[G::FM][G::FN];
#pragma unroll
    for (int i = 0; i < G::FM; ++i)
#pragma unroll
        for (int j = 0; j < G::FN; ++j) c[i][j] = u[i * G::FN + j];
    store_tile<kBf16Out, true, G::FM, G::FN, 1, 1>(c, area, ts, g.C, g.ldc, g.M, g.N, row0, col0, lane, g.amax_out);
}

template <bool kBf16Out, class G, bool kAnyK>
__global__ __launch_bounds__(G::kThreads, G::kBlocksPerUnit) void gemm_small_kernel(SmallArgs g0, SmallArgs g1, int n0_blocks)
{
    // one product, or two in one launch: the first n0_blocks blocks take g0, the others g1
    const bool first = (int)blockIdx.x < n0_blocks;   // uniform
    SmallArgs g = g0;
    if (!first) g = g1;
    extern __shared__ __align__(16) uint8_t smem[];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave % G::WM, kg = wave / G::WM;
    const int li = lane & 31, kb = lane >> 5;
    int tm, tn;
    tile_coords((int)blockIdx.x - (first ? 0 : n0_blocks), g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * G::BM, n0 = (int64_t)tn * G::BN;

    Sources<G> src;
    {
        const int64_t pitch = g.K / 2;
        const int off = 16 * (t & 7);
        auto row_of = [](int64_t r, int64_t rows) { return r < rows ? r : rows - 1; };
        if constexpr (G::kNarrow) {
            src.a0 = g.a_codes + m0 * pitch;
            src.b0 = g.b_codes + n0 * pitch;
#pragma unroll
            for (int p = 0; p < G::kPassA; ++p)
                src.a_off[p] = (uint32_t)(row_of(m0 + p * G::kRowsPerPass + (t >> 3), g.M) - m0) * (uint32_t)pitch + (uint32_t)off;
#pragma unroll
            for (int p = 0; p < G::kPassB; ++p)
                src.b_off[p] = (uint32_t)(row_of(n0 + p * G::kRowsPerPass + (t >> 3), g.N) - n0) * (uint32_t)pitch + (uint32_t)off;
            // (whole waves take A's rows or B's: BM and BN are multiples of 64; a wave beyond them loads no scales)
            static_assert(G::BM % 64 == 0 && G::BN % 64 == 0, "a wave's scale rows are one operand's");
            const bool of_a = wave * 64 < G::BM;   // uniform
            const ScaleView v = of_a ? g.as : g.bs;
            const int64_t first = of_a ? m0 : n0, row = row_of(first + t - (of_a ? 0 : G::BM), of_a ? g.M : g.N);
            src.s0 = scale_row(v, first);
            src.s_off = (uint32_t)(scale_row(v, row) - src.s0);
            src.kt_stride = v.kt_stride;
        } else {
#pragma unroll
            for (int p = 0; p < G::kPassA; ++p) src.a[p] = g.a_codes + row_of(m0 + p * G::kRowsPerPass + (t >> 3), g.M) * pitch + off;
#pragma unroll
            for (int p = 0; p < G::kPassB; ++p) src.b[p] = g.b_codes + row_of(n0 + p * G::kRowsPerPass + (t >> 3), g.N) * pitch + off;
            const bool of_a = t < G::BM;   // (threads beyond BM + BN load no scales)
            src.s = of_a ? scale_row(g.as, row_of(m0 + t, g.M)) : scale_row(g.bs, row_of(n0 + t - G::BM, g.N));
            src.kt_stride = of_a ? g.as.kt_stride : g.bs.kt_stride;
        }
    }

    floatx16 acc[G::kUnits];   // tile (i ^ row_flip, j ^ col_flip) of the wave at i NT + j
#pragma unroll
    for (int u = 0; u < G::kUnits; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][r] = 0.0f;

    // While tile kt is multiplied, tile kt + 1 goes from registers to the other LDS stage, tile kt + 2 takes
    // its place in the registers, and the barrier sits in the middle of the wave's last slice, whose
    // fragments are in registers by then: all reads of this tile's stage are done, and the first slice of
    // the next tile is read while the rest is multiplied.
    const int ktiles = (int)((g.K + BK - 1) / BK);
    const int partial = kAnyK ? ktiles - 1 : -1;   // the tile that K cuts
    float ts_a, ts_b;
    auto tensor_scales = [&]() {   // requested behind the first loads, not before them and not when the epilogue needs them
        __builtin_amdgcn_sched_barrier(0);
        ts_a = *g.a_ts;
        ts_b = *g.b_ts;
        __builtin_amdgcn_sched_barrier(0);
    };
    Staged<G> st;
    if constexpr (G::MT == 4) {   // the first two tiles are requested together: one memory latency before the loop, not two
        // (2048 x 2048 x 5632 46.7 -> 44.7 us, 2048 x 2048 x 16384 117 -> 110; the other forms, with two waves per
        // SIMD, lose 1-2 %)
        Staged<G> st0;
        load_tile<G, kAnyK, true>(st0, src, 0, g.K);
        if (ktiles > 1) load_tile<G, kAnyK, false>(st, src, 1, g.K);
        tensor_scales();
        if (partial == 0) finish_tail<G>(st0, 0, g.K);
        store_tile<G>(st0, smem);
    } else {
        load_tile<G, kAnyK, true>(st, src, 0, g.K);
        tensor_scales();
        if (partial == 0) finish_tail<G>(st, 0, g.K);
        store_tile<G>(st, smem);
        if (ktiles > 1) load_tile<G, kAnyK, false>(st, src, 1, g.K);
    }
    __syncthreads();
    const int j0 = kg * G::kSlices;
    RawFrags<G> f0, f1;
    read_slice<G>(f0, smem, j0, wm, kg, li, kb);
    if constexpr (G::MT == 4) {
        Frags<G> x, y;
#pragma unroll
        for (int i = 0; i < 16; ++i) dequant_chunk<G, 0>(x, f0, i);
        // one tile: fc holds its raw slice, x its first fragments; fn takes the next tile's slice
        auto one_tile = [&](int kt, RawFrags<G> &fc, RawFrags<G> &fn) {
            uint8_t *nxt = smem + ((kt + 1) & 1) * G::kStage;
            const bool more = kt + 2 < ktiles;
            if (kt + 1 == partial) finish_tail<G>(st, kt + 1, g.K);
            const TileOffsets o = tile_offsets<kAnyK>(more ? kt + 2 : 0, src.kt_stride, g.K, t & 7);
            uint8_t *dst = nxt + (t >> 3) * 128 + ((t & 7) ^ ((t >> 3) & 7)) * 16;
            auto no_side = [](int) {};
            auto move = [&](int i) {   // piece i of tile kt + 1 to LDS, its register takes tile kt + 2's piece
                if (i < G::kPassA) {
                    *reinterpret_cast<uint4 *>(dst + i * G::kRowsPerPass * 128) = st.a[i];
                    if (more) st.a[i] = load_codes16<G, kAnyK, true>(src, i, o);
                } else if (i < G::kPassA + G::kPassB) {
                    const int p = i - G::kPassA;
                    *reinterpret_cast<uint4 *>(dst + (G::BM + p * G::kRowsPerPass) * 128) = st.b[p];
                    if (more) st.b[p] = load_codes16<G, kAnyK, false>(src, p, o);
                } else if (i == G::kPassA + G::kPassB) {   // (256 threads, 256 rows)
                    *reinterpret_cast<uint4 *>(nxt + (G::BM + G::BN) * 128 + t * 16) = st.s;
                    if (more) st.s = load_scales16<kAnyK>(scales_at(src, o.s));
                }
            };
            const int slot = ((2 * j0 + kb) ^ (li & 7)) * 16, sc = 4 * j0 + 2 * kb;
            const uint8_t *codes = nxt + li * 128 + slot, *scales = nxt + (G::BM + G::BN) * 128 + li * 16 + sc;
            constexpr int kBand = 32 * 128;   // bytes of 32 rows of codes, 8 times those of their scale bytes
            const int flip = G::row_flip(kg) * kBand;   // (uniform)
            auto fetch = [&](int i) {   // (after the last tile: a stale stage, never multiplied)
                if (i < 4) {
                    const int band = (i * kBand) ^ flip;
                    fn.a[i] = *reinterpret_cast<const u32x4 *>(codes + band);
                    fn.sa[i] = *reinterpret_cast<const uint16_t *>(scales + (band >> 3));
                } else if (i < 8) {
                    fn.b[i - 4] = *reinterpret_cast<const u32x4 *>(codes + (G::BM + (i - 4) * 32) * 128);
                    fn.sb[i - 4] = *reinterpret_cast<const uint16_t *>(scales + (G::BM + (i - 4) * 32) * 16);
                }
            };
            mma_step<G, 1>(acc, x, y, fc, move);
            __syncthreads();
            mma_step<G, 2>(acc, y, x, fc, fetch);
            mma_step<G, 3>(acc, x, y, fc, no_side);
            mma_step<G, 0>(acc, y, x, fn, no_side);
        };
        // (an odd tile first: a way out in the middle of the loop makes the compiler spill the accumulators)
        int kt = 0;
        if (ktiles & 1) {
            one_tile(0, f0, f1);
            f0 = f1;
            kt = 1;
        }
        for (; kt < ktiles; kt += 2) {
            one_tile(kt, f0, f1);
            one_tile(kt + 1, f1, f0);
        }
    } else
    for (int kt = 0; kt < ktiles; ++kt) {
        uint8_t *cur = smem + (kt & 1) * G::kStage, *nxt = smem + ((kt + 1) & 1) * G::kStage;
        if (kt + 1 < ktiles) {
            if (kt + 1 == partial) finish_tail<G>(st, kt + 1, g.K);
            store_tile<G>(st, nxt);
            if (kt + 2 < ktiles) load_tile<G, kAnyK, false>(st, src, kt + 2, g.K);
        }
        if (G::kSlices == 2) {
            // (one set of raw fragments: the other block on the compute unit covers their latency)
            mma_first<G>(acc, f0);
            mma_second<G>(acc, f0);
            read_slice<G>(f0, cur, j0 + 1, wm, kg, li, kb);
            mma_first<G>(acc, f0);
            __syncthreads();
            mma_second<G>(acc, f0);
            if (kt + 1 < ktiles) read_slice<G>(f0, nxt, j0, wm, kg, li, kb);
        } else {
            mma_first<G>(acc, f0);
            __syncthreads();
            if (kt + 1 < ktiles) read_slice<G>(f1, nxt, j0, wm, kg, li, kb);
            mma_second<G>(acc, f0);
            f0 = f1;
        }
    }
    __syncthreads();   // the reduction overlays the stages

    const float ts = ts_a * ts_b;
    const int64_t row0 = m0 + wm * 32 * G::MT;
    floatx16 sum[G::kUnits / G::KG];
    uint8_t *const area = reduce_groups<G::WM, G::KG, G::kArea>(acc, sum, smem, kg, wm, lane);
    if constexpr (G::KG == 2) {   // groups finish the first and the last MT / 2 bands
        finish<kBf16Out, G>(sum, area, ts, g, row0 + kg * 32 * G::FM, n0, lane);
    } else {   // groups finish a band each, or (2 x 2) a tile each
        const bool band = G::FN == G::NT;
        finish<kBf16Out, G>(sum, area, ts, g, row0 + (band ? kg : kg >> 1) * 32, n0 + (band ? 0 : kg & 1) * 32, lane);
    }
}

// ---- the 4 x 4 form where gemm_wide_applies -------------------------------------------------------
// As the main kernel: codes and scale bytes go straight from memory to LDS (no staging registers, no LDS writes), four stages of
// a K tile, and the fragment reads are inline assembly with their own waits (the compiler would let them wait for the loads).  A wave has
// its slice of the next K tile in registers before it multiplies the last step of this one, so the barrier that shows the next tile
// frees this tile's stage too: the loads of tile kt + 4 follow it, one every 5 matrix instructions, the 16 reads of tile kt + 1 one every
// 2 (1 to 3 and 3 to 7 are all the same).  us, operands staged through registers : this: 1024 x 4096 x 4096 32.3 : 30.1, 2048 x 2048 x 5632 41.3 :
// 39.0, 2048 x 2048 x 16384 f32 105.1 : 98.2, 2048^3 19.1 : 18.3, 1500 x 2000 x 1024 12.2 : 11.7, 2048 x 2048 x 256 6.8 : 6.8, 2040 x 1999 x 768
// f32 13.7 : 13.7.  A K tile then takes 1.44 to 1.53 us by the box's clock where the main kernel takes 1.34 for as many matrix instructions, which has half the
// operand bytes and 10 LDS reads for each 64, where this has 16.  Copies of the kernel, us, as it is : without its loads behind the first four tiles :
// without its LDS reads : without both: 1024 x 4096 x 4096 31.8 : 29.4 : 27.4 : 25.3, 2048 x 2048 x 16384 105.4 : 94.4 : 81.9 : 75.1, per K tile 1.53 : 1.35 : 1.14 :
// 1.04 (without reads the operands do not change either, which draws less power).
constexpr int kWideStages = 4;
constexpr int64_t kMaxWideK = (int64_t)1 << 23;
constexpr int kLoadEvery = 5, kReadEvery = 2;

struct WideRaw {
    u32x4 a[4], b[4];
    uint32_t sa[4], sb[4];   // two scale bytes each
};

// LDS addresses of a lane's reads of one stage: A's bands in the order the reduction asks for, B's one after the other
struct WideAddr {
    uint32_t a[4], sa[4], b, sb;
};

template <int I>
__device__ __forceinline__ void wide_read_one(WideRaw &f, const WideAddr &r)
{
    constexpr int T = I >> 2;
    if constexpr ((I & 3) == 0) asm volatile("ds_read_b128 %0, %1" : "=v"(f.a[T]) : "v"(r.a[T]));
    else if constexpr ((I & 3) == 1) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.b[T]) : "v"(r.b), "n"(T * 4096));
    else if constexpr ((I & 3) == 2) asm volatile("ds_read_u16 %0, %1" : "=v"(f.sa[T]) : "v"(r.sa[T]));
    else asm volatile("ds_read_u16 %0, %1 offset:%2" : "=v"(f.sb[T]) : "v"(r.sb), "n"(T * 512));
}

template <int... I>
__device__ __forceinline__ void wide_read_all(std::integer_sequence<int, I...>, WideRaw &f, const WideAddr &r)
{
    (wide_read_one<I>(f, r), ...);
}

__device__ __forceinline__ void wide_read_wait(WideRaw &f)
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.a[2]), "+v"(f.a[3]), "+v"(f.b[0]), "+v"(f.b[1]), "+v"(f.b[2]), "+v"(f.b[3]),
                   "+v"(f.sa[0]), "+v"(f.sa[1]), "+v"(f.sa[2]), "+v"(f.sa[3]), "+v"(f.sb[0]), "+v"(f.sb[1]), "+v"(f.sb[2]), "+v"(f.sb[3]));
}

// what a wave loads from: buffer descriptors over the block's rows of A and B and over the scale bytes of the wave's 64 rows (rows beyond the
// matrix, and K tiles beyond the last, read as zeros), and a lane's offsets
struct WideSource {
    uint8_t *a, *b, *s;
    int a_bytes, b_bytes, s_bytes, kt_stride;
    uint32_t codes, row32, scales;
};

__device__ __forceinline__ WideSource wide_source(const SmallArgs &g, int64_t m0, int64_t n0, int wave, int t)
{
    const int64_t pitch = g.K / 2, rows_a = g.M - m0 < 128 ? g.M - m0 : 128, rows_b = g.N - n0 < 128 ? g.N - n0 : 128;
    WideSource w;
    w.a = const_cast<uint8_t *>(g.a_codes) + m0 * pitch;
    w.b = const_cast<uint8_t *>(g.b_codes) + n0 * pitch;
    w.a_bytes = (int)(rows_a * pitch);
    w.b_bytes = (int)(rows_b * pitch);
    // (the piece is chosen so that the LDS image is swizzled; rows of a thread differ by multiples of 32)
    w.codes = (uint32_t)((t >> 3) * pitch) + 16u * (uint32_t)((t & 7) ^ ((t >> 3) & 7));
    w.row32 = (uint32_t)(32 * pitch);
    const bool of_a = wave < 2;   // uniform: waves 0, 1 take the scale bytes of A's rows, 2, 3 of B's
    const ScaleView v = of_a ? g.as : g.bs;
    const int64_t row0 = (of_a ? m0 : n0) + 64 * (wave & 1), left = (of_a ? g.M : g.N) - row0, rows = left < 64 ? left : 64;
    w.s = const_cast<uint8_t *>(scale_row(v, row0));
    // (tiled: a K tile's rows lie side by side, and there is room for 256 of them)
    w.s_bytes = rows <= 0 ? 0 : v.tiled ? (int)((g.K / BK - 1) * 4096 + rows * 16) : (int)(rows * v.row_pitch);
    w.scales = (uint32_t)((t & 63) * (v.tiled ? 16 : (int)v.row_pitch));
    w.kt_stride = (int)v.kt_stride;
    return w;
}

// load I (0..8) of K tile kt: four passes of 32 rows of A's codes, four of B's, the scale bytes
template <int I>
__device__ __forceinline__ void wide_load_one(uint8_t *stage, const WideSource &w, int kt, int ktiles, int wave)
{
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const bool on = kt < ktiles;   // uniform
    if constexpr (I < 8) {
        constexpr int p = I & 3;
        const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(I < 4 ? w.a : w.b, 0, on ? (I < 4 ? w.a_bytes : w.b_bytes) : 0, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(d, (lds_ptr)(stage + (I < 4 ? 0 : 16384) + p * 4096 + wave * 1024), 16, w.codes + p * w.row32, kt * 128, 0, 0);
    } else {
        const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(w.s, 0, on ? w.s_bytes : 0, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(d, (lds_ptr)(stage + 32768 + wave * 1024), 16, w.scales, kt * w.kt_stride, 0, 0);
    }
}

template <int... I>
__device__ __forceinline__ void wide_load_all(std::integer_sequence<int, I...>, uint8_t *stage, const WideSource &w, int kt, int ktiles, int wave)
{
    (wide_load_one<I>(stage, w, kt, ktiles, wave), ...);
}

// step Q (0..3) of a K tile: the reads of the next one, the loads of the fourth after it
template <int Q>
struct WideSide {
    uint8_t *load_stage;
    const WideSource &w;
    int kt, ktiles, wave;
    WideRaw &fn;
    const WideAddr &r;
    template <int I>
    __device__ __forceinline__ void at() const
    {
        constexpr int n = 16 * Q + I;
        static_assert(16 * kReadEvery <= 48 && 3 + 8 * kLoadEvery < 64, "reads before step 3, loads within the tile");
        if constexpr (n % kReadEvery == kReadEvery - 1 && n / kReadEvery < 16) wide_read_one<n / kReadEvery>(fn, r);
        if constexpr (n % kLoadEvery == kLoadEvery / 2 && n / kLoadEvery < 9) wide_load_one<n / kLoadEvery>(load_stage, w, kt, ktiles, wave);
    }
};

template <int I, int D>
__device__ __forceinline__ void wide_dequant(half8_t (&na)[4], half8_t (&nb)[4], WideRaw &f)
{
    constexpr int t = (I >> 1) & 3, h = I & 1;
    if (I < 8) {
        if (D == 0 && h == 0) f.sa[t] = scale_halves(f.sa[t]);
        dequant_half<h, (D >> 1)>(na[t], f.a[t][D], f.sa[t]);
    } else {
        if (D == 0 && h == 0) f.sb[t] = scale_halves(f.sb[t]);
        dequant_half<h, (D >> 1)>(nb[t], f.b[t][D], f.sb[t]);
    }
}

template <int... I>
__device__ __forceinline__ void wide_dequant_all(std::integer_sequence<int, I...>, half8_t (&na)[4], half8_t (&nb)[4], WideRaw &f)
{
    (wide_dequant<I, 0>(na, nb, f), ...);
}

struct WideFrags {
    half8_t a[4], b[4];
};

template <int D, class Side, int... I>
__device__ __forceinline__ void wide_step(std::integer_sequence<int, I...>, floatx16 (&acc)[16], const WideFrags &cu, WideFrags &nx, WideRaw &f, const Side &side)
{
    ((acc[I] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cu.b[I & 3], cu.a[I >> 2], acc[I], 0, 0, 0), side.template at<I>(),
      wide_dequant<I, D>(nx.a, nx.b, f), __builtin_amdgcn_sched_barrier(0)), ...);
}

template <bool kBf16Out>
__global__ __launch_bounds__(256, 1) void gemm_wide_kernel(SmallArgs g0, SmallArgs g1, int n0_blocks)
{
    using G = Geo<4, 4, 1, 4>;
    const bool first = (int)blockIdx.x < n0_blocks;   // uniform
    SmallArgs g = g0;
    if (!first) g = g1;
    extern __shared__ __align__(16) uint8_t smem[];
    const int t = threadIdx.x, lane = t & 63;
    const int kg = __builtin_amdgcn_readfirstlane(t >> 6);   // (a group of waves is one wave)
    const int li = lane & 31, kb = lane >> 5;
    int tm, tn;
    tile_coords((int)blockIdx.x - (first ? 0 : n0_blocks), g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * G::BM, n0 = (int64_t)tn * G::BN;
    const int ktiles = (int)(g.K / BK);
    const WideSource src = wide_source(g, m0, n0, kg, t);
    const std::make_integer_sequence<int, 9> all_loads;
    const std::make_integer_sequence<int, 16> all_reads, all_steps;
    wide_load_all(all_loads, smem, src, 0, ktiles, kg);
    wide_load_all(all_loads, smem + G::kStage, src, 1, ktiles, kg);
    __builtin_amdgcn_sched_barrier(0);
    const float ts_a = *g.a_ts, ts_b = *g.b_ts;
    floatx16 acc[16];   // tile (i ^ row_flip, j ^ col_flip) of the wave at 4 i + j
#pragma unroll
    for (int u = 0; u < 16; ++u) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][r] = 0.0f;
        asm volatile("" : "+a"(acc[u]));
    }
    __builtin_amdgcn_sched_barrier(0);

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const uint32_t codes = (uint32_t)(li * 128 + ((2 * kg + kb) ^ (li & 7)) * 16), scales = (uint32_t)(32768 + li * 16 + 4 * kg + 2 * kb);
    const uint32_t flip = (uint32_t)G::row_flip(kg);   // (uniform)
    auto addresses = [&](int tile) {
        const uint32_t stage = lds0 + (uint32_t)(tile & (kWideStages - 1)) * G::kStage;
        WideAddr r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r.a[i] = codes + (stage + ((uint32_t)i ^ flip) * 4096u);
            r.sa[i] = scales + (stage + ((uint32_t)i ^ flip) * 512u);
        }
        r.b = codes + (stage + 16384u);
        r.sb = scales + (stage + 2048u);
        return r;
    };
    auto barrier = [&]() {   // (s_barrier alone: the waits are written out)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    asm volatile("s_waitcnt vmcnt(9)" ::: "memory");   // tile 0; tile 1 may be under way
    barrier();
    WideRaw f0, f1;
    WideFrags x, y;
    wide_read_all(all_reads, f0, addresses(0));
    wide_load_all(all_loads, smem + 2 * G::kStage, src, 2, ktiles, kg);
    wide_load_all(all_loads, smem + 3 * G::kStage, src, 3, ktiles, kg);
    wide_read_wait(f0);
    wide_dequant_all(all_steps, x.a, x.b, f0);
    // one tile: fc holds its raw slice, x its first fragments; fn takes the next tile's slice (after the last: zeros, never multiplied)
    auto one_tile = [&](int kt, WideRaw &fc, WideRaw &fn) {
        asm volatile("s_waitcnt vmcnt(18)" ::: "memory");   // tile kt + 1, behind it those of tiles kt + 2 and kt + 3
        barrier();
        const WideAddr r = addresses(kt + 1);
        uint8_t *const load_stage = smem + (kt & (kWideStages - 1)) * G::kStage;
        wide_step<1>(all_steps, acc, x, y, fc, WideSide<0>{load_stage, src, kt + kWideStages, ktiles, kg, fn, r});
        wide_step<2>(all_steps, acc, y, x, fc, WideSide<1>{load_stage, src, kt + kWideStages, ktiles, kg, fn, r});
        wide_step<3>(all_steps, acc, x, y, fc, WideSide<2>{load_stage, src, kt + kWideStages, ktiles, kg, fn, r});
        wide_read_wait(fn);
        wide_step<0>(all_steps, acc, y, x, fn, WideSide<3>{load_stage, src, kt + kWideStages, ktiles, kg, fn, r});
    };
    // (an odd tile first: a way out in the middle of the loop makes the compiler spill the accumulators)
    int kt = 0;
    if (ktiles & 1) {
        one_tile(0, f0, f1);
        f0 = f1;
        kt = 1;
    }
    for (; kt < ktiles; kt += 2) {
        one_tile(kt, f0, f1);
        one_tile(kt + 1, f1, f0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the reduction overlays the stages
    __syncthreads();
    floatx16 sum[G::kUnits / G::KG];
    uint8_t *const area = reduce_groups<G::WM, G::KG, G::kArea>(acc, sum, smem, kg, 0, lane);
    finish<kBf16Out, G>(sum, area, ts_a * ts_b, g, m0 + kg * 32, n0, lane);
}

template <auto kKernel>
hipError_t launch_kernel(int blocks, int threads, int lds, const SmallArgs *g, int count, hipStream_t s)
{
    const hipError_t e = allow_dynamic_lds<kKernel>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kKernel, dim3((unsigned)blocks), dim3(threads), lds, s, g[0], g[count - 1], g[0].tiles_m * g[0].tiles_n);
    return hipGetLastError();
}

// direct: gemm_wide_applies to every product
template <bool kBf16Out, class G>
hipError_t launch(SmallArgs *g, int count, bool direct, hipStream_t s)
{
    int blocks = 0;
    for (int i = 0; i < count; ++i) {
        g[i].tiles_m = (int)((g[i].M + G::BM - 1) / G::BM);
        g[i].tiles_n = (int)((g[i].N + G::BN - 1) / G::BN);
        blocks += g[i].tiles_m * g[i].tiles_n;
    }
    if constexpr (G::MT == 4) {
        constexpr int lds = kWideStages * G::kStage > G::kLds ? kWideStages * G::kStage : G::kLds;
        if (direct) return launch_kernel<gemm_wide_kernel<kBf16Out>>(blocks, G::kThreads, lds, g, count, s);
    }
    return g[0].K % BK != 0 ? launch_kernel<gemm_small_kernel<kBf16Out, G, true>>(blocks, G::kThreads, G::kLds, g, count, s)
                            : launch_kernel<gemm_small_kernel<kBf16Out, G, false>>(blocks, G::kThreads, G::kLds, g, count, s);
}

ScaleView view(const qii_nvfp4 &t, bool tiled)
{
    return tiled ? ScaleView{t.scales, t.cols * 16, 4096, 1} : ScaleView{t.scales, t.cols / 16, 16, 0};
}

}  // namespace

// Whether the 4 x 4 form takes a product's operands straight to LDS: whole K tiles, offsets below 2^31, and scale bytes that can be
// loaded 16 at a time, which row-major ones that begin 8 bytes off cannot: those are staged through registers like the codes, us, staged :
// for any K : straight: 2048 x 2048 x 2048 20.2 : 21.8 : 19.1, 1024 x 4096 x 4096 33.0 : 34.7 : 31.3, 2048 x 2048 x 16384 110 : 115 : 104.
bool gemm_wide_applies(const qii_nvfp4 &A, const qii_nvfp4 &B)
{
    return A.cols % BK == 0 && A.cols <= kMaxWideK && ((reinterpret_cast<uintptr_t>(A.scales) | reinterpret_cast<uintptr_t>(B.scales)) & 15) == 0;
}

hipError_t launch_gemm_small(const SmallGemm *c, int count, SmallTile tile, hipStream_t s)
{
    SmallArgs g[2];
    bool direct = true;
    for (int i = 0; i < count; ++i) {
        const qii_nvfp4 &A = *c[i].A, &B = *c[i].B;
        if ((A.cols % BK != 0) != (c[0].A->cols % BK != 0) || c[i].c_is_bf16 != c[0].c_is_bf16 ||
            (tile != kTile128Wide && A.cols > kMaxNarrowK))
            return hipErrorInvalidValue;
        g[i].a_codes = A.codes; g[i].b_codes = B.codes;
        g[i].as = view(A, c[i].a_tiled); g[i].bs = view(B, c[i].b_tiled);
        g[i].a_ts = A.tensor_scale; g[i].b_ts = B.tensor_scale;
        g[i].M = A.rows; g[i].N = B.rows; g[i].K = A.cols;
        g[i].C = c[i].C; g[i].ldc = c[i].ldc; g[i].amax_out = c[i].amax_out;
        direct = direct && gemm_wide_applies(A, B);
    }
    const int bf = c[0].c_is_bf16;
    if (tile == kTile64) return bf ? launch<true, Geo<2, 2, 1, 4>>(g, count, direct, s) : launch<false, Geo<2, 2, 1, 4>>(g, count, direct, s);
    if (tile == kTile128Wide) return bf ? launch<true, Geo<4, 4, 1, 4>>(g, count, direct, s) : launch<false, Geo<4, 4, 1, 4>>(g, count, direct, s);
    return bf ? launch<true, Geo<2, 4, 2, 2>>(g, count, direct, s) : launch<false, Geo<2, 4, 2, 2>>(g, count, direct, s);
}

}  // namespace qii
