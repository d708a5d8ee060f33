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
// Operands are staged through registers (global -> VGPR -> LDS): a tile is small enough for that (at
// most 36 registers), the next tile's loads then stay in flight for a whole tile's time, and a ragged K
// needs no padding of the operands: codes and scales beyond K are staged as zeros.  The scale bytes are
// read row-major or in the tiled layout, whichever the operand has: no re-tiling launch, no workspace.
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

template <auto kKernel>
hipError_t launch_kernel(int blocks, int threads, int lds, const SmallArgs *g, int count, hipStream_t s)
{
    const hipError_t e = allow_dynamic_lds<kKernel>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kKernel, dim3((unsigned)blocks), dim3(threads), lds, s, g[0], g[count - 1], g[0].tiles_m * g[0].tiles_n);
    return hipGetLastError();
}

template <bool kBf16Out, class G>
hipError_t launch(SmallArgs *g, int count, hipStream_t s)
{
    int blocks = 0;
    for (int i = 0; i < count; ++i) {
        g[i].tiles_m = (int)((g[i].M + G::BM - 1) / G::BM);
        g[i].tiles_n = (int)((g[i].N + G::BN - 1) / G::BN);
        blocks += g[i].tiles_m * g[i].tiles_n;
    }
    return g[0].K % BK != 0 ? launch_kernel<gemm_small_kernel<kBf16Out, G, true>>(blocks, G::kThreads, G::kLds, g, count, s)
                            : launch_kernel<gemm_small_kernel<kBf16Out, G, false>>(blocks, G::kThreads, G::kLds, g, count, s);
}

ScaleView view(const qii_nvfp4 &t, bool tiled)
{
    return tiled ? ScaleView{t.scales, t.cols * 16, 4096, 1} : ScaleView{t.scales, t.cols / 16, 16, 0};
}

}  // namespace

hipError_t launch_gemm_small(const SmallGemm *c, int count, SmallTile tile, hipStream_t s)
{
    SmallArgs g[2];
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
    }
    const int bf = c[0].c_is_bf16;
    if (tile == kTile64) return bf ? launch<true, Geo<2, 2, 1, 4>>(g, count, s) : launch<false, Geo<2, 2, 1, 4>>(g, count, s);
    if (tile == kTile128Wide) return bf ? launch<true, Geo<4, 4, 1, 4>>(g, count, s) : launch<false, Geo<4, 4, 1, 4>>(g, count, s);
    return bf ? launch<true, Geo<2, 4, 2, 2>>(g, count, s) : launch<false, Geo<2, 4, 2, 2>>(g, count, s);
}

}  // namespace qii
