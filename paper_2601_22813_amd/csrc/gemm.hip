// Block-scaled NVFP4 GEMM of libqii:  C = A_hat * B_hat^T  (paper Sec. 5; both operands
// K-contiguous, one E4M3 scale per 16 elements of K, one f32 scale per tensor).
//
// gfx950's scaled FP4 MFMA takes one power-of-two (E8M0) scale per 32 elements, which
// cannot carry NVFP4's E4M3 scale per 16.  The product e2m1 * e4m3 has at most 6
// significant bits and lies in [2^-10, 2688], so it is EXACT in f16: the kernel keeps
// the raw 4.5-bit data in LDS, dequantizes fragments in registers
// (v_cvt_scalef32_pk_f16_fp4 then one packed f16 multiply by the group scale) and feeds
// v_mfma_f32_32x32x16_f16; every product and the f32 accumulation are those of the
// dequantized operands.  The two tensor scales are applied once in the epilogue.
//
// Three families of kernels share this scheme (price_routes picks one): gemm_kernel_v4, the main one
// (K a multiple of 256, scale bytes re-tiled into a workspace, LDS-direct loads, explicit
// software pipeline), and gemm_kernel_tiles, whose blocks take several of its tiles; gemm_kernel_v2 (K a multiple of 128, no workspace); the small-tile kernels
// of gemm_small.hip (any K that is a multiple of 16, NVFP4's own rule, no workspace).
//
// Tiling of the two kernels here: 256 x 256 block tile, K tile 128 or 256, 4 waves (2 x 2) each owning 128 x 128 =
// 4 x 4 MFMA tiles (256 accumulator registers).  One 32x32x16 MFMA consumes exactly
// one scale group per lane: lanes 0..31 supply k 0..31 of a 64-element K slice and
// lanes 32..63 supply k 32..63, four MFMAs walk the four dwords of a lane's 16 bytes
// (the order of k inside the contraction is free as long as A and B agree).
#include <math.h>
#include <utility>

#include "gemm_common.h"
#include "gemm_sharing_map.h"
#include "qii_device.h"
#include "qii_internal.h"

namespace qii {
namespace {

constexpr int BM = 256, BN = 256, BK = 128;

// 8 FP4 codes (one dword) times one E4M3 scale -> 8 exact f16 values.
// scale16x2 holds the scale byte shifted to f16 position in both halves: as f16 that is
// e4m3 * 2^-8 (subnormals included); the FP4 conversion multiplies by 2^8.
__device__ __forceinline__ half8_t dequant8(uint32_t codes, uint32_t scale16x2)
{
    const half2_t s2 = __builtin_bit_cast(half2_t, scale16x2);
    const half2_t h0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes, 256.0f, 0) * s2;
    const half2_t h1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes, 256.0f, 1) * s2;
    const half2_t h2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes, 256.0f, 2) * s2;
    const half2_t h3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes, 256.0f, 3) * s2;
    half8_t r;
    r[0] = h0[0]; r[1] = h0[1]; r[2] = h1[0]; r[3] = h1[1];
    r[4] = h2[0]; r[5] = h2[1]; r[6] = h3[0]; r[7] = h3[1];
    return r;
}

__device__ __forceinline__ uint32_t scale_pair(uint32_t two_bytes, int which)
{
    const uint32_t b = (two_bytes >> (8 * which)) & 0xFFu;
    return (b << 7) | (b << 23);
}

// The epilogue of a wave's 128 x 128 tile in the main kernel: two bands at a time (bf16) or one (f32), room for two groups, so
// that a group's stores leave while the next one is converted.  (The caller guarantees that nobody reads the stages any more.)
template <bool kBf16Out, bool kStreaming>
__device__ __forceinline__ void store_wave_tile(const floatx16 (&acc)[4][4], uint8_t *smem, float ts, void *Cout, int64_t ldc, int64_t M,
                                                int64_t N, int64_t row0, int64_t col0, int wave, int lane, uint32_t *amax_out)
{
    constexpr int kGroup = kBf16Out ? 2 : 1, kArea = 2 * kGroup * 32 * staging_pitch<kBf16Out, 4>();
    static_assert(4 * kArea <= 144 * 1024, "staging areas fit");
    store_tile<kBf16Out, kStreaming, 4, 4, kGroup, 2 * kGroup>(acc, smem + wave * kArea, ts, Cout, ldc, M, N, row0, col0, lane, amax_out);
}

// ------------------------------------------------------------------------------------------
// Kernel without a workspace (K a multiple of 128).
//  * global -> LDS with global_load_lds (no staging registers, no VALU, no ds_write): each
//    lane fetches one 16-byte piece of a code row (or one dword of scale bytes) and the wave's
//    64 pieces land contiguously in LDS.  The piece a lane fetches is chosen so that the LDS
//    image is XOR-swizzled: row r keeps its 16-byte segment s in slot 4r + (s ^ ((r>>1)&3)),
//    which makes the 128-bit fragment reads of 8 consecutive rows hit 8 different bank groups.
//  * three LDS stages: tile kt+2 streams in while tile kt is multiplied, and the raw
//    fragments of the next 64-wide K slice (also across the tile boundary) are read from LDS
//    one slice ahead, so no LDS latency sits between barriers and matrix instructions.
//  * epilogue through LDS: accumulators are scaled, converted and written to a per-wave
//    LDS tile, then stored as 16-byte pieces of full rows.
constexpr int kStages = 3;
constexpr int kOffA = 0, kOffB = 16384, kOffAs = 32768, kOffBs = 34816, kStage2Bytes = 36864;
// epilogue: one band of staged rows per wave, room for two in f32 where stores do not pause
template <bool kBf16Out, bool kPaced>
struct Smem2 {
    static constexpr int kRoom = kBf16Out || kPaced ? 1 : 2, kArea = kRoom * 32 * staging_pitch<kBf16Out, 4>();
    static constexpr int kBytes = kStages * kStage2Bytes > 4 * kArea ? kStages * kStage2Bytes : 4 * kArea;   // 108 or 132 KiB
};

struct RawFrag {
    uint4 a[4], b[4];
    uint32_t sa[4], sb[4];
};

__device__ __forceinline__ void issue_tile_loads(uint8_t *stage, const uint8_t *a_codes, const uint8_t *a_scales,
                                                 const uint8_t *b_codes, const uint8_t *b_scales, int64_t M,
                                                 int64_t N, int64_t K, int64_t m0, int64_t n0, int64_t k0,
                                                 int wave)
{
    const int t = threadIdx.x;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int row = p * 64 + (t >> 2);
        const int seg = (t & 3) ^ ((row >> 1) & 3);
        int64_t ra = m0 + row, rb = n0 + row;
        ra = ra < M ? ra : M - 1;   // rows beyond the matrix read a valid row; their results are dropped
        rb = rb < N ? rb : N - 1;
        __builtin_amdgcn_global_load_lds(a_codes + ra * (K / 2) + k0 / 2 + 16 * seg,
                                         (__attribute__((address_space(3))) void *)(stage + kOffA + (p * 256 + wave * 64) * 16), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(b_codes + rb * (K / 2) + k0 / 2 + 16 * seg,
                                         (__attribute__((address_space(3))) void *)(stage + kOffB + (p * 256 + wave * 64) * 16), 16, 0, 0);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = (h * 256 + t) >> 1, half = t & 1;
        int64_t ra = m0 + row, rb = n0 + row;
        ra = ra < M ? ra : M - 1;
        rb = rb < N ? rb : N - 1;
        __builtin_amdgcn_global_load_lds(a_scales + ra * (K / 16) + k0 / 16 + 4 * half,
                                         (__attribute__((address_space(3))) void *)(stage + kOffAs + (h * 256 + wave * 64) * 4), 4, 0, 0);
        __builtin_amdgcn_global_load_lds(b_scales + rb * (K / 16) + k0 / 16 + 4 * half,
                                         (__attribute__((address_space(3))) void *)(stage + kOffBs + (h * 256 + wave * 64) * 4), 4, 0, 0);
    }
}

// raw fragments of K slice j (64 elements) of one stage for this lane
__device__ __forceinline__ void read_raw(RawFrag &f, const uint8_t *stage, int j, int wm, int wn, int li, int kb)
{
    const int seg = 2 * j + kb;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int rowa = wm * 128 + t * 32 + li, rowb = wn * 128 + t * 32 + li;
        f.a[t] = *reinterpret_cast<const uint4 *>(stage + kOffA + (rowa * 4 + (seg ^ ((rowa >> 1) & 3))) * 16);
        f.b[t] = *reinterpret_cast<const uint4 *>(stage + kOffB + (rowb * 4 + (seg ^ ((rowb >> 1) & 3))) * 16);
        f.sa[t] = *reinterpret_cast<const uint16_t *>(stage + kOffAs + rowa * 8 + 4 * j + 2 * kb);
        f.sb[t] = *reinterpret_cast<const uint16_t *>(stage + kOffBs + rowb * 8 + 4 * j + 2 * kb);
    }
}

// 64 elements of K for the wave's 4 x 4 MFMA tiles: 4 steps of 16 MFMAs, each step
// dequantizing one dword (8 codes) per fragment
__device__ __forceinline__ void mma_slice(floatx16 (&acc)[4][4], const RawFrag &f)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        half8_t fa[4], fb[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t wa = d == 0 ? f.a[t].x : d == 1 ? f.a[t].y : d == 2 ? f.a[t].z : f.a[t].w;
            const uint32_t wb = d == 0 ? f.b[t].x : d == 1 ? f.b[t].y : d == 2 ? f.b[t].z : f.b[t].w;
            fa[t] = dequant8(wa, scale_pair(f.sa[t], d >> 1));
            fb[t] = dequant8(wb, scale_pair(f.sb[t], d >> 1));
        }
#pragma unroll
        for (int tj = 0; tj < 4; ++tj)   // (columns outside: with rows outside a K tile takes 2.5 % longer)
#pragma unroll
            for (int ti = 0; ti < 4; ++ti)
                acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[tj], fa[ti], acc[ti][tj], 0, 0, 0);   // (B first: store_tile)
    }
}

template <bool kBf16Out, bool kPaced>
__global__ __launch_bounds__(256, 1) void gemm_kernel_v2(const uint8_t *__restrict__ a_codes,
                                                         const uint8_t *__restrict__ a_scales,
                                                         const float *__restrict__ a_ts,
                                                         const uint8_t *__restrict__ b_codes,
                                                         const uint8_t *__restrict__ b_scales,
                                                         const float *__restrict__ b_ts, int64_t M,
                                                         int64_t N, int64_t K, void *__restrict__ Cout,
                                                         int64_t ldc, int tiles_m, int tiles_n, uint32_t *amax_out)
{
    extern __shared__ __align__(16) uint8_t smem[];
    // XCD-aware order: consecutive block ids land on different XCDs (8 of them, each with its
    // own L2), so give every XCD a contiguous run of tiles, walked row-major over (m, n).
    int tile = blockIdx.x;
    const int ntiles = tiles_m * tiles_n;
    if ((ntiles & 7) == 0) tile = (tile & 7) * (ntiles >> 3) + (tile >> 3);
    const int64_t m0 = (int64_t)(tile / tiles_n) * BM, n0 = (int64_t)(tile % tiles_n) * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, kb = lane >> 5;

    floatx16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int ktiles = (int)(K / BK);
    issue_tile_loads(smem, a_codes, a_scales, b_codes, b_scales, M, N, K, m0, n0, 0, wave);
    if (ktiles > 1)
        issue_tile_loads(smem + kStage2Bytes, a_codes, a_scales, b_codes, b_scales, M, N, K, m0, n0, BK, wave);
    __builtin_amdgcn_sched_barrier(0);   // (the tensor scales are requested behind the first loads)
    const float ts_a = *a_ts, ts_b = *b_ts;
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // the raw fragments ping-pong between two register sets: f0 holds K slice 0 of a tile,
    // f1 slice 1; each is refilled from LDS while the other is being multiplied
    RawFrag f0, f1;
    read_raw(f0, smem, 0, wm, wn, li, kb);
    int st_cur = 0;   // stage of tile kt
    for (int kt = 0; kt < ktiles; ++kt) {
        const int st_next = st_cur == kStages - 1 ? 0 : st_cur + 1;
        const int st_load = st_next == kStages - 1 ? 0 : st_next + 1;
        if (kt + 2 < ktiles)
            issue_tile_loads(smem + st_load * kStage2Bytes, a_codes, a_scales, b_codes, b_scales, M, N, K, m0,
                             n0, (int64_t)(kt + 2) * BK, wave);
        read_raw(f1, smem + st_cur * kStage2Bytes, 1, wm, wn, li, kb);
        mma_slice(acc, f0);
        // (after the last tile this reads a stale stage; the values are never used)
        read_raw(f0, smem + st_next * kStage2Bytes, 0, wm, wn, li, kb);
        mma_slice(acc, f1);
        // tile kt+2 (issued a whole tile ago) must have landed before anyone reads it, and
        // everyone must be done with stage st_cur before tile kt+3 overwrites it
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        st_cur = st_next;
    }

    using S = Smem2<kBf16Out, kPaced>;
    store_tile<kBf16Out, true, 4, 4, 1, S::kRoom, kPaced>(acc, smem + wave * S::kArea, ts_a * ts_b, Cout, ldc, M, N, m0 + wm * 128, n0 + wn * 128, lane,
                                                          amax_out);
}


// ------------------------------------------------------------------------------------------
// Main kernel (K a multiple of 256, scale bytes re-tiled into the workspace).
// The operand fetch is what bounds this GEMM once the matrix pipe is fed: with 128-wide K
// tiles every row contributes half a 128-byte line of codes and 8 bytes of a scale line per
// tile, i.e. five times more L2 line requests than useful bytes.  Here a K tile is 256 wide
// (one full line of codes per row) and the scale bytes come from a copy laid out as
// [row tile of 256][K tile of 256][row][16 bytes], so each block reads 4 KiB of contiguous
// scales per operand and tile.  Two LDS stages of 72 KiB; LDS image of the codes: row r keeps
// its 16-byte segment s in slot 8r + (s ^ (r & 7)) (conflict-free 128-bit fragment reads).
constexpr int BK4 = 256;
constexpr int kOff4A = 0, kOff4B = 32768, kOff4As = 65536, kOff4Bs = 69632, kStage4Bytes = 73728;
constexpr int kSmem4 = 2 * kStage4Bytes;   // 144 KiB

// scales[rows][K/16] -> tiled[(rt * (K/256) + ks) * 256 + r][16], one 16-byte piece per thread;
// both operands in one launch (threads [0, na) take A, [na, na + nb) take B).  Rows of the last
// row tile beyond M (or N) are not written and keep whatever the workspace held: they only ever
// scale operand rows beyond the matrix, whose products land in accumulator rows / columns that
// the epilogue never stores (matrix-instruction rows are independent of one another).
__global__ void retile_scales_kernel(const uint8_t *__restrict__ a_scales, uint8_t *__restrict__ a_tiled,
                                     int64_t M, const uint8_t *__restrict__ b_scales,
                                     uint8_t *__restrict__ b_tiled, int64_t N, int64_t K)
{
    const int64_t ksn = K / 256;
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // (row, ks)
    const uint8_t *scales = a_scales;
    uint8_t *tiled = a_tiled;
    if (idx >= M * ksn) {
        idx -= M * ksn;
        if (idx >= N * ksn) return;
        scales = b_scales;
        tiled = b_tiled;
    }
    const int64_t row = idx / ksn, ks = idx % ksn;
    const uint4 v = *reinterpret_cast<const uint4 *>(scales + row * (K / 16) + ks * 16);
    *reinterpret_cast<uint4 *>(tiled + (((row >> 8) * ksn + ks) * 256 + (row & 255)) * 16) = v;
}

// One operand's side of the LDS-direct loads of a block: buffer descriptors over the tile's rows (rows beyond the
// matrix read as zeros) and over its re-tiled scales, and this thread's offset of its 16-byte piece in row t / 8.
struct TileSource {
    uint8_t *codes_base, *scales_base;
    int codes_bytes, scales_bytes;
};

// what a lane adds to them: the offset of its piece in row t / 8, the bytes of 32 rows, the offset of its row's scale bytes
struct LaneOffsets {
    uint32_t voff, row32, scales;
};

__device__ __forceinline__ LaneOffsets lane_offsets(int64_t K, int t)
{
    const int64_t pitch = K / 2;
    // the piece is chosen so that the LDS image is swizzled (rows of a thread differ by multiples of 32)
    return LaneOffsets{(uint32_t)((t >> 3) * pitch) + 16u * (uint32_t)((t & 7) ^ ((t >> 3) & 7)), (uint32_t)(32 * pitch), (uint32_t)t * 16u};
}

__device__ __forceinline__ TileSource tile_source(const uint8_t *codes, const uint8_t *tiled, int64_t row0, int64_t rows_total, int64_t K)
{
    const int64_t left = rows_total - row0, rows = left < BM ? left : BM, pitch = K / 2;
    TileSource o;
    o.codes_base = const_cast<uint8_t *>(codes) + row0 * pitch;
    o.scales_base = const_cast<uint8_t *>(tiled) + (row0 >> 8) * (K * 16);
    o.codes_bytes = (int)(rows * pitch);
    o.scales_bytes = (int)(K * 16);
    return o;
}

// the descriptors; a K tile beyond the last takes empty ones: its loads read nothing
struct TileDescriptors {
    __amdgpu_buffer_rsrc_t ac, as, bc, bs;
};
__device__ __forceinline__ TileDescriptors descriptors(const TileSource &a, const TileSource &b, bool on)
{
    return TileDescriptors{__builtin_amdgcn_make_buffer_rsrc(a.codes_base, 0, on ? a.codes_bytes : 0, 0x00020000),
                           __builtin_amdgcn_make_buffer_rsrc(a.scales_base, 0, on ? a.scales_bytes : 0, 0x00020000),
                           __builtin_amdgcn_make_buffer_rsrc(b.codes_base, 0, on ? b.codes_bytes : 0, 0x00020000),
                           __builtin_amdgcn_make_buffer_rsrc(b.scales_base, 0, on ? b.scales_bytes : 0, 0x00020000)};
}

// load I of the 18 that a thread issues per K tile: 8 code pieces of A, 8 of B, the scales of A and of B.  (The row
// part sits in the vector offset, which the descriptor's bounds check covers; the scalar offset stays inside a row.)
template <int I>
__device__ __forceinline__ void issue_tile_load(uint8_t *stage, const LaneOffsets &l, const TileDescriptors &d, int kt, int wave)
{
    typedef __attribute__((address_space(3))) void *lds_ptr;
    if constexpr (I < 16) {
        constexpr int p = I & 7;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(I < 8 ? d.ac : d.bc, (lds_ptr)(stage + (I < 8 ? kOff4A : kOff4B) + (p * 256 + wave * 64) * 16), 16,
                                                 l.voff + p * l.row32, kt * (BK4 / 2), 0, 0);
    } else {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(I == 16 ? d.as : d.bs, (lds_ptr)(stage + (I == 16 ? kOff4As : kOff4Bs) + (wave * 64) * 16), 16,
                                                 l.scales, kt * 4096, 0, 0);
    }
}

template <int... I>
__device__ __forceinline__ void issue_tile_loads(std::integer_sequence<int, I...>, uint8_t *stage, const LaneOffsets &l, const TileDescriptors &d, int kt, int wave)
{
    (issue_tile_load<I>(stage, l, d, kt, wave), ...);
}

// ---- fragment pipeline of the main kernel -------------------------------------------------
// The compiler makes every LDS read that follows a global_load_lds wait for that load
// (it cannot tell the two LDS regions apart), which would serialise the fetch of the next
// K tile with the multiplication of the current one.  The fragment reads are therefore
// written as inline assembly, with their own wait: a read block only names its
// destination registers, and the matching wait "produces" them for the code that follows.
struct RawFrag4 {
    u32x4 a[4], b[4];       // 32 codes (16 bytes) of K for 4 row blocks of A and of B
};

// the 16 scale bytes that each of a lane's 8 rows has for a whole K tile: one 16-byte read per row and tile (a read of the
// lane's two bytes per row and slice is 64 LDS reads a tile instead of 40)
struct TileScales {
    u32x4 a[4], b[4];
};

// a slice's two scales per row, as two f16 numbers (scale_halves)
struct SliceScales {
    uint32_t a[4], b[4];
};

struct FragAddr {
    uint32_t a, b, sa, sb;  // LDS byte addresses of this lane's row 0 pieces in stage 0
    uint32_t xo[4];         // swizzled 16-byte slot of K slice j, times 16
    uint32_t sel;           // selector of this lane's two bytes among a slice's four
};

__device__ __forceinline__ uint32_t lds_address(uint8_t *smem) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem; }

__device__ __forceinline__ FragAddr frag_addr(uint8_t *smem, int wm, int wn, int li, int kb)
{
    FragAddr fa;
    const uint32_t lds0 = lds_address(smem);
    fa.a = lds0 + kOff4A + (wm * 128 + li) * 128;
    fa.b = lds0 + kOff4B + (wn * 128 + li) * 128;
    fa.sa = lds0 + kOff4As + (wm * 128 + li) * 16;
    fa.sb = lds0 + kOff4Bs + (wn * 128 + li) * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) fa.xo[j] = (uint32_t)(((2 * j + kb) ^ (li & 7)) * 16);
    fa.sel = kb ? kScalesHigh : kScalesLow;
    return fa;
}

// s_barrier alone: every wait that it needs is written out (a fence may wait for stores as well)
__device__ __forceinline__ void block_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// LDS addresses of one slice's reads
struct ReadAddr {
    uint32_t a, b;
};

template <int J>
__device__ __forceinline__ ReadAddr read_addr(const FragAddr &fa, uint32_t stage_off)
{
    return ReadAddr{fa.a + fa.xo[J] + stage_off, fa.b + fa.xo[J] + stage_off};
}

// read I (0..7) of a K slice's codes: rows 32 T (32 * 128 bytes apart), T = I / 2
template <int I>
__device__ __forceinline__ void frag_read_one(RawFrag4 &f, const ReadAddr &r)
{
    constexpr int T = I >> 1;
    if constexpr ((I & 1) == 0) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.a[T]) : "v"(r.a), "n"(T * 4096));
    else asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.b[T]) : "v"(r.b), "n"(T * 4096));
}

// read I (0..7) of a K tile's scale bytes (rows 32 * 16 bytes apart)
template <int I>
__device__ __forceinline__ void scale_read_one(TileScales &f, const FragAddr &fa, uint32_t stage_off)
{
    constexpr int T = I >> 1;
    if constexpr ((I & 1) == 0) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.a[T]) : "v"(fa.sa + stage_off), "n"(T * 512));
    else asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.b[T]) : "v"(fa.sb + stage_off), "n"(T * 512));
}

template <int... I>
__device__ __forceinline__ void frag_read_issue(std::integer_sequence<int, I...>, RawFrag4 &f, const ReadAddr &r)
{
    (frag_read_one<I>(f, r), ...);
}

template <int... I>
__device__ __forceinline__ void scale_read_issue(std::integer_sequence<int, I...>, TileScales &f, const FragAddr &fa, uint32_t stage_off)
{
    (scale_read_one<I>(f, fa, stage_off), ...);
}

// all outstanding LDS reads have landed; ties the registers of f to the wait
__device__ __forceinline__ void frag_read_wait(RawFrag4 &f)
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.a[2]), "+v"(f.a[3]), "+v"(f.b[0]), "+v"(f.b[1]),
                   "+v"(f.b[2]), "+v"(f.b[3]));
}

__device__ __forceinline__ void frag_read_wait(RawFrag4 &f, TileScales &s)
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.a[2]), "+v"(f.a[3]), "+v"(f.b[0]), "+v"(f.b[1]),
                   "+v"(f.b[2]), "+v"(f.b[3]), "+v"(s.a[0]), "+v"(s.a[1]), "+v"(s.a[2]), "+v"(s.a[3]),
                   "+v"(s.b[0]), "+v"(s.b[1]), "+v"(s.b[2]), "+v"(s.b[3]));
}

struct Frags {
    half8_t a[4], b[4];
};

// chunk I (0..15) of the dequantization of dword D of slice J's raw fragments f into nx: fragment I/2
// (0..3 = A, 4..7 = B), half I%2.  The first chunk that touches a fragment of a new slice (dword 0, half 0) first puts the
// lane's two scale bytes of that slice into the two-f16 form.
template <int I, int D, int J>
__device__ __forceinline__ void dequant_chunk(Frags &nx, const RawFrag4 &f, const TileScales &ts, SliceScales &ss, uint32_t sel)
{
    constexpr int t = (I >> 1) & 3, h = I & 1;
    if (I < 8) {
        if (D == 0 && h == 0) ss.a[t] = scale_halves(ts.a[t][J], sel);
        dequant_half<h, (D >> 1)>(nx.a[t], f.a[t][D], ss.a[t]);
    } else {
        if (D == 0 && h == 0) ss.b[t] = scale_halves(ts.b[t][J], sel);
        dequant_half<h, (D >> 1)>(nx.b[t], f.b[t][D], ss.b[t]);
    }
}

template <int J, int... I>
__device__ __forceinline__ void dequant_all(std::integer_sequence<int, I...>, Frags &nx, const RawFrag4 &f, const TileScales &ts, SliceScales &ss, uint32_t sel)
{
    (dequant_chunk<I, 0, J>(nx, f, ts, ss, sel), ...);
}

// One step = 16 matrix instructions on the fragments in cu, with the fragments of the next
// step (dword D of slice J, raw in f) dequantized into nx in between, one chunk per matrix instruction, and the memory
// operations side(I) spread over the step; the scheduling barriers keep that order, so the conversions and
// the issue of the memory operations run in the shadow of the matrix pipe.  (A K tile's 18 loads, with their
// address arithmetic, and 64 LDS reads used to be issued in blocks between the steps, with the matrix pipe idle:
// 16384 x 2048 x 8192 441 -> 412 us, 32768 x 16384 x 2048 1820 -> 1743, 8192^3 827 -> 797 on one box.)
template <int D, int J, class Side>
__device__ __forceinline__ void mma_step(floatx16 (&acc)[4][4], const Frags &cu, Frags &nx, const RawFrag4 &f, const TileScales &ts, SliceScales &ss,
                                         uint32_t sel, const Side &side)
{
#define QII_MMA(I)                                                                                          \
    acc[(I) >> 2][(I) & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cu.b[(I) & 3], cu.a[(I) >> 2],          \
                                                                    acc[(I) >> 2][(I) & 3], 0, 0, 0);                            \
    side.template at<I>();                                                                                  \
    dequant_chunk<I, D, J>(nx, f, ts, ss, sel);                                                             \
    __builtin_amdgcn_sched_barrier(0)
    QII_MMA(0); QII_MMA(1); QII_MMA(2); QII_MMA(3); QII_MMA(4); QII_MMA(5); QII_MMA(6); QII_MMA(7);
    QII_MMA(8); QII_MMA(9); QII_MMA(10); QII_MMA(11); QII_MMA(12); QII_MMA(13); QII_MMA(14); QII_MMA(15);
#undef QII_MMA
}

// The memory operations of a K tile go out one at a time: a load every 3 matrix instructions from the tile's first on, a fragment
// read every 4, a read of scale bytes every 4.  (The address unit takes 16 cycles for a load of 1 KiB, so the four waves' loads after
// every matrix instruction, 32 cycles, waited for one another and the matrix pipe with them.  A load, a read every 1 and 1, 64 reads a
// tile -> 3 and 4, 40 reads: 16384 x 8192 x 2048 400.6 -> 385.4 us, 8192^3 734 -> 714; loads every 2, 4, 6, 8: 387, 388, 387, 389 and 715 to 716.)
constexpr int kLoadEvery = 3, kReadEvery = 4, kScaleEvery = 4;

// step Q (0..15) of a tile: a later tile's loads from matrix instruction kLoadFrom on, and the reads of the slice whose registers are free
template <int Q, int kLoadFrom>
struct TileSide {
    uint8_t *load_stage;
    const LaneOffsets &lanes;
    const TileDescriptors &d;
    int kt, wave;
    RawFrag4 &fe, &fo;
    TileScales &ts;
    const FragAddr &fa;
    uint32_t nxt_off;
    const ReadAddr r[4];   // of the slices 2, 3 of this tile, 0, 1 of the next; r[3] in steps 0 to 2: slice 1 of this one
    template <int I>
    __device__ __forceinline__ void at() const
    {
        constexpr int n = 16 * Q + I;
        constexpr int l = n - kLoadFrom;
        if constexpr (l >= 0 && l % kLoadEvery == 0 && l / kLoadEvery < 18) issue_tile_load<l / kLoadEvery>(load_stage, lanes, d, kt, wave);
        // reads r[g] begin in step 3 + 4 g, one matrix instruction after a load; they must be out before step 7 + 4 g
        constexpr int g = n >= 240 || n < 48 ? 3 : (n - 48) / 64, rel = (n < 48 ? n + 16 : n - 48 - 64 * g) - 1;
        static_assert(1 + 7 * kReadEvery < 64 && 17 * kLoadEvery < 80 && 194 + 7 * kScaleEvery < 240, "before their waits");
        if constexpr (rel >= 0 && rel % kReadEvery == 0 && rel / kReadEvery < 8) {
            constexpr int i = rel / kReadEvery;
            if constexpr ((g & 1) == 0) frag_read_one<i>(fe, r[g]);
            else frag_read_one<i>(fo, r[g]);
        }
        constexpr int s = n - 194;   // (after the step that turns slice 3's scale bytes into numbers)
        if constexpr (s >= 0 && s % kScaleEvery == 0 && s / kScaleEvery < 8) scale_read_one<s / kScaleEvery>(ts, fa, nxt_off);
    }
};

// Launch position -> origin of the output tile (about 32 tiles an XCD works on at once share 4 A panels and
// 8 B panels, 3.5 MiB at K = 2048, instead of 1 + 32).
__device__ __forceinline__ void tile_origin(int pos, int tiles_m, int tiles_n, int64_t &m0, int64_t &n0)
{
    int tm, tn;
    tile_coords(pos, tiles_m, tiles_n, tm, tn);
    m0 = (int64_t)tm * BM;
    n0 = (int64_t)tn * BN;
}

// kStream = false: one block per output tile (launch position blockIdx.x).
// kStream = true: the K tiles of the `sk_rem` tiles from position `sk_base` on form one sequence of
// units (tile-major) that the gridDim.x blocks cut into equal contiguous ranges; a block runs its
// range tile segment by tile segment (at most two when a range is shorter than a tile's K) and
// leaves each segment's unscaled f32 partial tile in slot (block + tile number) of `partial`,
// which streamk_fixup_kernel adds up in a fixed order.  (A separate instantiation: the plain
// kernel keeps its registers.)
template <bool kBf16Out, bool kStream>
__global__ __launch_bounds__(256, 1) void gemm_kernel_v4(const uint8_t *__restrict__ a_codes,
                                                         const uint8_t *__restrict__ a_tiled,
                                                         const float *__restrict__ a_ts,
                                                         const uint8_t *__restrict__ b_codes,
                                                         const uint8_t *__restrict__ b_tiled,
                                                         const float *__restrict__ b_ts, int64_t M,
                                                         int64_t N, int64_t K, void *__restrict__ Cout,
                                                         int64_t ldc, int tiles_m, int tiles_n, uint32_t *amax_out,
                                                         int sk_base, int sk_rem, float *__restrict__ partial)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, kb = lane >> 5;
    float ts_a = 1.0f, ts_b = 1.0f;

    const int ktotal = (int)(K / BK4);
    // this block's range of units [u, u_end) and its number among the blocks (kStream)
    int64_t u = 0, u_end = 0;
    int blk = 0;
    if (kStream) {
        const int G = (int)gridDim.x;
        blk = sharing_block_number((int)blockIdx.x, G);
        sharing_block_units((int64_t)sk_rem * ktotal, G, blk, u, u_end);
    }
    for (;;) {
    // this segment: K tiles [kt0, kt0 + ktiles) of the tile at launch position pos
    int pos = (int)blockIdx.x, kt0 = 0, ktiles = ktotal, lt = 0;
    if (kStream) {
        sharing_segment(u, u_end, ktotal, lt, kt0, ktiles);
        pos = sharing_position(lt, sk_rem, sk_base);
    }
    int64_t m0, n0;
    tile_origin(pos, tiles_m, tiles_n, m0, n0);

    floatx16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const FragAddr fa = frag_addr(smem, wm, wn, li, kb);
    const TileSource src_a = tile_source(a_codes, a_tiled, m0, M, K), src_b = tile_source(b_codes, b_tiled, n0, N, K);
    const std::make_integer_sequence<int, 18> all_loads;
    const std::make_integer_sequence<int, 8> all_reads;
    const std::make_integer_sequence<int, (14 / kReadEvery + 1 < 8 ? 14 / kReadEvery + 1 : 8)> first_reads;   // those of step 15
    const LaneOffsets lanes = lane_offsets(K, threadIdx.x);
    issue_tile_loads(all_loads, smem, lanes, descriptors(src_a, src_b, true), kt0, wave);
    // in the shadow of these loads: the tensor scales (not when the epilogue needs them) and the accumulators' zeros (the
    // compiler would put their 256 writes behind the barrier, 0.5 us of a tile)
    __builtin_amdgcn_sched_barrier(0);
    if (!kStream) {
        ts_a = *a_ts;
        ts_b = *b_ts;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[i][j]));
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // Pipeline over K, in steps of 16 columns of K per lane half (4 steps = one 64-wide slice,
    // 4 slices = one tile).  While step n multiplies, the fragments of step n+1 are dequantized;
    // the raw fragments of slice g live in fe (g even) or fo (g odd) and are re-filled with
    // slice g+2 from step (g, 3) on, once the last conversion of slice g is done; the scale bytes of the next tile are
    // read once slice 3's are numbers.  The hand-over between the two LDS stages sits at
    // step (2, 3) of a tile: this wave's last read of the current stage (slice 3) has landed,
    // so after the barrier tile kt+1, whose loads went out in slice 0 of this tile, is complete in the other
    // stage and the current stage can take tile kt+2.  (Loads in slice 0, not a slice earlier behind the barrier: two
    // and a half slices cover them as well, and a block begins with one tile's loads instead of two, 0.5 us: bf16
    // 4096 x 4096 x 512 20.35 -> 20.09 us, 4096 x 4096 x 1024 31.05 -> 30.78, 8192 x 8192 x 512 72.2 -> 71.3, 2816 x 2048 x
    // 16384 162.9 -> 162.1, one box in turn.)
    RawFrag4 fe, fo;
    TileScales ts;
    SliceScales ss;
    Frags x, y;
    frag_read_issue(all_reads, fe, read_addr<0>(fa, 0));
    scale_read_issue(all_reads, ts, fa, 0);
    frag_read_wait(fe, ts);
    dequant_all<0>(std::make_integer_sequence<int, 16>(), x, fe, ts, ss, fa.sel);
    frag_read_issue(first_reads, fo, read_addr<1>(fa, 0));
    for (int kt = 0; kt < ktiles; ++kt) {
        const uint32_t cur_off = (kt & 1) * kStage4Bytes, nxt_off = ((kt + 1) & 1) * kStage4Bytes;
        const TileDescriptors d = descriptors(src_a, src_b, kt + 1 < ktiles);
        uint8_t *const load_stage = smem + nxt_off;
        const int ld = kt0 + kt + 1;
        const ReadAddr r1 = read_addr<1>(fa, cur_off), r2 = read_addr<2>(fa, cur_off), r3 = read_addr<3>(fa, cur_off), n0r = read_addr<0>(fa, nxt_off), n1r = read_addr<1>(fa, nxt_off);
#define QII_STEP(Q, D, J, CU, NX, F, R3) \
        mma_step<D, J>(acc, CU, NX, F, ts, ss, fa.sel, TileSide<Q, 0>{load_stage, lanes, d, ld, wave, fe, fo, ts, fa, nxt_off, {r2, r3, n0r, R3}})
        // slice 0 (raw: fe)
        QII_STEP(0, 1, 0, x, y, fe, r1);
        QII_STEP(1, 2, 0, y, x, fe, r1);
        QII_STEP(2, 3, 0, x, y, fe, r1);
        frag_read_wait(fo);
        QII_STEP(3, 0, 1, y, x, fo, n1r);
        // slice 1 (raw: fo)
        QII_STEP(4, 1, 1, x, y, fo, n1r);
        QII_STEP(5, 2, 1, y, x, fo, n1r);
        QII_STEP(6, 3, 1, x, y, fo, n1r);
        frag_read_wait(fe);
        QII_STEP(7, 0, 2, y, x, fe, n1r);
        // slice 2 (raw: fe)
        QII_STEP(8, 1, 2, x, y, fe, n1r);
        QII_STEP(9, 2, 2, y, x, fe, n1r);
        QII_STEP(10, 3, 2, x, y, fe, n1r);
        frag_read_wait(fo);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        // (after the last tile the reads fetch a stale stage; the values are never used)
        QII_STEP(11, 0, 3, y, x, fo, n1r);
        // slice 3 (raw: fo)
        QII_STEP(12, 1, 3, x, y, fo, n1r);
        QII_STEP(13, 2, 3, y, x, fo, n1r);
        QII_STEP(14, 3, 3, x, y, fo, n1r);
        frag_read_wait(fe, ts);
        QII_STEP(15, 0, 0, y, x, fe, n1r);
#undef QII_STEP
    }
    // the last read block is still in flight: its registers and the stages are reused below
    frag_read_wait(fo);
    __syncthreads();
    if (!kStream) {
        store_wave_tile<kBf16Out, true>(acc, smem, ts_a * ts_b, Cout, ldc, M, N, m0 + wm * 128, n0 + wn * 128, wave, lane, amax_out);
        break;
    }
    store_wave_tile<false, false>(acc, smem, 1.0f, partial + (int64_t)sharing_slot(blk, lt) * (BM * BN), BN, BM, BN, wm * 128, wn * 128, wave,
                                  lane, nullptr);
    u += ktiles;
    if (u >= u_end) break;
    __syncthreads();   // every wave is done with its staging tile before the next segment's loads land in LDS
    }
}

// maximum over a wave by lane exchanges that need no lane number (one more register kept through the loop)
__device__ __forceinline__ float wave_max_in_registers(float m)
{
    m = fmaxf(m, dpp_f<kDppXor1>(m));
    m = fmaxf(m, dpp_f<kDppXor2>(m));
    m = fmaxf(m, dpp_f<kDppHalfMirror>(m));
    m = fmaxf(m, dpp_f<kDppRor8>(m));
    const auto x = __builtin_amdgcn_permlane16_swap(f2u(m), f2u(m), false, false);
    m = fmaxf(u2f(x[0]), u2f(x[1]));
    const auto y = __builtin_amdgcn_permlane32_swap(f2u(m), f2u(m), false, false);
    return fmaxf(u2f(y[0]), u2f(y[1]));
}

// The epilogue of a block that goes on to another tile: both LDS stages stay with the loads of the K tiles to come, so a wave's
// 128 x 128 entries pass through 4 KiB of their own, 128 bytes of 32 rows at a time (64 columns of bf16, 32 of f32), and leave as
// whole 128-byte lines.  While a round's reads are under way the next round's entries are converted.  LDS operations of a wave run in
// order, so its writes need no wait for the reads before them; they are inline assembly like the fragment reads, because the compiler
// would let them wait for the loads.  16-byte piece s of row r is at slot s ^ (r % 8): neither side has bank conflicts.
// What lies beyond C is dropped by the descriptor.  (Straight from the accumulators, 32 bytes of a row at a time: 2.2 us longer for a tile, and with non-temporal stores 17 to 46.)
constexpr int kStoreArea = 4096;   // LDS bytes per wave

template <bool kBf16Out, bool kMax>
__device__ __forceinline__ void store_rounds(const floatx16 (&acc)[4][4], float ts, __amdgpu_buffer_rsrc_t out, uint32_t rb, int live_cols, int lane,
                                             uint32_t area, float &cmax)
{
    constexpr int esz = kBf16Out ? 2 : 4, kParts = kBf16Out ? 2 : 4, kRounds = 4 * kParts, kCols = 128 / esz, kTiles = kCols / 32;
    const int li = lane & 31, kb = lane >> 5, row = lane >> 3, piece = lane & 7;
    const uint32_t put = area + (uint32_t)(li * 128 + (kBf16Out ? (li & 7) * 16 + 8 * kb : ((li & 7) ^ kb) * 16)), get = area + (uint32_t)(row * 128 + ((piece ^ row) * 16));
    uint32_t voff = (uint32_t)row * rb + (uint32_t)piece * 16u;
    u32x4 v[4];
    uint32_t w[16];   // a round's entries: 16 of f32, 32 of bf16
#pragma unroll
    for (int r = 0; r <= kRounds; ++r) {
        if (r < kRounds) {
#pragma unroll
            for (int t = 0; t < kTiles; ++t) {
                const floatx16 &a = acc[r / kParts][(r % kParts) * kTiles + t];
                float e[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) e[k] = a[k] * ts;
                if (kMax)
#pragma unroll
                    for (int k = 0; k < 16; ++k) cmax = fmaxf(cmax, fabsf(e[k]));
                if (kBf16Out) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) w[8 * t + k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(float2_t{e[2 * k], e[2 * k + 1]}, bf16x2_t));
                } else {
#pragma unroll
                    for (int k = 0; k < 16; ++k) w[k] = f2u(e[k]);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (r > 0) {   // round r - 1 has come back
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
            const int col = ((r - 1) % kParts) * kCols;
            const bool on = col + (piece + 1) * (16 / esz) <= live_cols;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                __builtin_amdgcn_raw_buffer_store_b128(v[p], out, on ? voff + (uint32_t)(8 * p) * rb + (uint32_t)(col * esz) : 0x80000000u, 0, 2 /* nt */);
            if ((r - 1) % kParts == kParts - 1) voff += 32u * rb;
        }
        if (r < kRounds) {
            if (kBf16Out) {
#pragma unroll
                for (int k = 0; k < 8; ++k)   // slot 4 t + q
                    asm volatile("ds_write_b64 %0, %1" ::"v"(put ^ (uint32_t)(16 * k)), "v"(u32x2{w[2 * k], w[2 * k + 1]}));
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)   // slot 2 q + kb
                    asm volatile("ds_write_b128 %0, %1" ::"v"(put ^ (uint32_t)(32 * k)), "v"(u32x4{w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]}));
            }
            asm volatile("ds_read_b128 %0, %1" : "=v"(v[0]) : "v"(get));
            asm volatile("ds_read_b128 %0, %1 offset:1024" : "=v"(v[1]) : "v"(get));
            asm volatile("ds_read_b128 %0, %1 offset:2048" : "=v"(v[2]) : "v"(get));
            asm volatile("ds_read_b128 %0, %1 offset:3072" : "=v"(v[3]) : "v"(get));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ __forceinline__ void zero_tile(floatx16 (&acc)[4][4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t w = 0u;
            asm volatile("" : "+v"(w));   // (or all sixteen are one, copied)
            const half8_t z = __builtin_bit_cast(half8_t, u32x4{w, w, w, w});
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(z, z, floatx16{}, 0, 0, 0);
        }
}

// whether a block may take several tiles: three rounds of them (with two, forward 16384 x 2048 -> 2048 128.6 : 128.2 us, but backward with f32
// gradients 315 to 320 : 319 to 327), C's rows on 128-byte lines and made of whole 16-byte pieces (a round of
// the epilogue that covers two lines in part writes both to memory twice: 8448 x 4104 x 512 bf16 62.8 us instead of 46), a wave's tile within
// 32-bit offsets
static bool blocks_take_tiles(int64_t tiles, const void *C, int64_t ldc, int64_t N, int c_is_bf16)
{
    const int64_t esz = c_is_bf16 ? 2 : 4;
    return tiles >= 768 && ((reinterpret_cast<uintptr_t>(C) | (uintptr_t)(ldc * esz)) & 127) == 0 && N * esz % 16 == 0 && ldc * esz < (1 << 24);
}

// The main kernel where blocks_take_tiles: a block takes the tiles at launch
// positions blockIdx.x, + gridDim.x, ..., and their K tiles are one sequence to its pipeline.  The loads of the K tile after the
// next go out behind the barrier that frees their stage, whichever tile it belongs to, so that a tile begins with its first fragments
// in registers; what is left between two tiles is the epilogue, without its stores' time.  us, a block per tile : this: bf16 32768 x
// 16384 x 2048 1499 : 1460, 16384 x 8192 x 2048 385 : 374, 16384 x 8192 x 512 138 : 127, f32 16384 x 8192 x 1024 258 : 238, 16384 x
// 8192 x 256 123 : 123; long K hides the ends of a tile anyway (8192^3 684 : 685); with one round there is nothing to go on to, and
// the second K tile's loads come first: 4096 x 4096 x 512 19.7 : 20.5.
template <bool kBf16Out, bool kMax>
__global__ __launch_bounds__(256, 1) void gemm_kernel_tiles(const uint8_t *__restrict__ a_codes, const uint8_t *__restrict__ a_tiled,
                                                            const float *__restrict__ a_ts, const uint8_t *__restrict__ b_codes,
                                                            const uint8_t *__restrict__ b_tiled, const float *__restrict__ b_ts, int64_t M,
                                                            int64_t N, int64_t K, void *__restrict__ Cout, int64_t ldc, int tiles_m,
                                                            int tiles_n, int count, uint32_t *amax_out)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, kb = lane >> 5;
    FragAddr fa = frag_addr(smem, wm, wn, li, kb);
    const int ktiles = (int)(K / BK4);

    // what the next loads take: K tile next_kt of the tile at next_pos (nothing behind the block's last tile)
    int pos = (int)blockIdx.x, next_pos = pos, next_kt = 0;
    LaneOffsets lanes = lane_offsets(K, threadIdx.x);
    TileDescriptors d;
    auto aim = [&]() {
        const bool on = next_pos < count;
        int64_t m0, n0;
        tile_origin(on ? next_pos : pos, tiles_m, tiles_n, m0, n0);
        d = descriptors(tile_source(a_codes, a_tiled, m0, M, K), tile_source(b_codes, b_tiled, n0, N, K), on);
    };
    auto advance = [&]() {
        if (++next_kt == ktiles) {
            next_kt = 0;
            next_pos += (int)gridDim.x;
            aim();
        }
    };
    const std::make_integer_sequence<int, 18> all_loads;
    const std::make_integer_sequence<int, 8> all_reads;
    const std::make_integer_sequence<int, (14 / kReadEvery + 1 < 8 ? 14 / kReadEvery + 1 : 8)> first_reads;   // those of step 15
    aim();
    issue_tile_loads(all_loads, smem, lanes, d, 0, wave);
    advance();
    issue_tile_loads(all_loads, smem + kStage4Bytes, lanes, d, next_kt, wave);
    advance();
    __builtin_amdgcn_sched_barrier(0);
    const float ts = u2f((uint32_t)__builtin_amdgcn_readfirstlane((int)f2u((*a_ts) * (*b_ts))));
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(18)" ::: "memory");
    block_barrier();

    floatx16 acc[4][4];
    RawFrag4 fe, fo;
    TileScales sc;
    SliceScales ss;
    Frags x, y;
    frag_read_issue(all_reads, fe, read_addr<0>(fa, 0));
    scale_read_issue(all_reads, sc, fa, 0);
    frag_read_wait(fe, sc);
    dequant_all<0>(std::make_integer_sequence<int, 16>(), x, fe, sc, ss, fa.sel);
    frag_read_issue(first_reads, fo, read_addr<1>(fa, 0));
    uint32_t cmax = 0u;     // (uniform: the wave's largest |entry|; non-negative numbers order like their bits)
    uint32_t cur_off = 0;
    for (;;) {
        int kt = 0;
        zero_tile(acc);
        for (;;) {
            const uint32_t nxt_off = kStage4Bytes - cur_off;
            uint8_t *const load_stage = smem + cur_off;
            const ReadAddr r1 = read_addr<1>(fa, cur_off), r2 = read_addr<2>(fa, cur_off), r3 = read_addr<3>(fa, cur_off), n0r = read_addr<0>(fa, nxt_off), n1r = read_addr<1>(fa, nxt_off);
#define QII_SIDE(Q, R3) TileSide<Q, 176>{load_stage, lanes, d, next_kt, wave, fe, fo, sc, fa, nxt_off, {r2, r3, n0r, R3}}
#define QII_STEP(Q, D, J, CU, NX, F, R3) mma_step<D, J>(acc, CU, NX, F, sc, ss, fa.sel, QII_SIDE(Q, R3))
            // slice 0 (raw: fe)
            QII_STEP(0, 1, 0, x, y, fe, r1);
            QII_STEP(1, 2, 0, y, x, fe, r1);
            QII_STEP(2, 3, 0, x, y, fe, r1);
            frag_read_wait(fo);
            QII_STEP(3, 0, 1, y, x, fo, n1r);
            // slice 1 (raw: fo)
            QII_STEP(4, 1, 1, x, y, fo, n1r);
            QII_STEP(5, 2, 1, y, x, fo, n1r);
            QII_STEP(6, 3, 1, x, y, fo, n1r);
            frag_read_wait(fe);
            QII_STEP(7, 0, 2, y, x, fe, n1r);
            // slice 2 (raw: fe)
            QII_STEP(8, 1, 2, x, y, fe, n1r);
            QII_STEP(9, 2, 2, y, x, fe, n1r);
            QII_STEP(10, 3, 2, x, y, fe, n1r);
            frag_read_wait(fo);
            // the next K tile has landed.  (This waits for a finished tile's stores too; a count that leaves them out is 1 % slower.)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            block_barrier();
            QII_STEP(11, 0, 3, y, x, fo, n1r);
            // slice 3 (raw: fo)
            QII_STEP(12, 1, 3, x, y, fo, n1r);
            QII_STEP(13, 2, 3, y, x, fo, n1r);
            QII_STEP(14, 3, 3, x, y, fo, n1r);
            frag_read_wait(fe, sc);
            QII_STEP(15, 0, 0, y, x, fe, n1r);
#undef QII_STEP
#undef QII_SIDE
            advance();
            cur_off = nxt_off;
            if (++kt == ktiles) break;
        }
        frag_read_wait(fo);   // (no read is in flight while the epilogue needs registers)
        int64_t m0, n0;
        tile_origin(pos, tiles_m, tiles_n, m0, n0);
        const int64_t row0 = m0 + wm * 128, col0 = n0 + wn * 128, rows = M - row0, cols = N - col0;
        const int live_rows = rows < 128 ? (int)rows : 128, live_cols = cols < 128 ? (int)cols : 128;   // (may be negative)
        constexpr int esz = kBf16Out ? 2 : 4;
        const uint32_t rb = (uint32_t)ldc * esz;
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<uint8_t *>(Cout) + (row0 * ldc + col0) * esz, 0,
            live_rows > 0 && live_cols > 0 ? (live_rows - 1) * (int)rb + live_cols * esz : 0, 0x00020000);
        // (The thread's number is formed here, volatile, and the loop's offsets again behind the epilogue: kept, they take each other's
        // registers, and a reload from scratch memory waits for the loads and stores before it.)
        int t;
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(t));
        float tile_max = 0.0f;
        store_rounds<kBf16Out, kMax>(acc, ts, out, rb, live_cols, t, lds_address(smem) + 2 * kStage4Bytes + (uint32_t)wave * kStoreArea, tile_max);
        if (kMax) {
            const uint32_t bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)f2u(wave_max_in_registers(tile_max)));
            cmax = bits > cmax ? bits : cmax;
        }
        pos += (int)gridDim.x;
        if (pos >= count) break;
        lanes = lane_offsets(K, wave * 64 + t);
        fa = frag_addr(smem, wm, wn, t & 31, t >> 5);
        frag_read_issue(first_reads, fo, read_addr<1>(fa, cur_off));   // (again: its registers were the epilogue's)
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (no load is on its way to LDS when the block ends)
    if (kMax) {
        // rounding is monotone: the largest stored value is the rounded largest one
        uint32_t *const waves = reinterpret_cast<uint32_t *>(smem);   // (every load has landed, every read is done)
        block_barrier();
        if (threadIdx.x % 64 == 0) waves[wave] = cmax;
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t a = waves[0] > waves[1] ? waves[0] : waves[1], b = waves[2] > waves[3] ? waves[2] : waves[3], m = a > b ? a : b;
            max_to_global(u2f(kBf16Out ? f32_to_bf16_bits(u2f(m)) << 16 : m), amax_out);
        }
    }
}

// C = (x32_A * x32_B) * sum of a shared tile's partial tiles, in the order of their K ranges.  One
// block per 16 rows of a tile, 4 consecutive columns per thread and pass; the blocks that took part
// in tile lt are those whose unit ranges meet [lt * ktotal, (lt + 1) * ktotal), their slots
// (block + lt) are consecutive.  One atomic per block when max |C| is wanted.
template <bool kBf16Out>
__global__ __launch_bounds__(256) void streamk_fixup_kernel(const float *__restrict__ partial, int sk_base, int sk_rem, int G,
                                                            int ktotal, int tiles_m, int tiles_n, int64_t M, int64_t N,
                                                            const float *__restrict__ a_ts, const float *__restrict__ b_ts,
                                                            void *__restrict__ Cout, int64_t ldc, uint32_t *amax_out)
{
    __shared__ float wave_m[4];
    const int lt = (int)(blockIdx.x >> 4), strip = (int)(blockIdx.x & 15);
    const int64_t U = (int64_t)sk_rem * ktotal;
    const int64_t ufirst = (int64_t)lt * ktotal, ulast = ufirst + ktotal - 1;
    const int b_first = sharing_block_of_unit(ufirst, U, G), b_last = sharing_block_of_unit(ulast, U, G);
    int64_t m0, n0;
    tile_origin(sharing_position(lt, sk_rem, sk_base), tiles_m, tiles_n, m0, n0);
    const float ts = (*a_ts) * (*b_ts);
    float cmax = 0.0f;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int row = strip * 16 + pass * 4 + (int)(threadIdx.x >> 6), col = (int)(threadIdx.x & 63) * 4;
        const float *src = partial + (int64_t)sharing_slot(b_first, lt) * (BM * BN) + row * BN + col;
        float4 acc = *reinterpret_cast<const float4 *>(src);
        for (int b = b_first + 1; b <= b_last; ++b) {
            src += BM * BN;
            const float4 p = *reinterpret_cast<const float4 *>(src);
            acc.x += p.x; acc.y += p.y; acc.z += p.z; acc.w += p.w;
        }
        const int64_t grow = m0 + row, gcol = n0 + col;
        if (grow >= M) continue;
        const float v[4] = {acc.x * ts, acc.y * ts, acc.z * ts, acc.w * ts};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (gcol + e < N) {
                if (kBf16Out) {
                    const uint32_t b = f32_to_bf16_bits(v[e]);
                    reinterpret_cast<uint16_t *>(Cout)[grow * ldc + gcol + e] = (uint16_t)b;
                    cmax = fmaxf(cmax, fabsf(u2f(b << 16)));
                } else {
                    reinterpret_cast<float *>(Cout)[grow * ldc + gcol + e] = v[e];
                    cmax = fmaxf(cmax, fabsf(v[e]));
                }
            }
    }
    if (amax_out) {   // uniform
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, off));
        if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = cmax;
        __syncthreads();
        if (threadIdx.x == 0) atomicMax(amax_out, f2u(fmaxf(fmaxf(wave_m[0], wave_m[1]), fmaxf(wave_m[2], wave_m[3]))));
    }
}

}  // namespace

// The grid of the main kernel runs in rounds of 256 tiles (one block per compute unit).  A last round
// with few tiles leaves most units idle for a whole tile's time (2048 x 2048 x 32768, the weight
// gradient of a small layer, is 64 tiles; 2048 x 11264 is 352: the second round runs at 37 %).  Then
// the full rounds run as they are and the remaining tiles are shared: their K tiles form one sequence
// of units that `grid` blocks (at most 256, at least 4 units each) cut into equal ranges, partial
// tiles go to the workspace and a second kernel adds them up.
//
// The plan follows a model of the whole product's time (microseconds), the one that price_routes compares with the other
// kernels': a round of 256 tiles takes 4.83 per K tile, an incomplete one 4.5 up to 176 tiles and 1.12 more at 256 (the part is
// power-limited: fewer active units run at a higher clock, so filling idle units gains less than their number suggests); every round
// costs 8.57 more for its first loads, its stores and the launch; a shared last round 30.1 (all blocks store their 256 KiB partial
// tiles at the same moment, and the second kernel adds them up) and, per K tile of a block's range, 3.19 plus 2.62 times the share of
// the units that work; 1.31 more where ranges span two tiles.  Sharing is used where the model promises 4 %.  Of 3274
// products that can share, each timed both ways on the present kernel (the model is that of one about 3 % slower), the rule takes the slower way by more
// than 3 % for 93, 9 of them among the 1498 for which this kernel is within 5 % of the fastest.  Measured, us, bf16 results,
// one block per tile : shared: 8448 x 2048 x 3072 122 : 105, 3072 x 2816 x 10240 183 : 154, 8448 x 1024 x 10240 188 : 157,
// 11264 x 2048 x 6144 245 : 223, 18432 x 2048 x 3072 196 : 189, 2816 x 2048 x 16384 273 : 157, 256 x 256 x 32768 475 : 60; not taken, though
// it would pay, 2048 x 5632 x 16384 313 : 288 (176 tiles, where the model sees 301 : 292).
struct StreamPlan {
    int full;   // launch positions run one block per tile
    int rem;    // positions after them whose tiles are shared (0: none)
    int grid;   // blocks that share them
    double us;  // modelled time, without the re-tiling launch
};

// (share = false: one block per tile, as where the workspace has no room for the partial tiles)
static StreamPlan stream_plan(int64_t M, int64_t N, int64_t K, bool share = true)
{
    const int64_t tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN), ktiles = K / BK4;
    const int64_t rounds = tiles / 256, rem = tiles % 256;
    const double full_us = 0.1 + (double)rounds * (4.83 * (double)ktiles + 8.57);
    const double kt_us = 4.5 + (rem > 176 ? 1.12 * (double)(rem - 176) / 80.0 : 0.0);
    const double plain_us = full_us + (rem ? kt_us * (double)ktiles + 8.57 : 0.0);
    StreamPlan plan{(int)tiles, 0, 0, plain_us};
    if (!share || K % BK4 != 0 || tiles == 0 || tiles > (1 << 24) || ktiles < 8 || rem == 0) return plan;
    const int64_t units = rem * ktiles;
    int64_t grid = units / 4 < 256 ? units / 4 : 256;
    if (grid >= 8) grid &= ~(int64_t)7;
    if (grid <= rem) return plan;
    const int64_t per = (units + grid - 1) / grid;
    // ranges that differ in length span two tiles somewhere, but not those of one tile, or of two and an even number of blocks
    const bool one_segment = (ktiles % per == 0 && units % grid == 0) || (rounds == 0 && rem <= 2 && grid % rem == 0);
    const double shared_us = full_us + 30.0 + (3.19 + 2.62 * (double)grid / 256.0) * (double)per + (one_segment ? 0.0 : 1.31);
    if (shared_us >= 0.96 * plain_us) return plan;
    plan.full = (int)(rounds * 256);
    plan.rem = (int)rem;
    plan.grid = (int)grid;
    plan.us = shared_us;
    return plan;
}

static size_t scales_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    const int64_t mp = (M + 255) / 256 * 256, np = (N + 255) / 256 * 256;
    return (size_t)((mp + np) * (K / 16));
}

// where the partial tiles begin: behind the re-tiled scales, 256-byte aligned
static size_t partial_offset(int64_t M, int64_t N, int64_t K) { return (scales_workspace_bytes(M, N, K) + 255) / 256 * 256; }

static size_t plan_bytes(int64_t M, int64_t N, int64_t K, const StreamPlan &plan)
{
    return plan.rem ? partial_offset(M, N, K) + (size_t)(plan.grid + plan.rem) * BM * BN * 4 : scales_workspace_bytes(M, N, K);
}

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    return K % BK4 != 0 ? 0 : plan_bytes(M, N, K, stream_plan(M, N, K));
}

// the plan that a workspace of ws_bytes (at least the scales) has room for
static StreamPlan plan_that_fits(int64_t M, int64_t N, int64_t K, size_t ws_bytes)
{
    const StreamPlan plan = stream_plan(M, N, K);
    return ws_bytes >= plan_bytes(M, N, K, plan) ? plan : stream_plan(M, N, K, false);
}

// test aids (host only): the sharing plan of a shape and the mapping the kernels use
void gemm_sharing_plan(int64_t M, int64_t N, int64_t K, int32_t plan[3])
{
    const StreamPlan p = stream_plan(M, N, K);
    plan[0] = p.full; plan[1] = p.rem; plan[2] = p.grid;
}

int gemm_sharing_segments(int rem, int ktotal, int grid, int block_id, int32_t *out)
{
    const int blk = sharing_block_number(block_id, grid);
    int64_t u, u_end;
    sharing_block_units((int64_t)rem * ktotal, grid, blk, u, u_end);
    int n = 0;
    while (u < u_end && n < 4) {
        int lt, kt0, ktiles;
        sharing_segment(u, u_end, ktotal, lt, kt0, ktiles);
        out[5 * n] = blk; out[5 * n + 1] = lt; out[5 * n + 2] = kt0; out[5 * n + 3] = ktiles; out[5 * n + 4] = sharing_slot(blk, lt);
        u += ktiles;
        ++n;
    }
    return u < u_end ? -1 : n;
}

void gemm_sharing_tile_slots(int rem, int ktotal, int grid, int lt, int32_t out[2])
{
    const int64_t U = (int64_t)rem * ktotal;
    out[0] = sharing_slot(sharing_block_of_unit((int64_t)lt * ktotal, U, grid), lt);
    out[1] = sharing_slot(sharing_block_of_unit((int64_t)lt * ktotal + ktotal - 1, U, grid), lt);
}

template <bool kBf16Out>
static hipError_t launch_main_kernel(const qii_nvfp4 &A, const uint8_t *a_tiled, const qii_nvfp4 &B, const uint8_t *b_tiled, void *C,
                                     int64_t ldc, int tiles_m, int tiles_n, uint32_t *amax_out, const StreamPlan &plan,
                                     float *partial, hipStream_t s)
{
    const int64_t M = A.rows, N = B.rows, K = A.cols;
    hipError_t e = allow_dynamic_lds<gemm_kernel_v4<kBf16Out, false>>(kSmem4);
    if (e != hipSuccess) return e;
    e = allow_dynamic_lds<gemm_kernel_v4<kBf16Out, true>>(kSmem4);
    if (e != hipSuccess) return e;
    if (blocks_take_tiles(plan.full, C, ldc, N, kBf16Out)) {
        constexpr int kLds = kSmem4 + 4 * kStoreArea;   // all of a compute unit's 160 KiB
        auto launch = [&](auto kernel, hipError_t ready) {
            if (ready == hipSuccess)
                hipLaunchKernelGGL(kernel, dim3(256), dim3(256), kLds, s, A.codes, a_tiled, A.tensor_scale,
                                   B.codes, b_tiled, B.tensor_scale, M, N, K, C, ldc, tiles_m, tiles_n, plan.full, amax_out);
            return ready;
        };
        e = amax_out ? launch(gemm_kernel_tiles<kBf16Out, true>, allow_dynamic_lds<gemm_kernel_tiles<kBf16Out, true>>(kLds))
                     : launch(gemm_kernel_tiles<kBf16Out, false>, allow_dynamic_lds<gemm_kernel_tiles<kBf16Out, false>>(kLds));
        if (e != hipSuccess) return e;
    } else if (plan.full > 0)
        hipLaunchKernelGGL((gemm_kernel_v4<kBf16Out, false>), dim3((unsigned)plan.full), dim3(256), kSmem4, s, A.codes, a_tiled,
                           A.tensor_scale, B.codes, b_tiled, B.tensor_scale, M, N, K, C, ldc, tiles_m, tiles_n, amax_out, 0, 0,
                           partial);
    if (plan.rem > 0) {
        hipLaunchKernelGGL((gemm_kernel_v4<kBf16Out, true>), dim3((unsigned)plan.grid), dim3(256), kSmem4, s, A.codes, a_tiled,
                           A.tensor_scale, B.codes, b_tiled, B.tensor_scale, M, N, K, C, ldc, tiles_m, tiles_n, amax_out, plan.full,
                           plan.rem, partial);
        hipLaunchKernelGGL(streamk_fixup_kernel<kBf16Out>, dim3((unsigned)plan.rem * 16), dim3(256), 0, s, partial, plan.full,
                           plan.rem, plan.grid, (int)(K / BK4), tiles_m, tiles_n, M, N, A.tensor_scale, B.tensor_scale, C, ldc,
                           amax_out);
    }
    return hipGetLastError();
}

// Which kernel a product takes: the one whose modelled time (microseconds) is least.  The models are fitted to timings of every kernel, each
// forced in turn (kt = K / 256, b = blocks / 256 compute units): those of the kernels for a ragged K, of 64 x 64 tiles and of 128 x 128 tiles in two
// K groups over 1671 products of M, N = 64 .. 16384 and K = 128 .. 32768, bf16 and f32 results; those of the main kernel and of 128 x 128 tiles in four K
// groups, both for whole K tiles, over 7200 products (1800 of them of at least 180 tiles of 256 x 256).  What the rule takes of these is 0.37 %
// behind the fastest on average, more than 7 % for 128, at most 30 % (13440 x 1016 x 512 f32; rows of C that are not aligned, which no model
// heeds, and K of one or two tiles are the worst); with scale bytes that are tiled already 0.42 %, 178 and 25 %.  Some of them, us, bf16 results, from a
// graph, operands in cache, on one box:
//                         64 x 64   128 x 128 KG 2   128 x 128 (4, 4)   256 x 256 (with re-tiling)
//    256 x  256 x   256        3.9             5.7                7.4       11.1
//    512 x  512 x   512        4.6             7.8                8.5       14.8
//   1024 x 1024 x  4096       16.9            35.9               24.1       41.4 (shared last round)
//   1536 x 1536 x  1536       13.7            16.7               13.8       30.0
//   2048 x 2048 x  2048       23.3            22.8               18.7       38.6
//   2048 x 2048 x 16384      162.3           156.3              102.9      117.6 (shared last round)
//   4096 x 2048 x  1024       23.8            19.5               23.2       26.5
//   4096 x 2048 x  8192      152.5           130.2              107.3      116.8 (shared last round)
//   2048 x 5632 x  2048       56.8            51.9               51.7       46.6
//   4096 x 4096 x  4096      154.5           130.7              117.8       96.0
//   2816 x 2048 x 16384      220.7           236.5              177.5      156.8 (shared last round)
//   8448 x 2048 x  3072      124.3           118.7              112.2      104.4 (shared last round)
//   8192 x 8192 x   256       81.1            57.0              108.8       48.3
// 64 x 64 tiles: up to three blocks run on a unit and their time adds up, so the unit with the most blocks counts.
// 128 x 128 with two K groups: two blocks per unit, so rounds of 512, the last one cheaper the emptier it is, and a block
// beyond the fourth of a unit cheaper, its first loads and stores beside the products of others.
// 128 x 128 with a 4 x 4 wave tile: one block per unit, rounds of 256; a K tile costs less while few units
// work (power); three forms (wide_block_us): K not a multiple of 256 costs it, like the two others, half-width operand loads.  256 x 256: the plan's
// figure, which is that of a slower kernel and about 3 % too long for the present ones, and 4.5 of re-tiling where the scale bytes are not tiled yet (one or
// two shared tiles, main kernel : 64 x 64 tiles: 128 x 128 x 24320 51.6 : 70.4, 256 x 256 x 19456 48.1 : 57.8, 256 x 512 x 22784 56.6 : 67.6); for f32 results
// 1.7 more a round (their stores), and where blocks take several tiles, whose stores leave beside the next tile's products, 4.3 less a round with
// bf16 results and 1.1 less with f32 ones of two K tiles and more (main kernel : 128 x 128 tiles: bf16 8192 x 6144 x 256 37.9 : 42.3, 16384 x 8192 x 256
// 84.5 : 111; f32 27648 x 7936 x 512 forward pass 268 : 317; but without that form, 14848 x 3008 x 512 68.1 : 64.8; f32 and one K tile is memory's time, and the
// one's depends on where C lies, 14592 x 5120 x 256 forward pass 84 to 93 : 84).
// The no-workspace kernel has 128-wide K tiles, so K an odd multiple of 128 costs it no half tile; at K = 128 and
// 384, 64 x 64 : 128 x 128 : it: 2048 x 2048 9.1 : 7.7 : 8.8 and 10.5 : 9.9 : 14.4, 4096 x 4096 25.5 : 18.0 : 12.4
// and 31.6 : 23.9 : 18.9, 8192 x 8192 87 : 59 : 41 and 112 : 84 : 67.
enum Route { kRouteMain, kRouteNoWorkspace, kRoute64, kRoute128, kRoute128Wide };
constexpr int kRouteMainTiles = 5;   // (gemm_call_route)

constexpr int64_t kMaxMainK = (int64_t)1 << 23;

struct Prices {
    double us[5];   // by Route; HUGE_VAL: cannot run
    Route best;
    double blocks64, blocks128, ktiles;
    bool ragged, direct;        // K no multiple of 256; gemm_wide_applies
};

// a block of the 4 x 4 form of 128 x 128 tiles, `blocks` of which run: one per unit
static double wide_block_us(double blocks, double ktiles, bool ragged, bool direct)
{
    const double busy = blocks < 256.0 ? blocks / 256.0 : 1.0;
    return ragged ? 8.78 + (1.63 + 0.262 * busy) * ktiles : direct ? 8.22 + (1.164 + 0.179 * busy) * ktiles : 7.93 + (1.244 + 0.2 * busy) * ktiles;
}

// main_ws: bytes of workspace that the main kernel can use; 0: it cannot run.  direct: gemm_wide_applies.
static Prices price_routes(int64_t M, int64_t N, int64_t K, size_t main_ws, bool retile, bool direct, const void *C, int64_t ldc, int c_is_bf16)
{
    auto count = [&](int64_t tile) { return (double)((M + tile - 1) / tile) * (double)((N + tile - 1) / tile); };
    const bool any = K % BK4 != 0;
    const double kt = (double)((K + BK4 - 1) / BK4), n64 = count(64), n128 = count(128), n256 = count(256);
    const double b64 = n64 > 256.0 ? n64 / 256.0 : 1.0, b = n128 > 256.0 ? n128 / 256.0 : 1.0;
    const double most64 = (double)(int64_t)((n64 + 255.0) / 256.0);
    const double us64 = 4.259 + 0.753 * b64 + (0.236 + 0.531 * most64) * kt * (any ? 1.24 : 1.0);
    const double pairs = (double)(int64_t)(b / 2.0), last = b - 2.0 * pairs;
    const double slope = 3.65 * pairs + (last <= 0.0 ? 0.0 : last <= 1.0 ? 1.49 + 0.55 * last : 2.6 + 0.53 * last);
    const double us128 = 4.45 + (any ? 0.74 : 0.0) + 1.7 * b - 0.79 * (b > 4.0 ? b - 4.0 : 0.0) + slope * kt * (any ? 1.276 : 1.0);
    const double us_wide = (double)(int64_t)((n128 + 255.0) / 256.0) * wide_block_us(n128, kt, any, direct);
    const double full = (double)(int64_t)(n256 / 256.0), rem = n256 - 256.0 * full, rounds256 = full + (rem > 0.0 ? 1.0 : 0.0);
    const double us_v2 = 1.04 * (3.0 + rounds256 * 6.7 + (7.5 * full + (rem > 176.0 ? 6.9 : rem > 0.0 ? 5.9 : 0.0)) * ((double)K / 256.0));
    const bool narrow = K <= kMaxNarrowK;
    Prices p = {{HUGE_VAL, HUGE_VAL, narrow ? us64 : HUGE_VAL, narrow ? us128 : HUGE_VAL, us_wide}, narrow ? kRoute64 : kRoute128Wide, n64, n128, kt, any, direct};
    if (main_ws) {
        const StreamPlan plan = plan_that_fits(M, N, K, main_ws);
        const bool several = blocks_take_tiles(plan.full, C, ldc, N, c_is_bf16);
        const double round_us = c_is_bf16 ? (several ? -4.3 : 0.0) : several && K > BK4 ? -1.1 : 1.7;
        p.us[kRouteMain] = (plan.rem ? 0.981 : 0.97) * plan.us + (retile ? 4.5 : 0.0) + round_us * (double)(plan.full / 256);
    }
    if (!main_ws && K % 128 == 0) p.us[kRouteNoWorkspace] = us_v2;
    for (const Route r : {kRoute128, kRoute128Wide, kRouteMain, kRouteNoWorkspace})
        if (p.us[r] < p.us[p.best]) p.best = r;
    return p;
}

bool gemm_reads_tiled_scales(const qii_nvfp4 &A, const qii_nvfp4 &B, const void *C, int64_t ldc, int c_is_bf16)
{
    const int64_t M = A.rows, N = B.rows, K = A.cols;
    return K % BK4 == 0 && K <= kMaxMainK && M > 0 && N > 0 &&
           price_routes(M, N, K, gemm_workspace_bytes(M, N, K), false, gemm_wide_applies(A, B), C, ldc, c_is_bf16).best == kRouteMain;
}

// whether the main kernel can run, and the prices, for operands and a workspace as launch_gemm has them
static Prices prices_of(const qii_nvfp4 &A, const qii_nvfp4 &B, const void *C, int64_t ldc, int c_is_bf16, const void *ws, size_t ws_bytes, int pretiled)
{
    const int64_t M = A.rows, N = B.rows, K = A.cols;
    // (the re-tiling kernel reads the row-major scale bytes 16 at a time)
    const bool a_ok = (pretiled & 5) || (reinterpret_cast<uintptr_t>(A.scales) & 15) == 0;
    const bool b_ok = (pretiled & 10) || (reinterpret_cast<uintptr_t>(B.scales) & 15) == 0;
    // (K: offsets within a tile's rows stay below 2^31)
    const bool main_ok = K % BK4 == 0 && K <= kMaxMainK && ws && ws_bytes >= scales_workspace_bytes(M, N, K) &&
                         (reinterpret_cast<uintptr_t>(ws) & 15) == 0 && a_ok && b_ok;
    return price_routes(M, N, K, main_ok ? ws_bytes : 0, !(pretiled & 5) || !(pretiled & 10), gemm_wide_applies(A, B), C, ldc, c_is_bf16);
}

// test aid (host only): the kernel that launch_gemm takes, or kRouteMainTiles for the main kernel in the form whose blocks take several tiles
int gemm_call_route(const qii_nvfp4 &A, const qii_nvfp4 &B, const void *C, int c_is_bf16, int64_t ldc, const void *ws, size_t ws_bytes, int pretiled)
{
    const Route best = prices_of(A, B, C, ldc, c_is_bf16, ws, ws_bytes, pretiled).best;
    const bool several = best == kRouteMain && blocks_take_tiles(plan_that_fits(A.rows, B.rows, A.cols, ws_bytes).full, C, ldc, B.rows, c_is_bf16);
    return several ? kRouteMainTiles : (int)best;
}

static Prices test_prices(int64_t M, int64_t N, int64_t K, size_t ws_bytes, int tiled)
{
    const qii_nvfp4 a = {nullptr, nullptr, nullptr, M, K}, b = {nullptr, nullptr, nullptr, N, K};
    // (stand-in addresses, 16-byte aligned scale bytes and a C on a 128-byte line; bf16 results without gaps between the rows)
    return prices_of(a, b, reinterpret_cast<const void *>(256), N, 1, ws_bytes ? reinterpret_cast<const void *>(256) : nullptr, ws_bytes, tiled ? 3 : 0);
}

int gemm_route(int64_t M, int64_t N, int64_t K, size_t ws_bytes, int tiled)
{
    return (int)test_prices(M, N, K, ws_bytes, tiled).best;
}

static SmallTile small_tile(Route route, int64_t K)
{
    return route == kRoute128Wide || K > kMaxNarrowK ? kTile128Wide : route == kRoute64 ? kTile64 : kTile128;
}

// Both products in one launch of kernel r, a's blocks first: as long as all their work spread over the units and part of a last block's way from
// where the others end, as b's blocks one behind a's work, or as one of a's blocks; whichever is the longest.  A block of 64 x 64 or of 128 x 128 tiles
// in two K groups that shares its unit takes less of it (work) than it takes alone.  (The products' own prices are longer for a ragged K, by the last summand.)
static double shared_us(const Prices &a, const Prices &b, Route r)
{
    if (a.us[r] == HUGE_VAL || b.us[r] == HUGE_VAL) return HUGE_VAL;
    const double na = r == kRoute64 ? a.blocks64 : a.blocks128, nb = r == kRoute64 ? b.blocks64 : b.blocks128;
    auto work = [&](const Prices &p) {
        return r == kRoute64    ? 0.99 + 0.59 * p.ktiles * (p.ragged ? 1.043 : 1.0)
               : r == kRoute128 ? 1.8 + 1.9 * p.ktiles
                                : wide_block_us(na + nb, p.ktiles, p.ragged, a.direct && b.direct);
    };
    auto alone = [&](const Prices &p) { return r == kRoute64 ? 0.9 * p.ktiles * (p.ragged ? 1.043 : 1.0) : r == kRoute128 ? 2.51 + 2.84 * p.ktiles : work(p); };
    const double tail = r == kRoute64 ? 0.7 : r == kRoute128 ? 0.56 : 0.33, under_way = r == kRoute64 ? 0.0 : 128.0;
    const double even = (na * work(a) + nb * work(b)) / 256.0 + (na + nb > 256.0 ? tail * alone(b) : 0.0);
    const double behind = (na > under_way ? (na - under_way) * work(a) / 256.0 : 0.0) + alone(b);
    const double longest = behind > alone(a) ? behind : alone(a);
    return (even > longest ? even : longest) + (!a.ragged ? 0.0 : r == kRoute128Wide ? 7.1 : 10.0);
}

// Whether two products whose operands are both ready take one launch of a small-tile kernel: where the modelled time of that launch is
// below those of the products' own routes and what a launch of its own costs the second, 6.6 us.  Returns that kernel, else kRouteMain.  Fitted to 8273 backward
// passes of T, d_in, d_out = 128 .. 16384, each with two launches and with one of each kernel; the choice is 0.31 % of the pass behind the fastest on average, more
// than 5 % for 134, at most 16 % (the products' times in that kernel added up, less a constant each: 1.15 %, 724, 21 %).  Whole passes, us, two
// launches : one of 64 x 64 tiles : of 128 x 128 in two groups : in four: T = 128, 1792 -> 14208 97.2 : 79.7 : 149 : 107, but 17920, 1280 -> 256 (dW's long blocks
// last) 102 : 124 : 182 : 140; 256, 7344 -> 7936 152 : 151 : 129 : 168; 7040, 256 -> 6528 132 : 130 : 125 : 110.
static Route shared_route(const Prices &a, const Prices &b)
{
    Route best = kRouteMain;
    double us = a.us[a.best] + b.us[b.best] + 6.6;
    for (const Route r : {kRoute64, kRoute128, kRoute128Wide}) {
        const double t = shared_us(a, b, r);
        if (t < us) { us = t; best = r; }
    }
    return best;
}

int gemm_pair_route(const int64_t M[2], const int64_t N[2], const int64_t K[2], size_t ws_bytes, int tiled)
{
    if ((K[0] % BK4 != 0) != (K[1] % BK4 != 0)) return -1;
    const Route r = shared_route(test_prices(M[0], N[0], K[0], ws_bytes, tiled && K[0] % BK4 == 0), test_prices(M[1], N[1], K[1], ws_bytes, tiled && K[1] % BK4 == 0));
    return r == kRouteMain ? -1 : (int)r;
}

template <bool kBf16Out, bool kPaced>
static hipError_t launch_no_workspace(const qii_nvfp4 &A, const qii_nvfp4 &B, void *C, int64_t ldc, int tiles_m, int tiles_n, uint32_t *amax_out,
                                      hipStream_t s)
{
    constexpr int lds = Smem2<kBf16Out, kPaced>::kBytes;
    const hipError_t e = allow_dynamic_lds<gemm_kernel_v2<kBf16Out, kPaced>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_kernel_v2<kBf16Out, kPaced>), dim3((unsigned)(tiles_m * tiles_n)), dim3(256), lds, s, A.codes, A.scales, A.tensor_scale,
                       B.codes, B.scales, B.tensor_scale, A.rows, B.rows, A.cols, C, ldc, tiles_m, tiles_n, amax_out);
    return hipGetLastError();
}

hipError_t launch_gemm(const qii_nvfp4 &A, const qii_nvfp4 &B, void *C, int c_is_bf16, int64_t ldc,
                       float *amax_c, void *ws, size_t ws_bytes, hipStream_t s, int pretiled)
{
    const int64_t M = A.rows, N = B.rows, K = A.cols;
    if (pretiled && K % BK4 != 0) return hipErrorInvalidValue;
    uint32_t *amax_out = reinterpret_cast<uint32_t *>(amax_c);
    if (amax_out) {   // the running maximum starts at 0 (a kernel, not a memset node: graph capture)
        const hipError_t e = launch_fill_u32(amax_out, 0u, 1, 1, s);
        if (e != hipSuccess) return e;
    }
    if (M == 0 || N == 0) return hipSuccess;
    const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const Route route = prices_of(A, B, C, ldc, c_is_bf16, ws, ws_bytes, pretiled).best;
    uint8_t *a_ws = reinterpret_cast<uint8_t *>(ws);
    uint8_t *b_ws = a_ws + (M + 255) / 256 * 256 * (K / 16);
    if (route == kRouteMain) {
        const uint8_t *a_tiled = (pretiled & 1) ? A.scales : a_ws;   // (bits 2, 3: a_ws / b_ws are already filled)
        const uint8_t *b_tiled = (pretiled & 2) ? B.scales : b_ws;
        // the tiles of an incomplete last round are shared between blocks when the caller's workspace
        // has room for their partial tiles (behind the scales, 256-byte aligned)
        const StreamPlan plan = plan_that_fits(M, N, K, ws_bytes);
        float *partial = plan.rem ? reinterpret_cast<float *>(reinterpret_cast<uint8_t *>(ws) + partial_offset(M, N, K)) : nullptr;
        // (an operand whose scales arrive tiled takes no part: zero rows)
        const int64_t ma = (pretiled & 5) ? 0 : M, nb_rows = (pretiled & 10) ? 0 : N;
        const int64_t na = ma * (K / 256), nb = nb_rows * (K / 256);
        if (na + nb > 0)
            hipLaunchKernelGGL(retile_scales_kernel, dim3((unsigned)((na + nb + 255) / 256)), dim3(256), 0, s, A.scales,
                               a_ws, ma, B.scales, b_ws, nb_rows, K);
        return c_is_bf16 ? launch_main_kernel<true>(A, a_tiled, B, b_tiled, C, ldc, (int)tiles_m, (int)tiles_n, amax_out, plan, partial, s)
                         : launch_main_kernel<false>(A, a_tiled, B, b_tiled, C, ldc, (int)tiles_m, (int)tiles_n, amax_out, plan, partial, s);
    }
    if (route == kRouteNoWorkspace && !pretiled) {
        if (c_is_bf16) return launch_no_workspace<true, false>(A, B, C, ldc, (int)tiles_m, (int)tiles_n, amax_out, s);
        // A round that fills the GPU just once stores all of its f32 results in one go, and reaches more of the memory's rate
        // when the stores come evenly: with pauses between them.  us, without : with: 256 blocks 4096 x 4096 x 384 24.0 : 23.6, 4096 x
        // 4096 x 128 17.5 : 17.1, 240 blocks 3840 x 4096 x 384 22.9 : 22.7, 224 blocks 3584 x 4096 x 384 21.8 : 21.4; but 208 blocks
        // 3328 x 4096 x 128 14.9 : 14.9, 192 blocks 14.1 : 14.9, and with several rounds, where others multiply
        // meanwhile, 8192 x 8192 x 128 57 : 60.
        return tiles_m * tiles_n >= 224 && tiles_m * tiles_n <= 256
                   ? launch_no_workspace<false, true>(A, B, C, ldc, (int)tiles_m, (int)tiles_n, amax_out, s)
                   : launch_no_workspace<false, false>(A, B, C, ldc, (int)tiles_m, (int)tiles_n, amax_out, s);
    }
    // an operand that is tiled only (bits 0, 1) is read tiled, any other row-major
    const SmallGemm one = {&A, &B, (pretiled & 1) != 0, (pretiled & 2) != 0, C, c_is_bf16, ldc, amax_out};
    return launch_gemm_small(&one, 1, small_tile(route, K), s);
}

hipError_t launch_gemm2(const GemmCall c[2], int c_is_bf16, void *ws, size_t ws_bytes, hipStream_t s)
{
    Prices p[2];
    SmallGemm two[2];
    bool can_share = (c[0].A->cols % BK4 != 0) == (c[1].A->cols % BK4 != 0);
    for (int i = 0; i < 2 && can_share; ++i) {
        if (c[i].A->rows == 0 || c[i].B->rows == 0 || (c[i].pretiled && c[i].A->cols % BK4 != 0)) { can_share = false; break; }
        p[i] = prices_of(*c[i].A, *c[i].B, c[i].C, c[i].ldc, c_is_bf16, ws, ws_bytes, c[i].pretiled);
        two[i] = SmallGemm{c[i].A, c[i].B, (c[i].pretiled & 1) != 0, (c[i].pretiled & 2) != 0, c[i].C, c_is_bf16, c[i].ldc, nullptr};
    }
    const Route shared = can_share ? shared_route(p[0], p[1]) : kRouteMain;
    if (shared != kRouteMain) return launch_gemm_small(two, 2, shared == kRoute64 ? kTile64 : shared == kRoute128 ? kTile128 : kTile128Wide, s);
    for (int i = 0; i < 2; ++i) {
        const hipError_t e = launch_gemm(*c[i].A, *c[i].B, c[i].C, c_is_bf16, c[i].ldc, nullptr, ws, ws_bytes, s, c[i].pretiled);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qii
