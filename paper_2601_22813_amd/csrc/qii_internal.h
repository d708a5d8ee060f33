// Host-side interfaces between the translation units of libqii.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/qii.h"

namespace qii {

// Some kernels need more dynamic LDS than the default limit; the attribute is set once per kernel
// (the kernel is the template argument: kernels of one signature each have their own flags) and device, not
// per launch (a launch may sit inside a stream capture).
template <auto kKernel>
hipError_t allow_dynamic_lds(int bytes)
{
    constexpr int kMaxDevices = 64;
    static bool done[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < kMaxDevices && done[dev]) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kKernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && dev >= 0 && dev < kMaxDevices) done[dev] = true;
    return e;
}

// Where the quantizer reads its logical R x C matrix from.
//   kind F32 / BF16: element (r, c) = x[r*ld + c]            (transpose == 0)
//                                     x[c*ld + r]            (transpose == 1)
//   kind NVFP4     : element (r, c) = dequantized in[r][c] or in[c][r]; in_cols is the
//                    number of columns of the stored tensor.
enum SourceKind { kSrcF32 = 0, kSrcBF16 = 1, kSrcNVFP4 = 2 };

struct Source {
    int kind;
    int transpose;
    const void *x;           // f32 / bf16 data, or the FP4 codes
    const uint8_t *scales;   // NVFP4 only
    const float *ts;         // NVFP4 only (device scalar)
    int64_t ld;              // elements (f32/bf16) or stored columns (NVFP4)
};

struct QuantizeArgs {
    Source src;
    int64_t R, C;            // logical shape: groups of 16 run along C
    int mode;                // qii_mode
    int rht;                 // 0 or 1
    uint64_t seed_rht, seed_sr;
    const float *amax;       // device scalar: max |rotated tensor|
    uint8_t *codes;
    uint8_t *scales;
    float *tensor_scale;
    // post hoc range alignment only (mode QII_MS_EDEN_PH): the heavy pass writes one f32 per
    // group into tbuf instead of scale bytes and folds the group maxima into the 64 words (256
    // bytes apart, a region of 16 KiB) at amax_accum (nullable: the caller supplies the maximum itself); launch_posthoc_scales finishes
    float *tbuf;
    uint32_t *amax_accum;
    int amax_words = 0;      // != 0: one word per block at amax_accum instead (posthoc_words, requant_blocks); in the other
                             // modes: words at amax whose maximum is the tensor's (absmax_words)
    // a second copy of the scale bytes in the main GEMM kernel's tiled layout (nullable; only where
    // rows_kernels_apply, no rotation, C a multiple of 256; room for R rounded up to 256 rows)
    uint8_t *scales_tiled = nullptr;
    // the scale bytes themselves in that layout (launch_quantize_backward only; C a multiple of 256, room as above)
    bool tiled = false;
};

// One read of a dense matrix producing Q(x) (side r: rows x cols) and Q(x^T) (side c: cols x rows),
// mode QII_MS_EDEN (amax of each rotated tensor supplied) or QII_MS_EDEN_PH (heavy pass: tbuf and
// amax_accum as in QuantizeArgs, per side); quantize_pair.hip
struct PairQuantizeArgs {
    Source src;
    int64_t rows, cols;
    int mode;
    int amax_words;          // QII_MS_EDEN_PH: one word per block ((rows / 128) (cols / 128) of them) per side; QII_MS_EDEN: words at amax, or 0
    struct Side {
        uint64_t seed_rht, seed_sr;
        const float *amax;
        uint8_t *codes;
        uint8_t *scales;
        float *tensor_scale;
        float *tbuf;
        uint32_t *amax_accum;
        bool tiled;          // QII_MS_EDEN: scale bytes in the main GEMM kernel's layout (that side's columns a multiple of 256, room for its rows rounded up)
    } r, c;
};
bool pair_kernel_applies(const Source &src, int64_t rows, int64_t cols);
hipError_t launch_quantize_pair(const PairQuantizeArgs &p, hipStream_t s);

bool absmax_tiles_pay(int64_t rows, int64_t cols);
hipError_t launch_absmax_tiles(const Source &src, int64_t rows, int64_t cols, uint64_t seed_rht_r, float *amax_r, uint64_t seed_rht_c,
                               float *amax_c, hipStream_t s, int words = 0);
int absmax_tiles_words(int64_t rows, int64_t cols, bool both);

// p[i * stride_words] = v for i < count (count <= 256); a kernel, not a memset node, so that the
// calls can be captured in a HIP graph
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int count, int stride_words, hipStream_t s);
hipError_t launch_absmax(const Source &src, int64_t R, int64_t C, int rht, uint64_t seed_rht,
                         float *amax /* must hold 0, or words (absmax_words) words to write */, hipStream_t s, int words = 0);
// One word per block of the abs-max pass over a small tensor, in the 256-byte slot: nothing to clear first (a launch of its own,
// about 2.4 us of a call), 0 where the blocks would be too many or too few for the tensor's size
int absmax_words(const Source &src, int64_t R, int64_t C, int rht);
hipError_t launch_rht(const Source &src, int64_t R, int64_t C, uint64_t seed_rht, float *y,
                      float *amax /* nullable, must hold 0 */, hipStream_t s);
hipError_t launch_quantize(const QuantizeArgs &a, hipStream_t s);
// The scales pass of one to four tensors in one launch.  The maximum is supplied by the caller (one word), or
// that of `words` words left by the heavy pass's blocks, or (words == 0) of its spread running maximum.  tiled (C
// a multiple of 256): the scale bytes go out in the layout the main GEMM kernel reads ([row / 256][C / 256][row %
// 256][16 bytes]; room for the row count rounded up to 256) instead of row-major
struct PosthocScales {
    const float *tbuf, *amax;
    bool supplied;
    int words;
    int64_t R, C;
    uint64_t seed_sr;
    uint8_t *scales;
    float *tensor_scale;
    bool tiled;
};
hipError_t launch_posthoc_scales(const PosthocScales *p, int count, hipStream_t s);
// number of blocks of the heavy pass that launch_quantize would run for this source, when it can leave one
// word per block (at most kMaxBlockWords, 16 KiB); else 0
int posthoc_words(const Source &src, int64_t R, int64_t C);
int rows_blocks(int64_t R, int64_t C);
int rows_per_wave(int64_t R, int64_t C, int mode);   // 4, or 1 where the tensor is small
int cols_blocks(int64_t R, int64_t C);
hipError_t launch_dequantize(const uint8_t *codes, const uint8_t *scales, const float *ts,
                             int64_t rows, int64_t cols, float *y, hipStream_t s);
// tuned kernels for dense sources quantized along their rows (quantize_rows.hip)
bool rows_kernels_apply(const Source &src, int64_t R, int64_t C);
hipError_t launch_absmax_rows(const Source &src, int64_t R, int64_t C, int rht, uint64_t seed_rht,
                              float *amax, hipStream_t s, int words);
int absmax_rows_words(const Source &src, int64_t R, int64_t C, int rht);
hipError_t launch_quantize_rows(const QuantizeArgs &a, hipStream_t s);
// a small tensor (no rotation; amax not needed) whose blocks measure it themselves
bool measures_itself(const QuantizeArgs &q);
hipError_t launch_quantize_small(const QuantizeArgs &q, hipStream_t s);
// Q(X) and Q(W) of a forward pass (no rotation, QII_RTN or QII_RTN_46) in one launch, after one that measures the
// maxima that are not supplied (amax null); words: room for 2 * kForwardMaxWords floats
constexpr int kForwardMaxWords = 1024;
bool forward_quantize_applies(const Source &x, int64_t T, const Source &w, int64_t d_out, int64_t d_in);
hipError_t launch_forward_quantize(const QuantizeArgs q[2], float *words, hipStream_t s);
// tuned kernels for dense sources quantized along their columns (quantize_cols.hip)
bool cols_kernels_apply(const Source &src, int64_t R, int64_t C);
hipError_t launch_absmax_cols(const Source &src, int64_t R, int64_t C, int rht, uint64_t seed_rht,
                              float *amax, hipStream_t s, int words);
int absmax_cols_words(int64_t R, int64_t C);
hipError_t launch_quantize_cols(const QuantizeArgs &a, hipStream_t s);
// a saved NVFP4 tensor quantized along its columns (quantize_requant.hip)
bool requant_kernels_apply(const Source &src, int64_t R, int64_t C);
// (one or two tensors in one launch, quantized in the same mode; requant_blocks: blocks of tensor i of such a launch)
int requant_blocks(const int64_t *R, const int64_t *C, int count, int i);
// words: one word per block at amax (requant_blocks of them, at most kSlotWords), else one word that must hold 0
hipError_t launch_absmax_requant(const Source *src, const int64_t *R, const int64_t *C, int rht, const uint64_t *seed_rht,
                                 float *const *amax, int count, hipStream_t s, int words = 0);
// words that the blocks of the abs-max pass over one such tensor leave: at most 64 (a 256-byte slot), else 0
int requant_amax_words(const Source &src, int64_t R, int64_t C);
hipError_t launch_quantize_requant(const QuantizeArgs *a, int count, hipStream_t s);
// Q(E), Q(E^T) and the re-quantizations q of W and X in one launch (pair_kernel_applies to E, requant_kernels_apply to
// both, all in one mode, the arguments as for the two launches; quantize_backward.hip)
hipError_t launch_quantize_backward(const PairQuantizeArgs &e, const QuantizeArgs q[2], hipStream_t s);
int backward_requant_blocks(int64_t R, int64_t C);   // its blocks for an R x C re-quantization (post hoc scheme)
// ws (nullable): gemm_workspace_bytes(M, N, K) bytes, 16-byte aligned, for the re-tiled scale
// bytes of the fast kernel; without it a slower kernel reads the row-major scales directly
size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K);
// amax_c (nullable): device float that receives max |C| over the values as stored
// pretiled: bit 0 / bit 1 say that A.scales / B.scales already hold the tiled layout (K a multiple
// of 256, see launch_posthoc_scales), bit 2 / bit 3 that A's / B's tiled scale bytes are already in
// their place in ws (QuantizeArgs::scales_tiled); either way that operand's re-tiling is skipped
hipError_t launch_gemm(const qii_nvfp4 &A, const qii_nvfp4 &B, void *C, int c_is_bf16, int64_t ldc,
                       float *amax_c, void *ws, size_t ws_bytes, hipStream_t s, int pretiled = 0);

// whether launch_gemm, given a workspace and tiled scale bytes, would run the main kernel: only then is
// it worth a quantizer's while to write the tiled copy
bool gemm_reads_tiled_scales(const qii_nvfp4 &A, const qii_nvfp4 &B, const void *C, int64_t ldc, int c_is_bf16);
// products by the small-tile kernels (gemm_small.hip), one or two in one launch (with one result type, and K a
// multiple of 256 in both or in neither): any K; each operand's scale bytes row-major or, K a multiple of 256, tiled
enum SmallTile { kTile64, kTile128, kTile128Wide };
constexpr int64_t kMaxNarrowK = (int64_t)1 << 25;   // of kTile64 and kTile128
struct SmallGemm {
    const qii_nvfp4 *A, *B;
    bool a_tiled, b_tiled;
    void *C;
    int c_is_bf16;
    int64_t ldc;
    uint32_t *amax_out;
};
hipError_t launch_gemm_small(const SmallGemm *c, int count, SmallTile tile, hipStream_t s);
bool gemm_wide_applies(const qii_nvfp4 &A, const qii_nvfp4 &B);   // whether kTile128Wide takes its operands straight to LDS
// two products whose operands are both ready: in one launch of a small-tile kernel where that is the faster way, else one
// launch_gemm after the other (arguments as there, no maxima)
struct GemmCall {
    const qii_nvfp4 *A, *B;
    void *C;
    int64_t ldc;
    int pretiled;
};
hipError_t launch_gemm2(const GemmCall c[2], int c_is_bf16, void *ws, size_t ws_bytes, hipStream_t s);

// host-only test aids for the shared last round of the main GEMM kernel (gemm_sharing_map.h):
// plan = {positions run one block per tile, shared tiles, sharing blocks}; the segments of a
// hardware block id as {block number, shared tile, first K tile, K tiles, slot} (returns their
// number, -1 beyond 4); the first and last partial-tile slot the fix-up kernel adds up for a tile
void gemm_sharing_plan(int64_t M, int64_t N, int64_t K, int32_t plan[3]);
int gemm_sharing_segments(int rem, int ktotal, int grid, int block_id, int32_t *out);
void gemm_sharing_tile_slots(int rem, int ktotal, int grid, int lt, int32_t out[2]);
// the kernel that launch_gemm would run: see qii_gemm_route
int gemm_call_route(const qii_nvfp4 &A, const qii_nvfp4 &B, const void *C, int c_is_bf16, int64_t ldc, const void *ws, size_t ws_bytes, int pretiled);
int gemm_route(int64_t M, int64_t N, int64_t K, size_t ws_bytes, int tiled);
int gemm_pair_route(const int64_t M[2], const int64_t N[2], const int64_t K[2], size_t ws_bytes, int tiled);

// sweeps of the hardware conversions and short division sequences against their value-space
// rules; counts[0..7] (device) receive the numbers of mismatches (selftest.hip)
// exploratory non-exact GEMM variants (gemm_inexact.hip); ws as gemm_inexact_workspace_bytes says
size_t gemm_inexact_workspace_bytes(int64_t M, int64_t N, int64_t K, int variant);
hipError_t launch_gemm_inexact(const qii_nvfp4 &A, const qii_nvfp4 &B, void *C, int c_is_bf16, int64_t ldc, int variant,
                               void *ws, hipStream_t s);
hipError_t launch_selftest_conversions(unsigned long long *counts, hipStream_t s);
hipError_t launch_microbench(int kind, void *a, void *b, uint64_t n, int blocks, int iters, hipStream_t s);

}  // namespace qii
