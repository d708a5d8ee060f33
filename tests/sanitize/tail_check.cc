// CPU check of the small-tile GEMM kernels' operand addresses (gemm_tail.h): every tile of rows of every length up to five K tiles, by 64-bit row
// addresses and by 32-bit offsets.  Every byte that a thread loads lies in its row, and what it stages is the row's bytes in their
// places, with zeros beyond K.
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <vector>

#define __device__
#define __forceinline__ inline
#include "../../paper_2601_22813_amd/csrc/gemm_tail.h"

struct V { uint32_t x, y, z, w; };

static int bad = 0;
static bool inside(const uint8_t *p, int n, const uint8_t *row, int64_t pitch, const char *what, int64_t K, int kt, int piece)
{
    // (as numbers: nothing is read at a wrong address)
    const intptr_t at = (intptr_t)p - (intptr_t)row;
    if (at >= 0 && at + n <= pitch) return true;
    if (bad++ < 20) printf("K %lld, K tile %d, %s %d: bytes %lld .. %lld of a row of %lld\n", (long long)K, kt, what, piece, (long long)at, (long long)at + n, (long long)pitch);
    return false;
}

template <bool kAnyK>
static void check(int64_t K)
{
    const int rows = 3, ktiles = (int)((K + 255) / 256), partial = kAnyK ? ktiles - 1 : -1;
    const int64_t pitch = K / 2, groups = K / 16;
    std::vector<uint8_t> codes(rows * pitch), scales(rows * groups);
    for (size_t i = 0; i < codes.size(); ++i) codes[i] = (uint8_t)(i * 37 + 11);
    for (size_t i = 0; i < scales.size(); ++i) scales[i] = (uint8_t)(i * 53 + 7);
    for (int kt = 0; kt < ktiles; ++kt)
        for (int r = 0; r < rows; ++r) {
            const uint8_t *row = codes.data() + r * pitch;
            const int tail = (int)(K - kt * 256);
            for (int piece = 0; piece < 8; ++piece) {
                const qii::TileOffsets o = qii::tile_offsets<kAnyK>(kt, 16, K, piece);
                const uint8_t *wide = qii::piece_at(row + 16 * piece, o), *narrow = qii::piece_at(codes.data(), (uint32_t)(r * pitch + 16 * piece), o);
                const int n = kAnyK && K < 32 ? 8 : 16;
                if (!inside(wide, n, row, pitch, "piece", K, kt, piece) || !inside(narrow, n, row, pitch, "piece by offset", K, kt, piece)) continue;
                V v = {0, 0, 0, 0};
                memcpy(n == 8 ? &v.z : &v.x, wide, n);
                if (wide != narrow) ++bad;
                if (kt == partial) qii::finish_piece(v, tail - 32 * piece);
                uint8_t want[16] = {};
                for (int i = 0; i < 16; ++i)
                    if (kt * 128 + piece * 16 + i < pitch) want[i] = row[kt * 128 + piece * 16 + i];
                if (memcmp(&v, want, 16) && bad++ < 20) printf("K %lld, K tile %d, piece %d: wrong bytes\n", (long long)K, kt, piece);
            }
            if (K < 256) continue;   // (rows of fewer than 16 scale bytes are read one by one)
            const uint8_t *srow = scales.data() + r * groups, *p = srow + qii::tile_offsets<kAnyK>(kt, 16, K, 0).s;
            if (!inside(p, 16, srow, groups, "scale bytes", K, kt, 0)) continue;
            V s;
            memcpy(&s, p, 16);
            if (kt == partial) qii::finish_scales(s, tail);
            uint8_t want[16] = {};
            for (int i = 0; i < 16 && kt * 16 + i < groups; ++i) want[i] = srow[kt * 16 + i];
            if (memcmp(&s, want, 16) && bad++ < 20) printf("K %lld, K tile %d: wrong scale bytes\n", (long long)K, kt);
        }
}

int main()
{
    for (int64_t K = 16; K <= 5 * 256; K += 16) K % 256 ? check<true>(K) : check<false>(K);
    if (bad == 0) printf("tail check: ok\n");
    return bad != 0;
}
