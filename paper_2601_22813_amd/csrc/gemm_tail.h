// Where a K tile's operand bytes are, and the last tile that K cuts, in the small-tile GEMM kernels (gemm_small.hip).  A header of
// its own so that a CPU can check every address and byte.
//
// Rows are 8-byte (codes) and byte (scales) aligned when K is an odd multiple of 16 (kAnyK), so a piece of codes is two loads
// of 8 bytes; the last tile may also end at K, half way through a piece: the pieces at or beyond the end are read as the 16 bytes
// that end with the row, the scale bytes likewise, and finish_tail puts them in their places, with zeros behind, when the
// tile goes to LDS.  So the last tile's loads are those of any other, in the same places between the matrix instructions.
// (As a burst of their own, each scale byte behind its own branch, they cost 1 us: the forward pass of
// 1900 x 1360 -> 2136 28.3 -> 27.6 us.  Both halves of a piece from one address: with an address for each, every K tile of the
// 4 x 4 form took 0.1 us longer.)
#pragma once
#include <stdint.h>

namespace qii {
namespace {

// byte offsets of a tile from a thread's source addresses (which are those of K tile 0)
struct TileOffsets {
    int64_t k;     // uniform: in a row of codes
    int piece;     // of the thread's pieces, beyond that; with the 16 piece_index that a source address holds never negative
    int64_t s;     // in a row of scale bytes
};

// piece_index: of the thread's pieces within a row, 0 .. 7
template <bool kAnyK>
__device__ __forceinline__ TileOffsets tile_offsets(int kt, int64_t kt_stride, int64_t K, int piece_index)
{
    const int64_t k0 = (int64_t)kt * 256;
    TileOffsets o = {k0 / 2, 0, kt * kt_stride};
    if (kAnyK && k0 + 256 > K) {   // uniform
        const int last = (int)(K - k0) / 2 - 16 - 16 * piece_index;   // from this piece to the row's last 16 bytes
        if (last < 0) o.piece = last;
        if (kt > 0) {
            o.s += (K - k0) / 16 - 16;
            o.k -= 16;   // (they may begin 8 bytes before the tile, and 32-bit offsets from a tile's first row are unsigned)
            o.piece += 16;
        } else if (K < 32) {
            o.piece += 8;   // (a row is the second half of such a piece)
        }
    }
    return o;
}

// a piece's address: from the row's own address, or by a 32-bit offset from the block tile's first row (uniform)
__device__ __forceinline__ const uint8_t *piece_at(const uint8_t *piece, const TileOffsets &o) { return piece + (o.k + o.piece); }
__device__ __forceinline__ const uint8_t *piece_at(const uint8_t *row0, uint32_t offset, const TileOffsets &o)
{
    return row0 + o.k + (uint32_t)(offset + (uint32_t)o.piece);
}

// pieces of the last tile as they came -> in their places; left: elements from this piece's first to K
template <class V>
__device__ __forceinline__ void finish_piece(V &v, int left)
{
    if (left == 16) { v.x = v.z; v.y = v.w; }
    if (left <= 0) { v.x = 0u; v.y = 0u; }
    if (left < 32) { v.z = 0u; v.w = 0u; }
}

// the same for a row's scale bytes; tail: elements of the tile, 16 .. 240
template <class V>
__device__ __forceinline__ void finish_scales(V &s, int tail)
{
    const int drop = 8 * (16 - tail / 16);   // bits, 8 .. 120
    uint64_t l = (uint64_t)s.y << 32 | s.x, h = (uint64_t)s.w << 32 | s.z;
    l = drop < 64 ? (l >> drop) | (h << (64 - drop)) : h >> (drop - 64);
    h = drop < 64 ? h >> drop : 0;
    s.x = (uint32_t)l; s.y = (uint32_t)(l >> 32); s.z = (uint32_t)h; s.w = (uint32_t)(h >> 32);
}

}  // namespace
}  // namespace qii
