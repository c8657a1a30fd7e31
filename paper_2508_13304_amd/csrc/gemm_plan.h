// Rules of the GEMM launches (plain C++, the block order also on the device).
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define DP_HD __host__ __device__
#else
#define DP_HD
#endif

namespace dp {

// How a dense operand's chunks are loaded: element by element (any alignment);
// 16 bytes at a time with guarded element loads at ragged edges (ld a multiple
// of 8 and the matrix 16-byte aligned); or always 16 bytes at a time (no
// chunk straddles the end of k or of the rows either).
enum Vec { kElems, kRagged, kWhole };

// kWhole loads take 32-bit byte offsets from the first element of a block's
// tile, at most 128 rows (k) of ld elements: below this ld the offset
// 2 (127 ld + 127) + 16 stays under 2^32 and the element index under 2^31.  The
// other two forms address with 64 bits.
constexpr int kWholeLd = 1 << 24;

// Whether a dense operand of `rows` rows and K columns (k-contiguous if kc,
// else row-contiguous) can take 16-byte loads.
inline Vec dense_vec(bool kc, int rows, int K, int ld, uintptr_t P)
{
    if (ld % 8 != 0 || (P & 15) != 0) return kElems;
    return (kc ? K : rows) % 8 == 0 && ld < kWholeLd ? kWhole : kRagged;
}

// The blocks of a launch come in groups that share operands (the column tiles
// of a row tile; all tiles of a split-K range), and consecutive blocks go to
// the eight XCDs in turn, each with its own L2.  So group and member are taken
// from the block number such that a group stays on one XCD, and neighbouring
// groups (whose convolution windows overlap) do too.
struct Groups {
    int count, size, per;  // groups, blocks per group, groups per XCD
    Groups(int c, int s) : count(c), size(s), per((c + 7) / 8) {}
    uint64_t blocks() const { return 8ull * (unsigned)per * (unsigned)size; }
    // pass: which of several passes over all groups this block belongs to
    DP_HD bool get(unsigned block, int& group, int& member, int pass = 0) const
    {
        const unsigned xcd = block & 7u, j = (block >> 3) - (unsigned)pass * (unsigned)per * (unsigned)size;
        const unsigned g = j / (unsigned)size;
        member = (int)(j - g * (unsigned)size);
        group = (int)(xcd * (unsigned)per + g);
        return g < (unsigned)per && group < count;
    }
};

// Grid of so many blocks of 256 threads (block = y * grid.x + x; blocks beyond the
// number do nothing): a launch takes less than 2^32 threads along x.
struct Grid {
    unsigned x, y;
};
inline Grid gemm_grid(uint64_t blocks)
{
    constexpr uint64_t row = 1u << 22;  // a multiple of the XCDs' eight
    return blocks <= row ? Grid{(unsigned)blocks, 1u} : Grid{(unsigned)row, (unsigned)((blocks + row - 1) / row)};
}

// The tm x tn tiles of a product's z split-K ranges as blocks.  A group holds the
// column tiles of a row tile (z = 1) or all tiles of a range, in as many equal
// parts as it takes for the XCDs to get about the same number of groups (within
// 5 %): 24 x 40000 x 64, whose one row tile kept seven XCDs idle, 15 us whole and
// 5 in parts.
struct TileMap {
    Groups gr;
    int lg, tn, tiles;  // log2 of the parts; tiles of an undivided group
    bool split;
    static int log2_parts(int units, int tiles)
    {
        int l = 0;
        while (1 << l < tiles && (((int64_t)units << l) + 7) / 8 * 8 > 1.05 * (double)((int64_t)units << l)) ++l;
        return l;
    }
    TileMap(int tm, int tn_, int z)
        : gr(1, 1), lg(0), tn(tn_), tiles(z > 1 ? tm * tn_ : tn_), split(z > 1)
    {
        const int units = z > 1 ? z : tm;
        lg = log2_parts(units, tiles);
        gr = Groups(units << lg, (tiles + (1 << lg) - 1) >> lg);
    }
    DP_HD bool get(unsigned block, int& row, int& col, int& z) const
    {
        int g, t;
        if (!gr.get(block, g, t)) return false;
        const int unit = g >> lg;
        t += (g - (unit << lg)) * gr.size;
        if (t >= tiles) return false;
        row = unit;
        col = t;
        z = 0;
        if (split) {
            z = unit;
            row = t / tn;
            col = t - row * tn;
        }
        return true;
    }
};

}  // namespace dp
