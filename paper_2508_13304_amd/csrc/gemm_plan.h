// Host rules of the GEMM launches (plain C++: no device code).
#pragma once

#include <stdint.h>

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

}  // namespace dp
