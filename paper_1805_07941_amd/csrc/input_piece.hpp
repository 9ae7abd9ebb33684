// Pieces of 16 input bytes that a block of groups reads: the last block may have fewer groups than the others and its last pieces
// begin past the tensor's end.
#pragma once
#include <stdint.h>

namespace dfq {

// By how many bytes a piece from byte b moves down that was read from `from` <= b, the last place where a whole piece fits, or -1: it
// has no byte inside (nor is 128 a shift that a 128-bit number has).
__host__ __device__ inline __attribute__((always_inline)) int piece_move(bool in, uint32_t b, uint32_t from)
{
    return in && b - from < 16u ? (int)(b - from) : -1;
}

}  // namespace dfq
