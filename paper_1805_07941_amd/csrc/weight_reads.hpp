// Runs of weights of any length at any byte, read by whole wide loads that stay inside the tensor: from the run's start, or from the
// last place where the load still fits and shifted down.  One path for all runs: byte loads for the last runs alone were a chain of
// trips to memory that every workgroup waited for.
#pragma once
#include <stdint.h>

namespace dfq {

// `count` weights (at most 16; none if <= 0) from byte o of a tensor of `total` bytes, zeros behind them
__host__ __device__ inline __attribute__((always_inline)) unsigned __int128 weight_piece(const int8_t *w, long long total, long long o, int count)
{
    unsigned __int128 v = 0;
    if (total >= 16) {
        const long long at = o < total - 16 ? o : total - 16;
        __builtin_memcpy(&v, w + at, 16);
        v = o - at < 16 ? v >> (8 * (int)(o - at)) : 0;
    } else {
        for (int e = 0; e < count; e++) v |= (unsigned __int128)(uint8_t)w[o + e] << (8 * e);
    }
    return count <= 0 ? 0 : count < 16 ? v & (((unsigned __int128)1 << (8 * count)) - 1) : v;
}

// 24 bytes from byte o (0 <= o < total) of a tensor of `total` >= 24 bytes, zeros behind its end
__host__ __device__ inline __attribute__((always_inline)) void weight_run24(const int8_t *w, int total, int o, unsigned long long (&q)[3])
{
    const int at = o < total - 24 ? o : total - 24, sh = o - at;
    __builtin_memcpy(q, w + at, 24);
    if (sh >= 16) { q[0] = q[2]; q[1] = q[2] = 0; }
    else if (sh >= 8) { q[0] = q[1]; q[1] = q[2]; q[2] = 0; }
    const int bits = 8 * (sh & 7);
    if (bits) {
        q[0] = q[0] >> bits | q[1] << (64 - bits);
        q[1] = q[1] >> bits | q[2] << (64 - bits);
        q[2] >>= bits;
    }
}

}  // namespace dfq
