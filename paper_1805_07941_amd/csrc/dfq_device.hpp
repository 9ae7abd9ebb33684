// Device-side arithmetic shared by every dfq kernel: the power-of-two requantization
// (rescale by alpha_x*alpha_y/alpha_z of Eq. 6 when all scales are powers of two), the
// symmetric clamp of Sec. 2.2, and small wavefront helpers.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dfq {

constexpr int kWave = 64;

// clamp to [-beta_max, beta_max] = [-127, 127]
__device__ __forceinline__ int sat8(int t) { return max(-127, min(127, t)); }

// sat8(v * 2^-s, rounded to nearest, ties to even) for any 32-bit v and any integer s.
//   s <= 0 : exact multiplication, then clamp (|v| is clamped first so the product fits);
//   1..31  : floor shift, then one increment decided from the discarded bits;
//   >= 32  : |v| * 2^-32 <= 1/2 and a tie goes to the even neighbour 0.
__device__ __forceinline__ int requant8(int v, int s)
{
    if (s <= 0) {
        int c = sat8(v);
        int k = -s;
        if (k >= 8) return c == 0 ? 0 : (c > 0 ? 127 : -127);
        return sat8(c << k);
    }
    if (s >= 32) return 0;
    int t = v >> s;                                   // floor
    uint32_t rem = (uint32_t)v & ((1u << s) - 1u);    // v - t*2^s, in [0, 2^s)
    uint32_t half = 1u << (s - 1);
    t += (rem > half || (rem == half && (t & 1))) ? 1 : 0;
    return sat8(t);
}

// Variant for a shift known to lie in [1, 31] (the common case inside conv epilogues).
__device__ __forceinline__ int requant8_rshift(int v, int s, uint32_t mask, uint32_t half)
{
    int t = v >> s;
    uint32_t rem = (uint32_t)v & mask;
    t += (rem > half || (rem == half && (t & 1))) ? 1 : 0;
    return sat8(t);
}

__device__ __forceinline__ uint32_t pack4(int a, int b, int c, int d)
{
    return (uint32_t)(a & 0xff) | ((uint32_t)(b & 0xff) << 8) | ((uint32_t)(c & 0xff) << 16) | ((uint32_t)d << 24);
}

__device__ __forceinline__ int byte_of(uint32_t w, int i)  // sign-extended byte i of w
{
    return (int)(w << (24 - 8 * i)) >> 24;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, kWave));
    return v;
}

// ---- float -> code
__device__ __forceinline__ int quant_one(float x, float scale)
{
    // x * 2^f is exact in float (power-of-two scale) except on overflow, which saturates,
    // and on underflow, which rounds to 0 either way.
    float t = __builtin_rintf(x * scale);  // v_rndne_f32: ties to even
    if (!(t == t)) return 0;               // NaN
    t = fminf(fmaxf(t, -127.0f), 127.0f);
    return (int)t;
}

__device__ __forceinline__ int saturate_i32(float t)
{
    if (!(t == t)) return 0;
    if (t >= 2147483648.0f) return 2147483647;
    if (t <= -2147483648.0f) return -2147483647;
    return (int)t;
}

// x * 2^f rounded to an integer; two exact power-of-two factors, so that a sum of fractional lengths beyond 127 cannot overflow the
// scale itself
__device__ __forceinline__ int quant_i32_one(float x, int f)
{
    return saturate_i32(__builtin_rintf(x * ldexpf(1.0f, f / 2) * ldexpf(1.0f, f - f / 2)));
}

// The largest f <= min(acc_frac, 32) with m <= top * 2^(acc_frac - f), at least -32 (dfq_fmt_from_absmax_i32, dfq_np_frac_from_absmax_u64)
__device__ __forceinline__ int frac_from_int(unsigned long long m, int acc_frac, unsigned long long top)
{
    int gap = 0;
    if (m > top) {
        gap = __clzll((long long)top) - __clzll((long long)m);       // m has that many bits more
        if (m > (top << gap)) gap++;                                 // top << gap has the bits of m: no overflow
    }
    return max(min(acc_frac - gap, 32), -32);
}

}  // namespace dfq
