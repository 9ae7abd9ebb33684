// Codes of the dynamic floating-point formats (Sec. 2.1, Eq. 1-5): float -> code, code -> integer -> base-64 digits.
#pragma once
#include "dfq_device.hpp"

namespace dfq {

struct NpFmt {
    int n, p;
    float scale;      // 2^frac (quantize) or 2^-frac (dequantize)
    float beta_max;   // Eq. 5; p+1 significant bits, exact in float
};

// Nearest representable magnitude, ties to the even significand.  v = |x| * 2^frac is exact in float; below
// 2^(p+1) the representable values are the integers, in [2^(p+k), 2^(p+k+1)) the multiples of 2^k, so the
// value is brought to an integer grid by an exact power-of-two factor, rounded by v_rndne_f32 and scaled back.
__device__ __forceinline__ uint32_t np_quant_one(float x, const NpFmt &f)
{
    float v = x * f.scale;
    if (!(v == v)) return 0u;                                        // NaN
    const float a = fminf(fabsf(v), f.beta_max);
    const int ex = (int)((__float_as_uint(a) >> 23) & 0xffu) - 127;  // floor(log2 a) for a >= 2^-126
    const int k = max(ex - f.p, 0);
    float r = ldexpf(__builtin_rintf(ldexpf(a, -k)), k);
    r = fminf(r, f.beta_max);
    if (r == 0.0f) return 0u;                                        // no negative zero
    const uint32_t bits = __float_as_uint(r);
    const int er = (int)((bits >> 23) & 0xffu) - 127;                // r = 2^er * 1.fraction, at most p fraction bits set
    uint32_t code;
    if (er < f.p) code = (uint32_t)(int)r;                           // subnormal: e = 0, m = r
    else code = ((uint32_t)(er - f.p + 1) << f.p) | ((bits >> (23 - f.p)) & ((1u << f.p) - 1u));
    return code | (v < 0.0f ? (1u << (f.n - 1)) : 0u);
}

// Eq. 2 inverted: the sign-and-magnitude code of a representable integer (8 bits, p significand bits); +0 for 0.
__device__ __forceinline__ unsigned np_code_of(int beta, int p)
{
    const int mag = beta < 0 ? -beta : beta;
    if (mag == 0) return 0u;
    const int msb = 31 - __clz(mag);
    const unsigned code = msb < p ? (unsigned)mag : (((unsigned)(msb - p + 1) << p) | (((unsigned)mag >> (msb - p)) & ((1u << p) - 1u)));
    return code | (beta < 0 ? 0x80u : 0u);
}

// Eq. 2: the integer of a code of the format (8, p)
__device__ __forceinline__ int np_beta_of(unsigned code, int p)
{
    const unsigned m = code & ((1u << p) - 1u);
    const unsigned e = (code >> p) & ((1u << (7 - p)) - 1u);
    const int mag = e ? (int)(((1u << p) + m) << (e - 1)) : (int)m;
    return (code & 0x80u) ? -mag : mag;
}

__device__ __forceinline__ void np_split(int beta, int &h, int &l)
{
    const int mag = beta < 0 ? -beta : beta;
    const int hu = mag >> 6, lu = mag & 63;
    h = beta < 0 ? -hu : hu;
    l = beta < 0 ? -lu : lu;
}

}  // namespace dfq
