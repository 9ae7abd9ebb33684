// Codes of the dynamic floating-point formats (Sec. 2.1, Eq. 1-5): float -> code, code -> integer -> base-64 digits.
#pragma once
#include "dfq_device.hpp"
#include "dfq_host.hpp"

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

// ---- scalar pieces ------------------------------------------------------------------------------------------------

struct NpRound {
    int shift;          // f_x + f_w - f_y
    int p;              // significand bits of the output format
    float beta_max;     // Eq. 5 for the output format (at most 12 bits: exact in float)
    int relu;
};

// The accumulator value v times 2^-shift, rounded to the nearest integer representable with p + 1 significant bits
// (step 1 below 2^(p+1)), ties to the even significand, magnitude clamped to beta_max.  |v| < 2^62.
// The magnitude is first cut to 23 bits with a sticky bit for what was cut (the rounding position is at least 15
// bits above it), which a float holds exactly; the rest is the conversion of a float to the format: scale by an exact
// power of two so that the step becomes 1, round to nearest even, scale back.
__device__ __forceinline__ int np_round_acc(long long v, const NpRound &f)
{
    if (f.relu && v < 0) v = 0;
    const bool neg = v < 0;
    const unsigned long long a = neg ? (unsigned long long)(-v) : (unsigned long long)v;
    const int lz = a ? __clzll((long long)a) : 64;
    const int t = max(41 - lz, 0);                       // bits to cut: the leading bit goes to position 22
    unsigned m = (unsigned)(a >> t);
    if (((unsigned long long)m << t) != a) m |= 1u;      // sticky
    float x = ldexpf((float)m, t - f.shift);
    x = fminf(x, f.beta_max);
    const int ex = (int)((__float_as_uint(x) >> 23) & 0xffu) - 127;
    const int k = max(ex - f.p, 0);
    float r = ldexpf(__builtin_rintf(ldexpf(x, -k)), k);
    r = fminf(r, f.beta_max);
    const int beta = (int)r;
    return neg ? -beta : beta;
}

// The same rounding for the matrix-core kernel's epilogue when 7 <= shift <= 36, through the double-precision adder.  The
// accumulator is V = 64 * T + c with T and c int32 (|V| < 2^37): a double holds it exactly.  With e the binade of |V| the
// result's step is 2^(e' - p) in units of V, e' = max(e, p + shift) (below 2^(p+1) output units the step is one unit).
// Adding M = 1.5 * 2^(e' + 52 - p) puts V into a binade whose unit in the last place is exactly that step, so the adder's
// own round-to-nearest-even does the rounding (M is an even multiple of the step: the parity of the sum's last bit is the
// parity of the quotient q = round(V / step), i.e. of the significand field), and q is the low word of the sum's bit
// pattern (the mantissa field holds 2^51 + q).  The result is q * 2^k, k = e' - p - shift.  Values beyond every format
// of this path (e' capped at p + shift + 11 - p: at least 2^12 output units) still give a q * 2^k >= 2^12 that fits 31
// bits because shift >= 7, and the clamp that follows cuts them.  Returns the signed integer before the clamp.
struct NpFast {
    unsigned base_b;     // biased exponent of the smallest e': 1023 + p + shift
    unsigned top_b;      // base_b + 11 - p
    unsigned m_const;    // ((52 - p) << 20) | 0x80000: exponent offset and the mantissa bit of the factor 1.5
    int bmax;
};

__device__ __forceinline__ int np_round_fast(int T, int c, const NpFast &f)
{
    const double x = __builtin_fma((double)T, 64.0, (double)c);
    const unsigned e_b = __builtin_amdgcn_ubfe((unsigned)__double2hiint(x), 20u, 11u);
    unsigned eb;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(eb) : "v"(e_b), "s"(f.base_b), "v"(f.top_b));      // clamp to [base_b, top_b]
    const double M = __hiloint2double((int)((eb << 20) + f.m_const), 0);
    const int q = __double2loint(x + M);
    return q << (eb - f.base_b);
}

// The conversion of a 32-bit sum t (|t| < 2^30) times 2^-shift, 0 <= shift <= 31, by the same device: (double)t is exact.
__device__ __forceinline__ int np_round_fast_i32(int t, const NpFast &f)
{
    const double x = (double)t;
    const unsigned e_b = __builtin_amdgcn_ubfe((unsigned)__double2hiint(x), 20u, 11u);
    unsigned eb;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(eb) : "v"(e_b), "s"(f.base_b), "v"(f.top_b));
    const double M = __hiloint2double((int)((eb << 20) + f.m_const), 0);
    const int q = __double2loint(x + M);
    return q << (eb - f.base_b);
}

// byte E of w = low byte of (v >> sh), of (v & msk), of (x - y): the operation writes its result's low byte straight
// into the packed word (sub-dword destination select), the other bytes are kept
template <int E>
__device__ __forceinline__ void put_shr(uint32_t &w, unsigned sh, unsigned v)
{
    if constexpr (E == 0) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
    if constexpr (E == 1) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
    if constexpr (E == 2) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
    if constexpr (E == 3) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
}
template <int E>
__device__ __forceinline__ void put_ashr(uint32_t &w, unsigned sh, int v)
{
    if constexpr (E == 0) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
    if constexpr (E == 1) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
    if constexpr (E == 2) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
    if constexpr (E == 3) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(sh), "v"(v));
}
template <int E>
__device__ __forceinline__ void put_and(uint32_t &w, unsigned msk, unsigned v)
{
    if constexpr (E == 0) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(msk), "v"(v));
    if constexpr (E == 1) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(msk), "v"(v));
    if constexpr (E == 2) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(msk), "v"(v));
    if constexpr (E == 3) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(msk), "v"(v));
}
template <int E>
__device__ __forceinline__ void put_sub(uint32_t &w, unsigned x, unsigned y)
{
    if constexpr (E == 0) asm("v_sub_u32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(x), "v"(y));
    if constexpr (E == 1) asm("v_sub_u32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(x), "v"(y));
    if constexpr (E == 2) asm("v_sub_u32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(x), "v"(y));
    if constexpr (E == 3) asm("v_sub_u32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(w) : "v"(x), "v"(y));
}

// Four neighbouring channels of one pixel: accumulators -> one packed word of codes, of high digits, of low digits.
// FAST: 7 <= shift <= 36 (32-bit rounding above), else the 64-bit form; RELU and CODES (codes wanted) as template
// parameters keep the sign handling and the encoding out of the variants that do not need them.
template <bool FAST, bool RELU, bool CODES, int E>
__device__ __forceinline__ void np_finish_one(int A, int Cc, int Bm, const NpRound &rnd, const NpFast &fr, int p_y, uint32_t &wc,
                                              uint32_t &whi, uint32_t &wlo)
{
    const int T = (A << 6) + Bm;                         // 64 A + B (the bias sits in the start values of B and C)
    int beta;
    if constexpr (FAST) {
        beta = np_round_fast(T, Cc, fr);
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(beta) : "v"(beta), "s"(RELU ? 0 : -fr.bmax), "v"(fr.bmax));
    } else {
        beta = np_round_acc((long long)T * 64 + (long long)Cc, rnd);
    }
    if constexpr (RELU) {
        put_shr<E>(whi, 6u, (unsigned)beta);
        put_and<E>(wlo, 63u, (unsigned)beta);
        if constexpr (CODES) wc |= np_code_of(beta, p_y) << (8 * E);
    } else {
        // digits of the sign of beta: h = trunc(beta / 64), l = beta - 64 h
        const int t = beta + ((beta >> 31) & 63);
        put_ashr<E>(whi, 6u, t);
        put_sub<E>(wlo, (unsigned)beta, (unsigned)t & ~63u);
        if constexpr (CODES) wc |= np_code_of(beta, p_y) << (8 * E);
    }
}

// The fused join: the layer's result (32-bit rounding, clamp with the layer's own ReLU as the lower bound), aligned with
// the other operand's integer 64 h + l, summed, converted a second time and split into digits.
template <bool RELU_OUT, int E>
__device__ __forceinline__ void np_finish_add_one(int A, int Cc, int Bm, uint32_t oh4, uint32_t ol4, int lo1, int sa, int sb, const NpFast &fr,
                                                  const NpFast &fr2, uint32_t &whi, uint32_t &wlo)
{
    int beta = np_round_fast((A << 6) + Bm, Cc, fr);
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(beta) : "v"(beta), "s"(lo1), "v"(fr.bmax));
    const int other = 64 * byte_of(oh4, E) + byte_of(ol4, E);
    const int t = (beta << sa) + (other << sb);
    int r = np_round_fast_i32(t, fr2);
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(r), "s"(RELU_OUT ? 0 : -fr2.bmax), "v"(fr2.bmax));
    if constexpr (RELU_OUT) {
        put_shr<E>(whi, 6u, (unsigned)r);
        put_and<E>(wlo, 63u, (unsigned)r);
    } else {
        const int u = r + ((r >> 31) & 63);
        put_ashr<E>(whi, 6u, u);
        put_sub<E>(wlo, (unsigned)r, (unsigned)u & ~63u);
    }
}

// The largest m of a workgroup raises one of `words` words, 128 bytes apart (they start at zero): atomics on one word are served one by
// one (512 workgroups, one each: 6 us).
constexpr int kMaxStride = 16;           // 8-byte words between them
__device__ __forceinline__ void block_max_to(unsigned long long *dst, unsigned long long m, int words)
{
    __shared__ unsigned long long best[16];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long other = __shfl_xor(m, o, 64);
        m = other > m ? other : m;
    }
    if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (unsigned i = 1; i < blockDim.x / 64; i++) m = best[i] > m ? best[i] : m;
        dst += (blockIdx.x % (unsigned)words) * kMaxStride;
        // the maximum only grows: a workgroup that sees that its own is no news spares the word the atomic
        if (m > __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(dst, m);
    }
}
__device__ __forceinline__ unsigned long long spread_max(const unsigned long long *p, int words)
{
    unsigned long long m = 0;
    for (int i = 0; i < words; i++) m = p[i * kMaxStride] > m ? p[i * kMaxStride] : m;
    return m;
}

// The layer's rescale shift: given, or - in a calibration whose formats stay on the device - from device words.
__device__ __forceinline__ int np_layer_shift(const NpConvArgs &a)
{
    if (!a.cal_fx) return a.shift;
    const int acc_frac = *a.cal_fx + *a.cal_fw;
    const int fy = a.cal_fixed ? a.cal_fixed_frac : frac_from_int(spread_max(a.cal_amax, a.amax_words), acc_frac, (unsigned long long)a.beta_max);
    const int shift = acc_frac - fy;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *a.cal_fy = fy;
        if (shift < -16 || shift > 48) atomicOr(a.cal_err, 2);           // refused at the end, as a call with these formats is
    }
    return min(max(shift, -16), 48);
}

}  // namespace dfq
