// Bandwidth-bound kernels of the quantized path: float<->code conversion, scaled addition
// (Eq. 10), concat with per-branch rescale, pooling, and the max-|.| reductions used by
// calibration (Sec. 3).  Every kernel moves 16 bytes per lane per access where alignment
// allows and falls back to narrower accesses otherwise; none keeps data in LDS because
// nothing is reused.
#include "dfq_device.hpp"
#include "dfq_host.hpp"
#include "conv_epilogue.hpp"
#include "np_device.hpp"
#include "reduce_device.hpp"

namespace dfq {

static inline int grid_for(size_t work_items)
{
    size_t blocks = (work_items + kBlock - 1) / kBlock;
    size_t cap = 256 * 16;  // 16 workgroups per compute unit, grid-stride beyond that
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

// ------------------------------------------------------------------------------------------
// quantize / dequantize
// ------------------------------------------------------------------------------------------

__global__ void __launch_bounds__(kBlock) quantize_vec4(const float4 *__restrict__ x, uint32_t *__restrict__ q,
                                                         size_t n4, float scale)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (size_t)gridDim.x * kBlock) {
        float4 v = x[i];
        q[i] = pack4(quant_one(v.x, scale), quant_one(v.y, scale), quant_one(v.z, scale), quant_one(v.w, scale));
    }
}

__global__ void __launch_bounds__(kBlock) quantize_scalar(const float *__restrict__ x, int8_t *__restrict__ q,
                                                           size_t n, float scale)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        q[i] = (int8_t)quant_one(x[i], scale);
}

__global__ void __launch_bounds__(kBlock) quantize_i32_kernel(const float *__restrict__ x, int32_t *__restrict__ q,
                                                               size_t n, float scale)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
        q[i] = saturate_i32(__builtin_rintf(x[i] * scale));   // exact product; overflow to Inf saturates
    }
}

__global__ void __launch_bounds__(kBlock) dequantize_vec4(const uint32_t *__restrict__ q, float4 *__restrict__ x,
                                                           size_t n4, float inv_scale)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (size_t)gridDim.x * kBlock) {
        uint32_t w = q[i];
        x[i] = make_float4((float)byte_of(w, 0) * inv_scale, (float)byte_of(w, 1) * inv_scale,
                           (float)byte_of(w, 2) * inv_scale, (float)byte_of(w, 3) * inv_scale);
    }
}

__global__ void __launch_bounds__(kBlock) dequantize_scalar(const int8_t *__restrict__ q, float *__restrict__ x,
                                                             size_t n, float inv_scale)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        x[i] = (float)q[i] * inv_scale;
}

// ------------------------------------------------------------------------------------------
// General (n, p) dynamic floating-point codes (Sec. 2.1, Eq. 1-5), n <= 8: one byte per code, bit n-1 the
// sign, bits n-2 .. p the exponent field e, bits p-1 .. 0 the significand field m; value
// 2^-frac * (e == 0 ? m : 2^(e-1) * (2^p + m)), every exponent code a number.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float np_dequant_one(uint32_t code, const NpFmt &f)
{
    const uint32_t m = code & ((1u << f.p) - 1u);
    const uint32_t e = (code >> f.p) & ((1u << (f.n - 1 - f.p)) - 1u);   // no exponent field when p = n-1
    const float mag = e == 0 ? (float)m : ldexpf((float)((1u << f.p) + m), (int)e - 1);
    const float val = mag * f.scale;
    return ((code >> (f.n - 1)) & 1u) ? -val : val;
}

__global__ void __launch_bounds__(kBlock) quantize_np_vec4(const float4 *__restrict__ x, uint32_t *__restrict__ q, size_t n4, NpFmt f)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (size_t)gridDim.x * kBlock) {
        const float4 v = x[i];
        q[i] = np_quant_one(v.x, f) | (np_quant_one(v.y, f) << 8) | (np_quant_one(v.z, f) << 16) | (np_quant_one(v.w, f) << 24);
    }
}

__global__ void __launch_bounds__(kBlock) quantize_np_scalar(const float *__restrict__ x, uint8_t *__restrict__ q, size_t n, NpFmt f)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        q[i] = (uint8_t)np_quant_one(x[i], f);
}

__global__ void __launch_bounds__(kBlock) dequantize_np_vec4(const uint32_t *__restrict__ q, float4 *__restrict__ x, size_t n4, NpFmt f)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (size_t)gridDim.x * kBlock) {
        const uint32_t w = q[i];
        x[i] = make_float4(np_dequant_one(w & 0xffu, f), np_dequant_one((w >> 8) & 0xffu, f), np_dequant_one((w >> 16) & 0xffu, f),
                           np_dequant_one(w >> 24, f));
    }
}

__global__ void __launch_bounds__(kBlock) dequantize_np_scalar(const uint8_t *__restrict__ q, float *__restrict__ x, size_t n, NpFmt f)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        x[i] = np_dequant_one(q[i], f);
}

// Row-wise forms for weights with one format per output channel: row r of x[rows][row_len] is
// converted at the fractional length frac[r] (+ frac_add), read from device memory.
__global__ void __launch_bounds__(kBlock) quantize_rows_kernel(const float *__restrict__ x, int8_t *__restrict__ q, size_t rows,
                                                                size_t row_len, const int32_t *__restrict__ frac)
{
    const size_t n = rows * row_len;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        q[i] = (int8_t)quant_one(x[i], ldexpf(1.0f, frac[i / row_len]));
}

__global__ void __launch_bounds__(kBlock) quantize_i32_rows_kernel(const float *__restrict__ x, int32_t *__restrict__ q, size_t rows,
                                                                    size_t row_len, const int32_t *__restrict__ frac, int frac_add)
{
    const size_t n = rows * row_len;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
        q[i] = quant_i32_one(x[i], frac[i / row_len] + frac_add);
    }
}

// Folding a per-channel affine layer (batch norm in its inference form, a scale layer) that follows a convolution
// into the convolution's float weights and bias, before anything is quantized: w'[k][.] = w[k][.] * scale[k],
// b'[k] = b[k] * scale[k] + shift[k].  Every product and the sum are rounded to float separately (no fused
// multiply-add), so that the result does not depend on how the compiler contracts the expression.
__global__ void __launch_bounds__(kBlock) fold_scale_kernel(const float *__restrict__ w, const float *__restrict__ b, size_t rows,
                                                             size_t row_len, const float *__restrict__ scale,
                                                             const float *__restrict__ shift, float *__restrict__ w_out,
                                                             float *__restrict__ b_out)
{
#pragma clang fp contract(off)
    const size_t n = rows * row_len;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n + rows; i += (size_t)gridDim.x * kBlock) {
        if (i < n) {
            w_out[i] = w[i] * scale[i / row_len];
        } else if (b_out) {
            const size_t r = i - n;
            float prod = (b ? b[r] : 0.0f) * scale[r];
            asm volatile("" : "+v"(prod));        // the product is rounded on its own: no fused multiply-add
            b_out[r] = prod + (shift ? shift[r] : 0.0f);
        }
    }
}

static inline bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

hipError_t launch_fold_scale(const float *w, const float *b, size_t rows, size_t row_len, const float *scale, const float *shift,
                             float *w_out, float *b_out, hipStream_t st)
{
    fold_scale_kernel<<<grid_for(rows * row_len + rows), kBlock, 0, st>>>(w, b, rows, row_len, scale, shift, w_out, b_out);
    return hipGetLastError();
}

hipError_t launch_quantize_rows(const float *x, int8_t *q, size_t rows, size_t row_len, const int32_t *frac, hipStream_t st)
{
    quantize_rows_kernel<<<grid_for(rows * row_len), kBlock, 0, st>>>(x, q, rows, row_len, frac);
    return hipGetLastError();
}

hipError_t launch_quantize_i32_rows(const float *x, int32_t *q, size_t rows, size_t row_len, const int32_t *frac, int frac_add,
                                    hipStream_t st)
{
    quantize_i32_rows_kernel<<<grid_for(rows * row_len), kBlock, 0, st>>>(x, q, rows, row_len, frac, frac_add);
    return hipGetLastError();
}

hipError_t launch_quantize(const float *x, int8_t *q, size_t n, int frac, hipStream_t st)
{
    float scale = ldexpf(1.0f, frac);
    if (aligned(x, 16) && aligned(q, 4)) {
        size_t n4 = n / 4;
        if (n4) quantize_vec4<<<grid_for(n4), kBlock, 0, st>>>((const float4 *)x, (uint32_t *)q, n4, scale);
        size_t tail = n - n4 * 4;
        if (tail) quantize_scalar<<<1, kBlock, 0, st>>>(x + n4 * 4, q + n4 * 4, tail, scale);
    } else {
        quantize_scalar<<<grid_for(n), kBlock, 0, st>>>(x, q, n, scale);
    }
    return hipGetLastError();
}

hipError_t launch_quantize_i32(const float *x, int32_t *q, size_t n, int frac, hipStream_t st)
{
    quantize_i32_kernel<<<grid_for(n), kBlock, 0, st>>>(x, q, n, ldexpf(1.0f, frac));
    return hipGetLastError();
}

static NpFmt make_npfmt(int nbits, int p, int frac_signed)
{
    NpFmt f;
    f.n = nbits;
    f.p = p;
    f.scale = ldexpf(1.0f, frac_signed);
    const int emax = p == nbits - 1 ? 1 : (1 << (nbits - 1 - p)) - 1;
    f.beta_max = p == nbits - 1 ? (float)((1 << (nbits - 1)) - 1) : ldexpf((float)((1 << (p + 1)) - 1), emax - 1);
    return f;
}

hipError_t launch_quantize_np(const float *x, uint8_t *q, size_t n, int nbits, int p, int frac, hipStream_t st)
{
    const NpFmt f = make_npfmt(nbits, p, frac);
    if (aligned(x, 16) && aligned(q, 4)) {
        size_t n4 = n / 4;
        if (n4) quantize_np_vec4<<<grid_for(n4), kBlock, 0, st>>>((const float4 *)x, (uint32_t *)q, n4, f);
        size_t tail = n - n4 * 4;
        if (tail) quantize_np_scalar<<<1, kBlock, 0, st>>>(x + n4 * 4, q + n4 * 4, tail, f);
    } else {
        quantize_np_scalar<<<grid_for(n), kBlock, 0, st>>>(x, q, n, f);
    }
    return hipGetLastError();
}

hipError_t launch_dequantize_np(const uint8_t *q, float *x, size_t n, int nbits, int p, int frac, hipStream_t st)
{
    const NpFmt f = make_npfmt(nbits, p, -frac);
    if (aligned(x, 16) && aligned(q, 4)) {
        size_t n4 = n / 4;
        if (n4) dequantize_np_vec4<<<grid_for(n4), kBlock, 0, st>>>((const uint32_t *)q, (float4 *)x, n4, f);
        size_t tail = n - n4 * 4;
        if (tail) dequantize_np_scalar<<<1, kBlock, 0, st>>>(q + n4 * 4, x + n4 * 4, tail, f);
    } else {
        dequantize_np_scalar<<<grid_for(n), kBlock, 0, st>>>(q, x, n, f);
    }
    return hipGetLastError();
}

hipError_t launch_dequantize(const int8_t *q, float *x, size_t n, int frac, hipStream_t st)
{
    float inv = ldexpf(1.0f, -frac);
    if (aligned(x, 16) && aligned(q, 4)) {
        size_t n4 = n / 4;
        if (n4) dequantize_vec4<<<grid_for(n4), kBlock, 0, st>>>((const uint32_t *)q, (float4 *)x, n4, inv);
        size_t tail = n - n4 * 4;
        if (tail) dequantize_scalar<<<1, kBlock, 0, st>>>(q + n4 * 4, x + n4 * 4, tail, inv);
    } else {
        dequantize_scalar<<<grid_for(n), kBlock, 0, st>>>(q, x, n, inv);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// eltwise_q: exact alignment to the finer scale, one add, one rounding
// ------------------------------------------------------------------------------------------

struct EltParams {
    int sa, sb;   // left shifts that bring a and b to the common fractional length F
    int s;        // F - f_y
    int relu;
};

__device__ __forceinline__ int elt_one(int a, int b, const EltParams &p, int &sum_out)
{
    int sum = a * (1 << p.sa) + b * (1 << p.sb);
    sum_out = sum;
    if (p.relu) sum = max(sum, 0);
    return requant8(sum, p.s);
}

template <bool kWantY, bool kWantAcc>
__global__ void __launch_bounds__(kBlock) eltwise_vec16(const uint4 *__restrict__ a, const uint4 *__restrict__ b,
                                                         uint4 *__restrict__ y, int4 *__restrict__ acc, size_t n16,
                                                         EltParams p)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n16; i += (size_t)gridDim.x * kBlock) {
        uint4 va = a[i], vb = b[i];
        const uint32_t wa[4] = {va.x, va.y, va.z, va.w};
        const uint32_t wb[4] = {vb.x, vb.y, vb.z, vb.w};
        uint32_t out[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            int s0, s1, s2, s3;
            int r0 = elt_one(byte_of(wa[j], 0), byte_of(wb[j], 0), p, s0);
            int r1 = elt_one(byte_of(wa[j], 1), byte_of(wb[j], 1), p, s1);
            int r2 = elt_one(byte_of(wa[j], 2), byte_of(wb[j], 2), p, s2);
            int r3 = elt_one(byte_of(wa[j], 3), byte_of(wb[j], 3), p, s3);
            out[j] = pack4(r0, r1, r2, r3);
            if (kWantAcc) acc[i * 4 + j] = make_int4(s0, s1, s2, s3);
        }
        if (kWantY) y[i] = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

// The common case - int8 result only, final shift in [0, 23] - with the branch-free rounding
// shift of the convolution epilogue: per element two sign-extracting field reads, a shift, a
// shift-add, then clamp / rounding bit / add / shift-into-byte.
__global__ void __launch_bounds__(kBlock) eltwise_fast16(const uint4 *__restrict__ a, const uint4 *__restrict__ b,
                                                          uint4 *__restrict__ y, size_t n16, EltParams p)
{
    Requant rq;
    rq.init(p.s, p.relu);
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n16; i += (size_t)gridDim.x * kBlock) {
        const uint4 va = a[i], vb = b[i];
        const uint32_t wa[4] = {va.x, va.y, va.z, va.w};
        const uint32_t wb[4] = {vb.x, vb.y, vb.z, vb.w};
        uint32_t out[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            int t[4];
#pragma unroll
            for (int e = 0; e < 4; e++)
                t[e] = (int)((unsigned)byte_of(wa[j], e) << p.sa) + (int)((unsigned)byte_of(wb[j], e) << p.sb);
            out[j] = rq.fast_four(t[0], t[1], t[2], t[3]);
        }
        y[i] = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

__global__ void __launch_bounds__(kBlock) eltwise_scalar(const int8_t *__restrict__ a, const int8_t *__restrict__ b,
                                                          int8_t *__restrict__ y, int32_t *__restrict__ acc, size_t n,
                                                          EltParams p)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
        int sum;
        int r = elt_one(a[i], b[i], p, sum);
        if (acc) acc[i] = sum;
        if (y) y[i] = (int8_t)r;
    }
}

hipError_t launch_eltwise(const int8_t *a, int fa, const int8_t *b, int fb, int8_t *y, int fy, int32_t *acc, size_t n,
                          int relu, hipStream_t st)
{
    int F = fa > fb ? fa : fb;
    EltParams p{F - fa, F - fb, F - fy, relu};
    bool vec = aligned(a, 16) && aligned(b, 16) && (!y || aligned(y, 16)) && (!acc || aligned(acc, 16));
    size_t n16 = vec ? n / 16 : 0;
    if (n16) {
        int g = grid_for(n16);
        if (y && !acc && p.s >= 0 && p.s <= 23) eltwise_fast16<<<g, kBlock, 0, st>>>((const uint4 *)a, (const uint4 *)b, (uint4 *)y, n16, p);
        else if (y && acc) eltwise_vec16<true, true><<<g, kBlock, 0, st>>>((const uint4 *)a, (const uint4 *)b, (uint4 *)y, (int4 *)acc, n16, p);
        else if (y) eltwise_vec16<true, false><<<g, kBlock, 0, st>>>((const uint4 *)a, (const uint4 *)b, (uint4 *)y, nullptr, n16, p);
        else eltwise_vec16<false, true><<<g, kBlock, 0, st>>>((const uint4 *)a, (const uint4 *)b, nullptr, (int4 *)acc, n16, p);
    }
    size_t done = n16 * 16;
    if (n > done)
        eltwise_scalar<<<grid_for(n - done), kBlock, 0, st>>>(a + done, b + done, y ? y + done : nullptr,
                                                               acc ? acc + done : nullptr, n - done, p);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// concat_q: one launch, every lane produces a piece of VEC output bytes of one branch
// ------------------------------------------------------------------------------------------

struct ConcatParams {
    const int8_t *x[8];
    int C[8];       // channels of each branch
    int off[8];     // channel offset of each branch in y
    int s[8];       // f_i - f_y
    int pieces[9];  // pieces of the branches before this one; pieces[nb]: of a whole pixel
    int nb;
    FastDiv div_pieces;
    // formats in device words (calibration)
    const int32_t *frac;
    int idx[8];
    int fixed, fixed_frac;
    int32_t *frac_out;
};

// VEC bytes at any byte address.  Channel counts that are no multiple of VEC are covered by pieces that overlap: the last piece of a
// pixel (of a branch) starts VEC channels before its end, so every access is whole and the bytes two lanes write are the same.
template <int VEC>
struct __attribute__((packed, aligned(1))) Piece {
    uint32_t w[VEC / 4];
};
template <>
struct Piece<1> {
    int8_t w[1];
};

// ldy: bytes between consecutive pixels of y (>= the branches' channels together).  FAST: every branch's shift lies in [0, 23].
// Memory-bound: 3 branches of 90 channels over 24 x 45 x 61 pixels (35 MB) took 43 us with byte accesses, now 10.
// DEV: the formats are device words; the result's is derived and stored.
template <int VEC, bool FAST, bool DEV = false>
__global__ void __launch_bounds__(kBlock) concat_kernel(ConcatParams p, int8_t *__restrict__ y, size_t pixels, int ldy)
{
    if constexpr (DEV) {
        int fy = p.fixed ? p.fixed_frac : p.frac[p.idx[0]];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            p.s[j] = j < p.nb ? p.frac[p.idx[j]] : 0;
            if (!p.fixed && j < p.nb) fy = min(fy, p.s[j]);
        }
#pragma unroll
        for (int j = 0; j < 8; j++) p.s[j] -= fy;
        if (blockIdx.x == 0 && threadIdx.x == 0) *p.frac_out = fy;
    }
    const size_t total = pixels * (size_t)p.pieces[p.nb];
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (size_t)gridDim.x * kBlock) {
        const size_t px = total < (1ull << 31) ? (size_t)fastdiv((int)i, p.div_pieces) : i / (size_t)p.pieces[p.nb];
        const int pc = (int)(i - px * p.pieces[p.nb]);
        const int8_t *src = p.x[0];
        int C = p.C[0], off = 0, first = 0, s = p.s[0];
        if constexpr (VEC == 1) {
            // (one byte per lane: the branch's number alone is cheaper to select; 50176 pixels of 3 + 64 channels 10.0 us, else 10.7)
            int br = 0;
#pragma unroll
            for (int j = 1; j < 8; j++)
                if (j < p.nb && pc >= p.pieces[j]) br = j;
            src = p.x[br]; C = p.C[br]; off = p.off[br]; first = p.pieces[br]; s = p.s[br];
        } else {
#pragma unroll
            for (int j = 1; j < 8; j++)
                if (j < p.nb && pc >= p.pieces[j]) { src = p.x[j]; C = p.C[j]; off = p.off[j]; first = p.pieces[j]; s = p.s[j]; }
        }
        const int c = min((pc - first) * VEC, C - VEC);
        const Piece<VEC> v = *(const Piece<VEC> *)(src + px * (size_t)C + c);
        Piece<VEC> o;
        if constexpr (VEC == 1) {
            o.w[0] = (int8_t)requant8(v.w[0], s);
        } else if constexpr (FAST) {
            const int hi = 127 << s, badd = s > 0 ? (1 << (s - 1)) - 1 : 0;
            const int4 s4 = make_int4(s, s, s, s), h4 = make_int4(hi, hi, hi, hi), b4 = make_int4(badd, badd, badd, badd);
#pragma unroll
            for (int j = 0; j < VEC / 4; j++)
                o.w[j] = requant_four_per_channel(byte_of(v.w[j], 0), byte_of(v.w[j], 1), byte_of(v.w[j], 2), byte_of(v.w[j], 3), s4, h4, b4, 0);
        } else {
#pragma unroll
            for (int j = 0; j < VEC / 4; j++)
                o.w[j] = pack4(requant8(byte_of(v.w[j], 0), s), requant8(byte_of(v.w[j], 1), s), requant8(byte_of(v.w[j], 2), s),
                               requant8(byte_of(v.w[j], 3), s));
        }
        *(Piece<VEC> *)(y + px * (size_t)ldy + off + c) = o;
    }
}

template <int VEC>
static void launch_concat_vec(ConcatParams &p, int8_t *y, int ldy, size_t pixels, hipStream_t st)
{
    bool fast = true;
    p.pieces[0] = 0;
    for (int i = 0; i < p.nb; i++) {
        p.pieces[i + 1] = p.pieces[i] + (p.C[i] + VEC - 1) / VEC;
        fast = fast && p.s[i] >= 0 && p.s[i] <= 23;
    }
    p.div_pieces = make_fastdiv(p.pieces[p.nb]);
    const int g = grid_for(pixels * (size_t)p.pieces[p.nb]);
    if (p.frac) concat_kernel<VEC, false, true><<<g, kBlock, 0, st>>>(p, y, pixels, ldy);
    else if (VEC > 1 && fast) concat_kernel<VEC, true><<<g, kBlock, 0, st>>>(p, y, pixels, ldy);
    else concat_kernel<VEC, false><<<g, kBlock, 0, st>>>(p, y, pixels, ldy);
}

hipError_t launch_concat(int nb, const int8_t *const *xs, const int *Cs, const int *fs, int8_t *y, int ldy, int fy,
                         size_t pixels, hipStream_t st, const CalConcat &cal)
{
    ConcatParams p{};
    p.nb = nb;
    p.frac = cal.frac;
    p.fixed = cal.fixed;
    p.fixed_frac = cal.fixed_frac;
    p.frac_out = cal.frac_out;
    int off = 0, least = Cs[0];
    for (int i = 0; i < nb; i++) {
        p.x[i] = xs[i];
        p.C[i] = Cs[i];
        p.off[i] = off;
        p.s[i] = cal.frac ? 0 : fs[i] - fy;
        p.idx[i] = cal.frac ? cal.idx[i] : 0;
        off += Cs[i];
        least = Cs[i] < least ? Cs[i] : least;
    }
    // a piece lies inside one branch, so the narrowest branch decides
    if (least >= 16) launch_concat_vec<16>(p, y, ldy, pixels, st);
    else if (least >= 4) launch_concat_vec<4>(p, y, ldy, pixels, st);
    else launch_concat_vec<1>(p, y, ldy, pixels, st);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// pool_q
// ------------------------------------------------------------------------------------------

struct PoolParams {
    int N, H, W, C, P, Q, k, stride, pad;
    int mode;   // 0 max, 1 avg
    int d;      // f_out - f_in
};

// (sum * 2^d) / (k*k) rounded to nearest, ties to even, clamped.  |sum| <= 128 * 4096.
__device__ __forceinline__ int avg_round(int sum, int win, int d)
{
    if (d >= 32) return sum == 0 ? 0 : (sum > 0 ? 127 : -127);
    if (d <= -40) return 0;
    long long num = sum, den = win;
    if (d >= 0) num <<= d; else den <<= -d;
    long long t = num / den;
    long long rem = num - t * den;
    if (rem < 0) { t -= 1; rem += den; }          // floor
    if (2 * rem > den || (2 * rem == den && (t & 1))) t += 1;
    t = t > 127 ? 127 : (t < -127 ? -127 : t);
    return (int)t;
}

// Any window over any number of channels: one output element per lane.  Pools of fewer than four channels (and images beyond 2^31 pieces).
__global__ void __launch_bounds__(kBlock) pool_scalar_kernel(const int8_t *__restrict__ x, int8_t *__restrict__ y, PoolParams p)
{
    const size_t total = (size_t)p.N * p.P * p.Q * p.C;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (size_t)gridDim.x * kBlock) {
        const int c = (int)(i % p.C);
        const size_t px = i / p.C;
        const int q = (int)(px % p.Q);
        const size_t t = px / p.Q;
        const int pp = (int)(t % p.P);
        const int n = (int)(t / p.P);
        int acc = p.mode == 0 ? -1000 : 0;
        for (int r = 0; r < p.k; r++) {
            const int ih = pp * p.stride - p.pad + r;
            if (ih < 0 || ih >= p.H) continue;
            const int first = max(0, p.pad - q * p.stride), end = min(p.k, p.W + p.pad - q * p.stride);
            const int8_t *src = x + (((size_t)n * p.H + ih) * p.W + (q * p.stride - p.pad + first)) * p.C + c;
#pragma unroll 4
            for (int s = first; s < end; s++, src += p.C) {
                const int v = *src;
                acc = p.mode == 0 ? max(acc, v) : acc + v;
            }
        }
        y[i] = (int8_t)(p.mode == 0 ? requant8(acc, -p.d) : avg_round(acc, p.k * p.k, p.d));
    }
}

// VEC channels per lane, at any byte address (Piece: the last piece of a pixel overlaps the one before where C is no multiple of VEC).
// Window positions in the padding are replaced by the nearest one inside the image - for the maximum it lies in the same window
// (pad < k), for the mean its bytes are dropped - so no load depends on a branch: with K > 0 the K*K loads of a window are all in
// flight together, with a window size only known at run time (K == 0) four of a row at a time.
// Bound by memory and issue; 24 x 45 x 61 x 90, 3x3 / 1: 48.9 us with byte accesses, now 10.3.
struct PoolVecParams {
    PoolParams p;
    int pieces;          // of a pixel
    int total;           // N * P * Q * pieces (below 2^31)
    FastDiv div_pieces, div_q, div_p;
    FastDiv div_den;     // mean: the divisor k*k << max(-d, 0)
    int num_shift;       // mean: max(d, 0)
    int exact32;         // mean: sum << num_shift and the divisor fit 31 bits
};

typedef short v2s __attribute__((ext_vector_type(2)));

template <int E>
__device__ __forceinline__ int add_byte(int acc, uint32_t w)
{
    if constexpr (E == 0) asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(acc) : "v"(acc), "v"(w));
    else if constexpr (E == 1) asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(acc) : "v"(acc), "v"(w));
    else if constexpr (E == 2) asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(acc) : "v"(acc), "v"(w));
    else asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(acc) : "v"(acc), "v"(w));
    return acc;
}

// The mean of avg_round by one multiplication with the divisor's reciprocal: rounding to nearest, ties to even, is symmetric, so
// quotient and remainder of the magnitude decide it.
__device__ __forceinline__ int mean_round(int sum, const PoolVecParams &prm)
{
    if (!prm.exact32) return avg_round(sum, prm.p.k * prm.p.k, prm.p.d);
    const int mag = (sum < 0 ? -sum : sum) << prm.num_shift;
    int q = fastdiv(mag, prm.div_den);
    const int rem2 = 2 * (mag - q * prm.div_den.d);
    q += (rem2 > prm.div_den.d || (rem2 == prm.div_den.d && (q & 1))) ? 1 : 0;
    q = min(q, 127);
    return sum < 0 ? -q : q;
}

// The maxima of a word's bytes, held as the high bytes of packed 16-bit numbers, rescaled by 2^d and packed.
__device__ __forceinline__ uint32_t max_word(v2s odd, v2s even, int d)
{
    // no rescale: the high bytes as they are, -128 saturated (sixteen branches that skip the rescale value by value took longer
    // than the maxima: 64 x 28 x 28 x 192, 3x3 / 2, 5.6 us, now 4.7)
    if (d == 0) {
        const v2s least = {(short)(-127 * 256), (short)(-127 * 256)};
        return (__builtin_bit_cast(uint32_t, __builtin_elementwise_max(odd, least)) & 0xff00ff00u) |
               ((__builtin_bit_cast(uint32_t, __builtin_elementwise_max(even, least)) >> 8) & 0x00ff00ffu);
    }
    return pack4(requant8(even[0] >> 8, -d), requant8(odd[0] >> 8, -d), requant8(even[1] >> 8, -d), requant8(odd[1] >> 8, -d));
}

template <int VEC, int K, bool MEAN>
__global__ void __launch_bounds__(kBlock) pool_kernel(const int8_t *__restrict__ x, int8_t *__restrict__ y, PoolVecParams prm)
{
    constexpr int W = VEC / 4;                   // words of a piece
    const PoolParams &p = prm.p;
    const int k = K > 0 ? K : p.k;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < prm.total; i += gridDim.x * kBlock) {
        const int px = fastdiv(i, prm.div_pieces);
        const int c = min((i - px * prm.pieces) * VEC, p.C - VEC);
        const int t = fastdiv(px, prm.div_q);
        const int q = px - t * p.Q;
        const int n = fastdiv(t, prm.div_p);
        const int pp = t - n * p.P;
        const int8_t *img = x + (size_t)n * p.H * p.W * p.C + c;
        const int h0 = pp * p.stride - p.pad, w0 = q * p.stride - p.pad;
        // maximum: odd and even bytes of a word are kept as the high bytes of packed 16-bit numbers (what stands in the low byte never
        // decides between different high bytes): one shift and two packed maxima per word
        v2s odd[W], even[W];
        int sum[VEC];
#pragma unroll
        for (int j = 0; j < W; j++) odd[j] = even[j] = v2s{(short)-32768, (short)-32768};
#pragma unroll
        for (int j = 0; j < VEC; j++) sum[j] = 0;
        auto load = [&](int r, int s) {
            const int ih = min(max(h0 + r, 0), p.H - 1), iw = min(max(w0 + s, 0), p.W - 1);
            return *(const Piece<VEC> *)(img + (size_t)(ih * p.W + iw) * p.C);
        };
        auto take = [&](const Piece<VEC> &u, bool inside) {
#pragma unroll
            for (int j = 0; j < W; j++) {
                uint32_t w = u.w[j];
                if constexpr (MEAN) {
                    w = inside ? w : 0u;
                    sum[4 * j + 0] = add_byte<0>(sum[4 * j + 0], w);
                    sum[4 * j + 1] = add_byte<1>(sum[4 * j + 1], w);
                    sum[4 * j + 2] = add_byte<2>(sum[4 * j + 2], w);
                    sum[4 * j + 3] = add_byte<3>(sum[4 * j + 3], w);
                } else {
                    odd[j] = __builtin_elementwise_max(odd[j], __builtin_bit_cast(v2s, w));
                    even[j] = __builtin_elementwise_max(even[j], __builtin_bit_cast(v2s, w << 8));
                }
            }
        };
        auto inside = [&](int r, int s) { return (unsigned)(h0 + r) < (unsigned)p.H && (unsigned)(w0 + s) < (unsigned)p.W; };
        if constexpr (K > 0) {
            Piece<VEC> u[K * K];
#pragma unroll
            for (int r = 0; r < K; r++)
#pragma unroll
                for (int s = 0; s < K; s++) u[r * K + s] = load(r, s);
#pragma unroll
            for (int r = 0; r < K; r++)
#pragma unroll
                for (int s = 0; s < K; s++) take(u[r * K + s], inside(r, s));
        } else {
            for (int r = 0; r < k; r++)
                for (int s = 0; s < k; s += 4) {
                    Piece<VEC> u[4];
#pragma unroll
                    for (int j = 0; j < 4; j++) u[j] = load(r, min(s + j, k - 1));
#pragma unroll
                    for (int j = 0; j < 4; j++) take(u[j], s + j < k && inside(r, s + j));
                }
        }
        Piece<VEC> o;
        if constexpr (MEAN) {
#pragma unroll
            for (int j = 0; j < W; j++) {
                int v[4];
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = mean_round(sum[4 * j + e], prm);
                o.w[j] = pack4(v[0], v[1], v[2], v[3]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < W; j++) o.w[j] = max_word(odd[j], even[j], p.d);
        }
        *(Piece<VEC> *)(y + (size_t)px * p.C + c) = o;
    }
}

// 3x3 maximum at stride 1 (a pooling branch that keeps the image's size), 16 channels of kRows output pixels below each other per lane:
// a row's three pieces are read once for the three windows they lie in, and their maximum is taken once (18 reads and 72 packed
// maxima for four outputs instead of 36 and 72 with twice the unpacking).  Positions outside the image by the nearest one inside, as above.
// Bound by the address path of the loads (2-byte aligned pieces of 90 channels).  24 x 45 x 61 x 90:
// 10.4 us, here 8.1; 64 x 28 x 28 x 192: 8.4, here 7.4.
struct Pool3Params {
    PoolParams p;
    int pieces, total;                       // total: N * ceil(P / kRows) * Q * pieces
    FastDiv div_pieces, div_q, div_strips;
};

template <int ROWS>
__global__ void __launch_bounds__(kBlock) maxpool3_s1_kernel(const int8_t *__restrict__ x, int8_t *__restrict__ y, Pool3Params prm)
{
    const PoolParams &p = prm.p;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < prm.total; i += gridDim.x * kBlock) {
        const int col = fastdiv(i, prm.div_pieces);
        const int c = min((i - col * prm.pieces) * 16, p.C - 16);
        const int t = fastdiv(col, prm.div_q);
        const int q = col - t * p.Q;
        const int n = fastdiv(t, prm.div_strips);
        const int p0 = (t - n * prm.div_strips.d) * ROWS;
        const int8_t *img = x + (size_t)n * p.H * p.W * p.C + c;
        int cols[3];
#pragma unroll
        for (int s = 0; s < 3; s++) cols[s] = min(max(q - p.pad + s, 0), p.W - 1) * p.C;
        Piece<16> u[ROWS + 2][3];
#pragma unroll
        for (int r = 0; r < ROWS + 2; r++) {
            const int8_t *row = img + (size_t)min(max(p0 - p.pad + r, 0), p.H - 1) * (p.W * p.C);
#pragma unroll
            for (int s = 0; s < 3; s++) u[r][s] = *(const Piece<16> *)(row + cols[s]);
        }
        v2s odd[ROWS + 2][4], even[ROWS + 2][4];
#pragma unroll
        for (int r = 0; r < ROWS + 2; r++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                odd[r][j] = __builtin_bit_cast(v2s, u[r][0].w[j]);
                even[r][j] = __builtin_bit_cast(v2s, u[r][0].w[j] << 8);
#pragma unroll
                for (int s = 1; s < 3; s++) {
                    odd[r][j] = __builtin_elementwise_max(odd[r][j], __builtin_bit_cast(v2s, u[r][s].w[j]));
                    even[r][j] = __builtin_elementwise_max(even[r][j], __builtin_bit_cast(v2s, u[r][s].w[j] << 8));
                }
            }
        int8_t *out = y + ((size_t)(n * p.P + p0) * p.Q + q) * p.C + c;
#pragma unroll
        for (int r = 0; r < ROWS; r++) {
            Piece<16> o;
#pragma unroll
            for (int j = 0; j < 4; j++)
                o.w[j] = max_word(__builtin_elementwise_max(__builtin_elementwise_max(odd[r][j], odd[r + 1][j]), odd[r + 2][j]),
                                  __builtin_elementwise_max(__builtin_elementwise_max(even[r][j], even[r + 1][j]), even[r + 2][j]), p.d);
            if (p0 + r < p.P) *(Piece<16> *)(out + (size_t)r * (p.Q * p.C)) = o;
        }
    }
}

// Global average pooling (the window is the whole image, one output pixel): a workgroup takes 32 words of four channels - whole
// cache lines - and its eight groups of 32 lanes share the pixels, seven loads in flight at a time; the partial sums meet in LDS and
// 128 lanes round one channel each.  Bound by latency.  One lane per word over all pixels with 64-bit divisions: 7 x 7 x 2048, one
// image: 5.3 us, here 2.8; 256 images 8.7, here 7.2.
constexpr int kAvgWords = 32, kAvgGroups = kBlock / kAvgWords;

__global__ void __launch_bounds__(kBlock) avgpool_global_kernel(const int8_t *__restrict__ x, int8_t *__restrict__ y, int pixels,
                                                                 int words, PoolVecParams prm)
{
    __shared__ int4 part[kAvgGroups][kAvgWords];
    const int C = prm.p.C, cw = C / 4;
    const int lw = threadIdx.x % kAvgWords, group = threadIdx.x / kAvgWords;
    const int i = blockIdx.x * kAvgWords + lw;                     // word of the result
    int acc[4] = {0, 0, 0, 0};
    if (i < words) {
        const int n = fastdiv(i, prm.div_pieces);
        const uint32_t *src = (const uint32_t *)x + (size_t)n * pixels * cw + (i - n * cw);
        for (int px = group; px < pixels; px += 7 * kAvgGroups) {
            uint32_t w[7];
#pragma unroll
            for (int j = 0; j < 7; j++) w[j] = px + j * kAvgGroups < pixels ? src[(size_t)(px + j * kAvgGroups) * cw] : 0u;
#pragma unroll
            for (int j = 0; j < 7; j++) {
                acc[0] = add_byte<0>(acc[0], w[j]); acc[1] = add_byte<1>(acc[1], w[j]);
                acc[2] = add_byte<2>(acc[2], w[j]); acc[3] = add_byte<3>(acc[3], w[j]);
            }
        }
    }
    part[group][lw] = make_int4(acc[0], acc[1], acc[2], acc[3]);
    __syncthreads();
    const int b = threadIdx.x;                                     // byte of the workgroup's part of the result
    if (b >= 4 * kAvgWords || blockIdx.x * kAvgWords + b / 4 >= words) return;
    int sum = 0;
#pragma unroll
    for (int g = 0; g < kAvgGroups; g++) sum += ((const int *)&part[g][0])[b];
    y[(size_t)blockIdx.x * (4 * kAvgWords) + b] = (int8_t)mean_round(sum, prm);
}

hipError_t launch_pool(const int8_t *x, int8_t *y, int mode, int N, int H, int W, int C, int P, int Q, int k, int stride,
                       int pad, int fin, int fout, hipStream_t st)
{
    PoolParams p{N, H, W, C, P, Q, k, stride, pad, mode, fout - fin};
    if (C < 4 || (long long)P * Q * ((C + 3) / 4) >= (1LL << 31) - 256LL * 16 * kBlock) {
        pool_scalar_kernel<<<grid_for((size_t)N * P * Q * C), kBlock, 0, st>>>(x, y, p);
        return hipGetLastError();
    }
    PoolVecParams prm{};
    prm.div_q = make_fastdiv(Q);
    prm.div_p = make_fastdiv(P);
    const int d = fout - fin;
    // |sum| <= 128 k^2 <= 2^19
    prm.exact32 = d <= 11 && d >= -17;
    prm.num_shift = d > 0 ? d : 0;
    prm.div_den = make_fastdiv(prm.exact32 && d < 0 ? (k * k) << -d : k * k);
    if (mode == 1 && k == H && k == W && pad == 0 && C % 4 == 0 && aligned(x, 4) && (long long)N * (C / 4) < (1LL << 31) - kBlock) {
        const int words = N * (C / 4);
        prm.p = p;
        prm.div_pieces = make_fastdiv(C / 4);
        avgpool_global_kernel<<<(words + kAvgWords - 1) / kAvgWords, kBlock, 0, st>>>(x, y, H * W, words, prm);
        return hipGetLastError();
    }
    // few outputs (a global pool): narrower lanes give the machine four times the wavefronts
    const bool wide = C >= 16 && (size_t)N * P * Q * (C / 16) >= (size_t)64 * 1024;
    const int vec = wide ? 16 : 4;
    prm.pieces = (C + vec - 1) / vec;
    prm.div_pieces = make_fastdiv(prm.pieces);
    // as many images per launch as 31-bit piece numbers reach
    const long long per_image = (long long)P * Q * prm.pieces;
    long long most = ((1LL << 31) - 256LL * 16 * kBlock - 1) / per_image;
    for (long long n = 0; n < N; n += most) {
        prm.p = p;
        prm.p.N = (int)(N - n < most ? N - n : most);
        prm.total = (int)(prm.p.N * per_image);
        const int8_t *xs = x + (size_t)n * H * W * C;
        int8_t *ys = y + (size_t)n * P * Q * C;
        // (strips of four that leave most of the chip idle are slower: 12 x 7 x 7 x 2048 3.2 us by the general kernel, 4.1)
        constexpr int kRows = 4;
        if (wide && k == 3 && stride == 1 && mode == 0 && (long long)prm.p.N * ((P + kRows - 1) / kRows) * Q * prm.pieces >= 64 * 1024) {
            Pool3Params strip{};
            strip.p = prm.p;
            strip.pieces = prm.pieces;
            strip.div_pieces = prm.div_pieces;
            strip.div_q = prm.div_q;
            strip.div_strips = make_fastdiv((P + kRows - 1) / kRows);
            strip.total = prm.p.N * strip.div_strips.d * Q * prm.pieces;
            maxpool3_s1_kernel<kRows><<<grid_for((size_t)strip.total), kBlock, 0, st>>>(xs, ys, strip);
            continue;
        }
        const int g = grid_for((size_t)prm.total);
#define DFQ_POOL(V, KK) \
    do { \
        if (mode == 1) pool_kernel<V, KK, true><<<g, kBlock, 0, st>>>(xs, ys, prm); \
        else pool_kernel<V, KK, false><<<g, kBlock, 0, st>>>(xs, ys, prm); \
    } while (0)
        if (wide && k == 2) DFQ_POOL(16, 2);
        else if (wide && k == 3) DFQ_POOL(16, 3);
        else if (wide) DFQ_POOL(16, 0);
        else if (k == 2) DFQ_POOL(4, 2);
        else if (k == 3) DFQ_POOL(4, 3);
        else DFQ_POOL(4, 0);
#undef DFQ_POOL
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// max |.| reductions.  The result scalar is first cleared by a one-lane kernel (not a memset,
// so that the sequence can be captured into a HIP graph), then every workgroup folds its
// share with one atomic max.  Non-negative floats order like their bit patterns.
// ------------------------------------------------------------------------------------------

__global__ void clear_u32(uint32_t *p) { *p = 0u; }

// Every workgroup of a reduction ends with an atomic on the same few words, which serve them one by one: 4096 workgroups over the 2 M
// weights of a layer spent 17 us there, 512 (two per compute unit, each lane with several loads in flight) 5 us.
static inline int grid_for_reduction(size_t work_items)
{
    const int g = grid_for(work_items);
    return g < 512 ? g : 512;
}

// 16 bytes at any boundary of four
template <class T>
struct __attribute__((packed, aligned(4))) Four {
    T v[4];
};

// 16 bytes per lane and access; the first lanes of the launch take the tail.  (50 M values that start 4 bytes behind such a boundary:
// a value per lane and access 170 us, here 36.)
__global__ void __launch_bounds__(kBlock) absmax_f32_kernel(const float *__restrict__ x, size_t n, uint32_t *out)
{
    uint32_t m = 0;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x, threads = (size_t)gridDim.x * kBlock, n4 = n / 4;
    const Four<float> *x4 = (const Four<float> *)x;
#pragma unroll 4
    for (size_t i = t; i < n4; i += threads) {
        const Four<float> q = x4[i];
        m = max(max(m, float_magnitude(q.v[0])), max(float_magnitude(q.v[1]), max(float_magnitude(q.v[2]), float_magnitude(q.v[3]))));
    }
    if (t < n % 4) m = max(m, float_magnitude(x[n4 * 4 + t]));
    block_max_to(m, out);
}

__global__ void __launch_bounds__(kBlock) absmax_i32_kernel(const int32_t *__restrict__ x, size_t n, int relu, uint32_t *out)
{
    uint32_t m = 0;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x, threads = (size_t)gridDim.x * kBlock, n4 = n / 4;
    const Four<int32_t> *x4 = (const Four<int32_t> *)x;
#pragma unroll 4
    for (size_t i = t; i < n4; i += threads) {
        const Four<int32_t> q = x4[i];
        m = max(max(m, magnitude(q.v[0], relu)), max(magnitude(q.v[1], relu), max(magnitude(q.v[2], relu), magnitude(q.v[3], relu))));
    }
    if (t < n % 4) m = max(m, magnitude(x[n4 * 4 + t], relu));
    block_max_to(m, out);
}

__global__ void clear_u32_n(uint32_t *p, int n)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// The same maximum per channel of a [pixels][K] array.  A lane keeps VEC neighbouring channels and walks down the pixels; `lanes` of
// them (at most a wavefront) read a window of a row, a workgroup holds as many rows of its window as fit; they meet in LDS,
// and one lane per channel raises the result.  Windows of 64 lanes and not of the whole workgroup: with the same number of
// workgroups fewer share a channel's word, and few pixels still make several of them (us, a thread per element and
// an atomic per thread / windows of 256 lanes / here: 6272 x 1024 sums 25, 32, 11; 49 x 2048 4.8, 7.4, 5.0; 100352 x 64 311, 20, 18).
template <int VEC>
__global__ void __launch_bounds__(kBlock) absmax_i32_channels_kernel(const int32_t *__restrict__ x, size_t pixels, int K, int relu,
                                                                      uint32_t *out, int lanes, int windows)
{
    __shared__ uint32_t best[kWave * VEC];
    const int chunks = K / VEC;                                         // VEC-channel pieces of a pixel
    const int rows = kBlock / lanes, r = threadIdx.x / lanes, c = threadIdx.x - r * lanes;
    for (int w = blockIdx.y; w < windows; w += gridDim.y) {
        const int c0 = w * lanes, mine = min(chunks - c0, lanes);
        if ((int)threadIdx.x < mine * VEC) best[threadIdx.x] = 0u;      // lanes * VEC <= kBlock
        uint32_t m[VEC];
#pragma unroll
        for (int e = 0; e < VEC; e++) m[e] = 0u;
        if (r < rows && c < mine) {
            const size_t step = (size_t)gridDim.x * rows;
#pragma unroll 4
            for (size_t p = (size_t)blockIdx.x * rows + r; p < pixels; p += step) {
                const int32_t *src = x + p * (size_t)K + (size_t)(c0 + c) * VEC;
                if constexpr (VEC == 4) {
                    const int4 v = *(const int4 *)src;
                    m[0] = max(m[0], magnitude(v.x, relu));
                    m[1] = max(m[1], magnitude(v.y, relu));
                    m[2] = max(m[2], magnitude(v.z, relu));
                    m[3] = max(m[3], magnitude(v.w, relu));
                } else {
                    m[0] = max(m[0], magnitude(*src, relu));
                }
            }
        }
        __syncthreads();
        if (r < rows && c < mine) {
#pragma unroll
            for (int e = 0; e < VEC; e++) atomicMax(&best[c * VEC + e], m[e]);
        }
        __syncthreads();
        if ((int)threadIdx.x < mine * VEC) raise_to(out + (size_t)c0 * VEC + threadIdx.x, best[threadIdx.x], gridDim.x);
        __syncthreads();
    }
}

// max |.| of every row of x[rows][row_len]: one workgroup per row at a time, no atomics
__global__ void __launch_bounds__(kBlock) absmax_f32_rows_kernel(const float *__restrict__ x, size_t rows, size_t row_len, uint32_t *out)
{
    __shared__ uint32_t part[kBlock / kWave];
    for (size_t r = blockIdx.x; r < rows; r += gridDim.x) {
        uint32_t m = 0;
#pragma unroll 4
        for (size_t i = threadIdx.x; i < row_len; i += kBlock) m = max(m, float_magnitude(x[r * row_len + i]));
        m = wave_max_u32(m);
        if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t = part[0];
#pragma unroll
            for (int i = 1; i < kBlock / kWave; i++) t = max(t, part[i]);
            out[r] = t;
        }
        __syncthreads();
    }
}

hipError_t launch_absmax_f32_rows(const float *x, size_t rows, size_t row_len, float *out, hipStream_t st)
{
    size_t g = rows < 4096 ? rows : 4096;
    absmax_f32_rows_kernel<<<(unsigned)g, kBlock, 0, st>>>(x, rows, row_len, (uint32_t *)out);
    return hipGetLastError();
}

hipError_t launch_absmax_f32(const float *x, size_t n, float *out, hipStream_t st)
{
    const int g = n ? grid_for_reduction(n / 4 + 1) : 0;
    if (g != 1) clear_u32<<<1, 1, 0, st>>>((uint32_t *)out);           // one workgroup stores its maximum
    if (g) absmax_f32_kernel<<<g, kBlock, 0, st>>>(x, n, (uint32_t *)out);
    return hipGetLastError();
}

hipError_t launch_absmax_i32(const int32_t *x, size_t n, int relu, uint32_t *out, hipStream_t st)
{
    const int g = n ? grid_for_reduction(n / 4 + 1) : 0;
    if (g != 1) clear_u32<<<1, 1, 0, st>>>(out);                       // one workgroup stores its maximum
    if (g) absmax_i32_kernel<<<g, kBlock, 0, st>>>(x, n, relu, out);
    return hipGetLastError();
}

// Histogram of |x| >> shift over kHistBins bins (Algorithm 1, first step): each workgroup counts its
// share in LDS and adds its non-empty bins to the result, which a small kernel cleared first.  A
// magnitude beyond the last bin (a shift smaller than the caller was told to use) lands in the last bin.
constexpr int kHistBins = 2048;

__global__ void __launch_bounds__(kBlock) hist_i32_kernel(const int32_t *__restrict__ x, size_t n, int relu, int shift, uint32_t *out)
{
    __shared__ uint32_t bins[kHistBins];
    for (int i = threadIdx.x; i < kHistBins; i += kBlock) bins[i] = 0u;
    __syncthreads();
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x, threads = (size_t)gridDim.x * kBlock;
    auto count = [&](int v) { atomicAdd(&bins[min(magnitude(v, relu) >> shift, (uint32_t)(kHistBins - 1))], 1u); };
    size_t n4 = 0;
    if (((uintptr_t)x & 15) == 0) {
        n4 = n / 4;
        const int4 *x4 = (const int4 *)x;
        for (size_t i = t; i < n4; i += threads) {
            const int4 v = x4[i];
            count(v.x); count(v.y); count(v.z); count(v.w);
        }
    }
    for (size_t i = n4 * 4 + t; i < n; i += threads) count(x[i]);
    __syncthreads();
    for (int i = threadIdx.x; i < kHistBins; i += kBlock)
        if (bins[i]) atomicAdd(out + i, bins[i]);
}

hipError_t launch_hist_i32(const int32_t *x, size_t n, int relu, int shift, uint32_t *out, hipStream_t st)
{
    clear_u32_n<<<kHistBins / kBlock, kBlock, 0, st>>>(out, kHistBins);
    if (n) {
        int g = grid_for(n);
        if (g > 1024) g = 1024;                 // every workgroup ends with up to 2048 atomics on the result
        hist_i32_kernel<<<g, kBlock, 0, st>>>(x, n, relu, shift, out);
    }
    return hipGetLastError();
}

hipError_t launch_absmax_i32_channels(const int32_t *x, size_t pixels, int K, int relu, uint32_t *out, hipStream_t st, bool cleared)
{
    const bool vec = K % 4 == 0 && aligned(x, 16);
    const int chunks = vec ? K / 4 : K, windows = (chunks + kWave - 1) / kWave, lanes = (chunks + windows - 1) / windows;
    // four rows per lane or more; two workgroups per compute unit, or four where they are spread over many windows
    const int target = windows < 8 ? 512 : 1024;
    const size_t rows = (size_t)(kBlock / lanes) * 4, full = (pixels + rows - 1) / rows, most = windows < target ? target / windows : 1;
    const unsigned gx = (unsigned)(full < most ? full : most);
    if (gx != 1 && !cleared) clear_u32_n<<<(K + kBlock - 1) / kBlock, kBlock, 0, st>>>(out, K);        // one workgroup stores its maxima
    if (gx) {
        const dim3 grid(gx, (unsigned)(windows < 4096 ? windows : 4096));
        if (vec) absmax_i32_channels_kernel<4><<<grid, kBlock, 0, st>>>(x, pixels, K, relu, out, lanes, windows);
        else absmax_i32_channels_kernel<1><<<grid, kBlock, 0, st>>>(x, pixels, K, relu, out, lanes, windows);
    }
    return hipGetLastError();
}

}  // namespace dfq
