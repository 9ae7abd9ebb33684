// Calibration (Sec. 3) with the formats chosen on the device.  A layer's output format follows from the largest of its 32-bit sums;
// read back to the host, that number costs a synchronization per layer with the chip idle around it (MobileNet-shaped network, 8
// images, per channel: 4.0 ms for 1.1 ms of kernels).  Here the maxima, the formats that follow from them and the rescale that
// uses them stay on the device: every kernel below derives the format it needs from device words - each workgroup for itself, from at
// most a few thousand words in L2 - and the first workgroup stores it for the kernels and the host behind.  The sums a layer's
// maximum is taken over are rescaled themselves (a streaming pass over 4 B per output) instead of running the layer again.
// Every kernel is bound by launch latency or memory; 16-byte accesses where the layout has them.
#include "dfq_host.hpp"
#include "conv_epilogue.hpp"
#include "np_device.hpp"
#include "reduce_device.hpp"

namespace dfq {

namespace {

inline int blocks_for(size_t work, size_t per_block, size_t most)
{
    const size_t b = (work + per_block - 1) / per_block;
    return (int)(b < 1 ? 1 : b > most ? most : b);
}

// The largest f in [-32, 32] with gamma * 2^f <= top, gamma given by its bits, top = top_mant * 2^top_exp, top_mant in [1/2, 1).  gamma =
// m * 2^e with m in [1/2, 1): f = top_exp - e, one less when m > top_mant.  (dfq_fmt_from_absmax_f32, dfq_np_frac_from_absmax_f32)
__device__ __forceinline__ int frac_from_float(uint32_t gamma_bits, float top_mant, int top_exp)
{
    const float g = __uint_as_float(gamma_bits);
    if (!(g > 0.0f)) return 32;
    int e;
    const float m = frexpf(g, &e);
    return min(max(top_exp - e - (m > top_mant ? 1 : 0), -32), 32);
}

__device__ __forceinline__ bool is_infinite(uint32_t gamma_bits) { return gamma_bits >= 0x7f800000u; }

// ---- weights and bias of a layer: one wavefront per output channel ---------------------------------------------------
// PER_ROW: the format of a channel from its own maximum; else the layer's, from the rows' maxima in gamma.
template <bool PER_ROW>
__device__ __forceinline__ uint32_t weight_threshold(const float *__restrict__ row, size_t row_len, const uint32_t *__restrict__ gamma, size_t rows, int lane)
{
    uint32_t m = 0;
    if (PER_ROW) {
#pragma unroll 4
        for (size_t i = lane; i < row_len; i += kWave) m = max(m, float_magnitude(row[i]));
    } else {
#pragma unroll 4
        for (size_t i = lane; i < rows; i += kWave) m = max(m, gamma[i]);
    }
    return wave_max_u32(m);
}

template <bool PER_ROW>
__global__ void __launch_bounds__(kBlock) cal_weights_kernel(const float *__restrict__ w, const float *__restrict__ bias, size_t rows, size_t row_len,
                                                              const uint32_t *__restrict__ gamma, const int32_t *__restrict__ frac_in,
                                                              int8_t *__restrict__ q, int32_t *__restrict__ w_frac, int32_t *__restrict__ b,
                                                              int32_t *err, int vec)
{
    const int lane = threadIdx.x % kWave;
    const size_t r = (size_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (r >= rows) return;
    const float *row = w + r * row_len;
    const uint32_t m = weight_threshold<PER_ROW>(row, row_len, gamma, rows, lane);
    const int f = frac_from_float(m, 127.0f / 128.0f, 7);
    const float scale = ldexpf(1.0f, f);
    if (vec) {
        const float4 *row4 = (const float4 *)row;
        uint32_t *q4 = (uint32_t *)(q + r * row_len);
        for (size_t i = lane; i < row_len / 4; i += kWave) {
            const float4 v = row4[i];
            q4[i] = pack4(quant_one(v.x, scale), quant_one(v.y, scale), quant_one(v.z, scale), quant_one(v.w, scale));
        }
    } else {
        for (size_t i = lane; i < row_len; i += kWave) q[r * row_len + i] = (int8_t)quant_one(row[i], scale);
    }
    if (lane == 0) {
        if (PER_ROW || r == 0) {
            w_frac[PER_ROW ? r : 0] = f;
            if (is_infinite(m)) atomicOr(err, 1);
        }
        b[r] = quant_i32_one(bias[r], f + *frac_in);
    }
}

// The same for a layer on (8, p) codes (one format per layer): codes, their digit planes and the bias.
__global__ void __launch_bounds__(kBlock) cal_np_weights_kernel(const float *__restrict__ w, const float *__restrict__ bias, size_t rows, size_t row_len,
                                                                 const uint32_t *__restrict__ gamma, const int32_t *__restrict__ frac_in, NpFmt fmt,
                                                                 float top_mant, int top_exp, uint8_t *__restrict__ codes, int8_t *__restrict__ hi,
                                                                 int8_t *__restrict__ lo, int32_t *__restrict__ w_frac, int32_t *__restrict__ b,
                                                                 int32_t *err, int vec)
{
    const int lane = threadIdx.x % kWave;
    const size_t r = (size_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (r >= rows) return;
    const float *row = w + r * row_len;
    const uint32_t m = weight_threshold<false>(row, row_len, gamma, rows, lane);
    const int f = frac_from_float(m, top_mant, top_exp);
    fmt.scale = ldexpf(1.0f, f);
    if (vec) {
        const float4 *row4 = (const float4 *)row;
        for (size_t i = lane; i < row_len / 4; i += kWave) {
            const float4 v4 = row4[i];
            const float v[4] = {v4.x, v4.y, v4.z, v4.w};
            uint32_t c4 = 0, h4 = 0, l4 = 0;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t c = np_quant_one(v[e], fmt);
                int h, l;
                np_split(np_beta_of(c, fmt.p), h, l);
                c4 |= c << (8 * e);
                h4 |= ((uint32_t)h & 0xffu) << (8 * e);
                l4 |= ((uint32_t)l & 0xffu) << (8 * e);
            }
            ((uint32_t *)(codes + r * row_len))[i] = c4;
            ((uint32_t *)(hi + r * row_len))[i] = h4;
            ((uint32_t *)(lo + r * row_len))[i] = l4;
        }
    } else {
        for (size_t i = lane; i < row_len; i += kWave) {
            const uint32_t c = np_quant_one(row[i], fmt);
            int h, l;
            np_split(np_beta_of(c, fmt.p), h, l);
            codes[r * row_len + i] = (uint8_t)c;
            hi[r * row_len + i] = (int8_t)h;
            lo[r * row_len + i] = (int8_t)l;
        }
    }
    if (lane == 0) {
        if (r == 0) {
            *w_frac = f;
            if (is_infinite(m)) atomicOr(err, 1);
        }
        b[r] = quant_i32_one(bias[r], f + *frac_in);
    }
}

// ---- input ---------------------------------------------------------------------------------------------------------

__global__ void __launch_bounds__(kBlock) cal_quantize_kernel(const float *__restrict__ x, size_t n, const uint32_t *__restrict__ gamma,
                                                               int8_t *__restrict__ q, int32_t *__restrict__ frac, int32_t *err, int vec)
{
    const uint32_t m = *gamma;
    const int f = frac_from_float(m, 127.0f / 128.0f, 7);
    const float scale = ldexpf(1.0f, f);
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x, threads = (size_t)gridDim.x * kBlock, n4 = vec ? n / 4 : 0;
    for (size_t i = t; i < n4; i += threads) {
        const float4 v = ((const float4 *)x)[i];
        ((uint32_t *)q)[i] = pack4(quant_one(v.x, scale), quant_one(v.y, scale), quant_one(v.z, scale), quant_one(v.w, scale));
    }
    for (size_t i = n4 * 4 + t; i < n; i += threads) q[i] = (int8_t)quant_one(x[i], scale);
    if (t == 0) {
        *frac = f;
        if (is_infinite(m)) atomicOr(err, 1);
    }
}

__global__ void __launch_bounds__(kBlock) cal_np_quantize_kernel(const float *__restrict__ x, size_t n, const uint32_t *__restrict__ gamma, NpFmt fmt,
                                                                  float top_mant, int top_exp, int8_t *__restrict__ hi, int8_t *__restrict__ lo,
                                                                  int32_t *__restrict__ frac, int32_t *err)
{
    const uint32_t m = *gamma;
    const int f = frac_from_float(m, top_mant, top_exp);
    fmt.scale = ldexpf(1.0f, f);
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x, threads = (size_t)gridDim.x * kBlock;
    for (size_t i = t; i < n; i += threads) {
        int h, l;
        np_split(np_beta_of(np_quant_one(x[i], fmt), fmt.p), h, l);
        hi[i] = (int8_t)h;
        lo[i] = (int8_t)l;
    }
    if (t == 0) {
        *frac = f;
        if (is_infinite(m)) atomicOr(err, 1);
    }
}

// ---- a layer's sums ------------------------------------------------------------------------------------------------

struct CalConvParams {
    const int32_t *acc;
    size_t pixels;
    int K, relu;
    const int32_t *frac_in, *w_frac;
    int w_step;                  // 1: a format per channel, 0: one
    const uint32_t *maxima;      // of every channel
    int fixed, fixed_frac;
    int8_t *y;
    int32_t *frac_out;
    int vec;                     // K % 4 == 0 and aligned: four channels per lane
};

__global__ void __launch_bounds__(kBlock) cal_rescale_kernel(CalConvParams p)
{
    __shared__ int part[kBlock / kWave];
    const int f_in = *p.frac_in;
    int f = p.fixed_frac;
    if (!p.fixed) {
        f = 32;
        for (int k = threadIdx.x; k < p.K; k += kBlock) f = min(f, frac_from_int(p.maxima[k], f_in + p.w_frac[k * p.w_step], 127u));
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) f = min(f, __shfl_xor(f, o, kWave));
        if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = f;
        __syncthreads();
        f = min(min(part[0], part[1]), min(part[2], part[3]));
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *p.frac_out = f;
    const int base = f_in - f;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x, threads = (size_t)gridDim.x * kBlock;
    const int kv = p.vec ? p.K / 4 : p.K;                 // pieces of a pixel
    const size_t total = p.pixels * (size_t)kv;
    int k = (int)(t % (size_t)kv);
    const int step = (int)(threads % (size_t)kv);
    for (size_t i = t; i < total; i += threads) {
        if (p.vec) {
            const int4 v4 = ((const int4 *)p.acc)[i];
            const int v[4] = {v4.x, v4.y, v4.z, v4.w};
            int o[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                ChannelRequant cr;
                cr.init(base + p.w_frac[(4 * k + e) * p.w_step]);
                o[e] = cr.apply(v[e], p.relu);
            }
            ((uint32_t *)p.y)[i] = pack4(o[0], o[1], o[2], o[3]);
        } else {
            ChannelRequant cr;
            cr.init(base + p.w_frac[k * p.w_step]);
            p.y[i] = (int8_t)cr.apply(p.acc[i], p.relu);
        }
        k += step;
        if (k >= kv) k -= kv;
    }
}

// ---- element-wise add (Eq. 10) -------------------------------------------------------------------------------------

// left shifts of the two operands to the finer scale, at most `most` (beyond: the call is refused at the end, err)
__device__ __forceinline__ int align_shifts(const int32_t *fa, const int32_t *fb, int most, int &sa, int &sb, int32_t *err)
{
    const int a = *fa, b = *fb, F = max(a, b);
    sa = F - a;
    sb = F - b;
    if (max(sa, sb) > most) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(err, 2);
        sa = min(sa, most);
        sb = min(sb, most);
    }
    return F;
}

// four neighbouring values by one word where the operands are aligned
template <class F>
__device__ __forceinline__ void each_four(const int8_t *a, const int8_t *b, size_t n, int vec, F &&f)
{
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x, threads = (size_t)gridDim.x * kBlock, n4 = vec ? n / 4 : 0;
    for (size_t i = t; i < n4; i += threads) {
        const uint32_t wa = ((const uint32_t *)a)[i], wb = ((const uint32_t *)b)[i];
        const int va[4] = {byte_of(wa, 0), byte_of(wa, 1), byte_of(wa, 2), byte_of(wa, 3)};
        const int vb[4] = {byte_of(wb, 0), byte_of(wb, 1), byte_of(wb, 2), byte_of(wb, 3)};
        f(va, vb, i * 4, 4);
    }
    for (size_t i = n4 * 4 + t; i < n; i += threads) {
        const int va[4] = {a[i], 0, 0, 0}, vb[4] = {b[i], 0, 0, 0};
        f(va, vb, i, 1);
    }
}

__global__ void __launch_bounds__(kBlock) cal_add_max_kernel(const int8_t *__restrict__ a, const int8_t *__restrict__ b, const int32_t *fa,
                                                              const int32_t *fb, size_t n, int relu, uint32_t *out, int32_t *err, int vec)
{
    int sa, sb;
    align_shifts(fa, fb, 22, sa, sb, err);
    uint32_t m = 0;
    each_four(a, b, n, vec, [&](const int (&va)[4], const int (&vb)[4], size_t, int) {
#pragma unroll
        for (int e = 0; e < 4; e++) m = max(m, magnitude((int)(((unsigned)va[e] << sa) + ((unsigned)vb[e] << sb)), relu));
    });
    block_max_to(m, out);
}

__global__ void __launch_bounds__(kBlock) cal_add_kernel(const int8_t *__restrict__ a, const int8_t *__restrict__ b, const int32_t *fa, const int32_t *fb,
                                                          size_t n, int relu, const uint32_t *maximum, int8_t *__restrict__ y, int32_t *frac_out,
                                                          int32_t *err, int vec)
{
    int sa, sb;
    const int F = align_shifts(fa, fb, 22, sa, sb, err);
    const int f = frac_from_int(*maximum, F, 127u);
    if (blockIdx.x == 0 && threadIdx.x == 0) *frac_out = f;
    ChannelRequant cr;
    cr.init(F - f);
    each_four(a, b, n, vec, [&](const int (&va)[4], const int (&vb)[4], size_t i, int count) {
        int o[4];
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = cr.apply((int)(((unsigned)va[e] << sa) + ((unsigned)vb[e] << sb)), relu);
        if (count == 4) *(uint32_t *)(y + i) = pack4(o[0], o[1], o[2], o[3]);
        else y[i] = (int8_t)o[0];
    });
}

}  // namespace

hipError_t launch_cal_weights(const float *w, const float *bias, size_t rows, size_t row_len, int per_row, float *gamma, const int32_t *frac_in,
                              int8_t *q, int32_t *w_frac, int32_t *b, int32_t *err, hipStream_t st)
{
    const int vec = row_len % 4 == 0 && (((uintptr_t)w & 15) | ((uintptr_t)q & 3)) == 0;
    const unsigned grid = (unsigned)((rows + kBlock / kWave - 1) / (kBlock / kWave));
    if (per_row) {
        cal_weights_kernel<true><<<grid, kBlock, 0, st>>>(w, bias, rows, row_len, nullptr, frac_in, q, w_frac, b, err, vec);
    } else {
        const hipError_t e = launch_absmax_f32_rows(w, rows, row_len, gamma, st);
        if (e != hipSuccess) return e;
        cal_weights_kernel<false><<<grid, kBlock, 0, st>>>(w, bias, rows, row_len, (const uint32_t *)gamma, frac_in, q, w_frac, b, err, vec);
    }
    return hipGetLastError();
}

hipError_t launch_cal_np_weights(const float *w, const float *bias, size_t rows, size_t row_len, int p, int beta_max, float *gamma,
                                 const int32_t *frac_in, uint8_t *codes, int8_t *hi, int8_t *lo, int32_t *w_frac, int32_t *b, int32_t *err,
                                 hipStream_t st)
{
    const int vec = row_len % 4 == 0 && (((uintptr_t)w & 15) | (((uintptr_t)codes | (uintptr_t)hi | (uintptr_t)lo) & 3)) == 0;
    const hipError_t e = launch_absmax_f32_rows(w, rows, row_len, gamma, st);
    if (e != hipSuccess) return e;
    int top_exp = 0;
    const float top_mant = frexpf((float)beta_max, &top_exp);
    const NpFmt fmt{8, p, 1.0f, (float)beta_max};
    cal_np_weights_kernel<<<(unsigned)((rows + kBlock / kWave - 1) / (kBlock / kWave)), kBlock, 0, st>>>(
        w, bias, rows, row_len, (const uint32_t *)gamma, frac_in, fmt, top_mant, top_exp, codes, hi, lo, w_frac, b, err, vec);
    return hipGetLastError();
}

hipError_t launch_cal_quantize(const float *x, size_t n, float *gamma, int8_t *q, int32_t *frac, int32_t *err, hipStream_t st)
{
    const hipError_t e = launch_absmax_f32(x, n, gamma, st);
    if (e != hipSuccess) return e;
    const int vec = (((uintptr_t)x & 15) | ((uintptr_t)q & 3)) == 0;
    cal_quantize_kernel<<<blocks_for(n, 4 * kBlock, 4096), kBlock, 0, st>>>(x, n, (const uint32_t *)gamma, q, frac, err, vec);
    return hipGetLastError();
}

hipError_t launch_cal_np_quantize(const float *x, size_t n, int p, int beta_max, float *gamma, int8_t *hi, int8_t *lo, int32_t *frac, int32_t *err,
                                  hipStream_t st)
{
    const hipError_t e = launch_absmax_f32(x, n, gamma, st);
    if (e != hipSuccess) return e;
    int top_exp = 0;
    const float top_mant = frexpf((float)beta_max, &top_exp);
    const NpFmt fmt{8, p, 1.0f, (float)beta_max};
    cal_np_quantize_kernel<<<blocks_for(n, 2 * kBlock, 4096), kBlock, 0, st>>>(x, n, (const uint32_t *)gamma, fmt, top_mant, top_exp, hi, lo, frac, err);
    return hipGetLastError();
}

hipError_t launch_cal_rescale(const int32_t *acc, size_t pixels, int K, int relu, const int32_t *frac_in, const int32_t *w_frac, int per_channel,
                              uint32_t *maxima, int fixed, int fixed_frac, int8_t *y, int32_t *frac_out, hipStream_t st)
{
    if (!fixed) {
        const hipError_t e = launch_absmax_i32_channels(acc, pixels, K, relu, maxima, st, true);
        if (e != hipSuccess) return e;
    }
    CalConvParams p{acc, pixels, K, relu, frac_in, w_frac, per_channel ? 1 : 0, maxima, fixed, fixed_frac, y, frac_out, 0};
    p.vec = K % 4 == 0 && (((uintptr_t)acc & 15) | ((uintptr_t)y & 3)) == 0;
    // (eight pieces per lane: every workgroup looks the layer's maxima through first)
    cal_rescale_kernel<<<blocks_for(pixels * (size_t)(p.vec ? K / 4 : K), 8 * kBlock, 2048), kBlock, 0, st>>>(p);
    return hipGetLastError();
}

hipError_t launch_cal_add(const int8_t *a, const int32_t *fa, const int8_t *b, const int32_t *fb, size_t n, int relu, uint32_t *maximum, int8_t *y,
                          int32_t *frac_out, int32_t *err, hipStream_t st)
{
    const int vec = (((uintptr_t)a | (uintptr_t)b | (uintptr_t)y) & 3) == 0;
    // (`maximum` starts at zero, and one workgroup alone stores its own)
    cal_add_max_kernel<<<blocks_for(n, 16 * kBlock, 512), kBlock, 0, st>>>(a, b, fa, fb, n, relu, maximum, err, vec);
    cal_add_kernel<<<blocks_for(n, 8 * kBlock, 4096), kBlock, 0, st>>>(a, b, fa, fb, n, relu, maximum, y, frac_out, err, vec);
    return hipGetLastError();
}

}  // namespace dfq
