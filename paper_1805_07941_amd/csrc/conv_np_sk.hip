// Dense layers on (8, p) codes whose result is too small to fill the chip with the 128 x 64 tiles of conv_np_mfma_kernel (a few images,
// the late stages, the fully connected layer, calibration batches): the reduction is split inside a workgroup, as conv_sk.hip does for int8.
//
// The layer is the product of conv_np.hip - four int8 matrix products per block into three int32 accumulator sets.  With one image a
// 3x3 x 512 layer at 7 x 7 had 8 workgroups, each walking 72 steps of 64 bytes with a barrier in each (41 us).  Here a workgroup owns
// 16*PT pixels x 16*CT channels; its NW wavefronts take the 128-byte steps v, v + NW, ... of the whole tile, each with a private LDS
// ring filled by direct loads of whole cache lines of the four digit planes and awaited by the count of younger loads; the partial
// sums meet in LDS (integer sums: exact in any order) behind the only barrier, and all threads convert and store four channels each.
// Bound by latency.  One image: 3x3 512 -> 512 at 7 x 7 38.4 -> 6.3 us, fully connected 2048 -> 1000 18.3 -> 4.7 (64 images: 28 -> 6).
#include <type_traits>

#include "conv_ring.hpp"
#include "np_device.hpp"
#include "reduce_device.hpp"

namespace dfq {

namespace {

constexpr int kRow = 128;        // bytes of the reduction axis per step and digit plane: a whole cache line

struct NpSkParams {
    NpConvArgs a;
    int M;            // N*P*Q
    int Kgemm;        // R*S*C
    int nsteps;       // ceil(Kgemm / 128)
    int csteps;       // C / 128
    int nst;          // ring stages in use
    int region;       // bytes of LDS per wavefront
    unsigned x_bytes, w_bytes;
    FastDiv div_tp, div_pq, div_q, div_c, div_s, div_cs;
    int tiles_p;
};

template <int LP, int MAX>
__device__ __forceinline__ void wait_steps(int ahead)
{
    if constexpr (MAX > 0) {
        if (ahead >= MAX) wait_loads<LP * MAX>();
        else wait_steps<LP, MAX - 1>(ahead);
    } else {
        wait_loads<0>();
    }
}

// MODE 0: a step may straddle taps (C a multiple of 64); 1: C a multiple of 128; 2: additionally unpadded 1x1 at stride 1.
template <int PT, int CT, int NW, int NST, int MODE>
__global__ void __launch_bounds__(NW * 64) conv_np_sk_kernel(NpSkParams prm)
{
    constexpr int ROWS = 16 * (PT + CT);               // LDS rows of a digit's part of a stage
    constexpr int LPW = 4 * (PT + CT);                 // loads per wavefront and step
    constexpr int kStage = 2 * ROWS * kRow;
    constexpr int NQ = (PT * CT + NW - 1) / NW;        // groups of four outputs per thread
    static_assert(NST * LPW < 64, "outstanding loads must fit the 6-bit counter");
    extern __shared__ uint4 lds[];
    const NpConvArgs &a = prm.a;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int nmine = prm.nsteps > wave ? (prm.nsteps - wave + NW - 1) / NW : 0;

    // each XCD owns a contiguous range of tiles: the pixel tiles of one channel tile, which read the same weights, share an L2
    const int G = gridDim.x;
    int lb = blockIdx.x;
    {
        const int per = G / 8, rem = G % 8, xcd = lb % 8, idx = lb / 8;
        lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
    }
    const int ct = fastdiv(lb, prm.div_tp);
    const int m0 = (lb - ct * prm.tiles_p) * (16 * PT), k0 = ct * (16 * CT);

    const v4i xh_rsrc = make_rsrc(a.xh, prm.x_bytes), xl_rsrc = make_rsrc(a.xl, prm.x_bytes);
    const v4i wh_rsrc = make_rsrc(a.wh, prm.w_bytes), wl_rsrc = make_rsrc(a.wl, prm.w_bytes);
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char *)(char *)&lds[0];
    const unsigned ring_base = lds_base + (unsigned)(wave * prm.region);

    // ---- what this thread's epilogue will need (group: the four registers of a lane of 16 x 16 block b = c * PT + p)
    int4 bias[NQ];
    uint32_t oh4[NQ], ol4[NQ];
#pragma unroll
    for (int i = 0; i < NQ; i++) {
        const int b = wave + i * NW;
        const int m = m0 + 16 * (b % PT) + l16, kc = k0 + 16 * (b / PT) + 4 * lq;
        const bool live = b < PT * CT && m < prm.M && kc < a.K;            // K is a multiple of 16
        bias[i] = live && a.b ? *(const int4 *)(a.b + kc) : make_int4(0, 0, 0, 0);
        oh4[i] = live && a.oh ? *(const uint32_t *)(a.oh + (size_t)m * a.K + kc) : 0u;
        ol4[i] = live && a.oh ? *(const uint32_t *)(a.ol + (size_t)m * a.K + kc) : 0u;
    }

    // ---- producer: a load covers 8 rows, lane l supplies row l/8, physical piece l%8 = logical piece (l%8) ^ ((row>>1)&7)
    const int lrow = lane >> 3;
    const int lpe = (lane & 7) ^ (lrow >> 1), lpo = (lane & 7) ^ (4 + (lrow >> 1));
    unsigned xoff[2 * PT], woff[2 * CT];
    int ih0[2 * PT], iw0[2 * PT];
#pragma unroll
    for (int j = 0; j < 2 * PT; j++) {
        const int m = m0 + 8 * j + lrow;
        const unsigned piece = (unsigned)((j & 1) ? lpo : lpe) * 16u;
        ih0[j] = iw0[j] = 0;
        if (MODE == 2) {
            xoff[j] = m < prm.M ? (unsigned)(m * a.C) + piece : kOutOfRange;
            continue;
        }
        const int mi = min(m, prm.M - 1);
        const int n = fastdiv(mi, prm.div_pq), pq = mi - n * (a.P * a.Q);
        const int p = fastdiv(pq, prm.div_q), q = pq - p * a.Q;
        ih0[j] = m < prm.M ? p * a.stride - a.pad : -0x10000000;
        iw0[j] = q * a.stride - a.pad;
        xoff[j] = (unsigned)(((n * a.H + p * a.stride - a.pad) * a.W + iw0[j]) * a.C) + (MODE ? piece : 0u);
    }
#pragma unroll
    for (int j = 0; j < 2 * CT; j++) {
        const int k = k0 + 8 * j + lrow;
        woff[j] = k < a.K ? (unsigned)(k * prm.Kgemm) + (unsigned)((j & 1) ? lpo : lpe) * 16u : kOutOfRange;
    }
    auto load_both = [&](unsigned off, const v4i &h, const v4i &l, unsigned at) __attribute__((always_inline)) {
        load_piece_to_lds(off, h, at);
        load_piece_to_lds(off, l, at + (unsigned)(ROWS * kRow));
    };
    auto issue = [&](int i, int stage) __attribute__((always_inline)) {
        const unsigned base = (unsigned)__builtin_amdgcn_readfirstlane((int)(ring_base + (unsigned)(stage * kStage)));
        const int step = wave + NW * i;
        const unsigned skb = (unsigned)step * kRow;
        if (MODE == 2) {
#pragma unroll
            for (int j = 0; j < 2 * PT; j++) load_both(xoff[j] + skb, xh_rsrc, xl_rsrc, base + (unsigned)j * 1024u);
        } else if (MODE == 1) {
            const int tap = fastdiv(step, prm.div_cs);
            const int tr = fastdiv(tap, prm.div_s), ts = tap - tr * a.S;
            const unsigned toff = (unsigned)((tr * a.W + ts) * a.C + (step - tap * prm.csteps) * kRow);
#pragma unroll
            for (int j = 0; j < 2 * PT; j++) {
                const bool in = (unsigned)(ih0[j] + tr) < (unsigned)a.H && (unsigned)(iw0[j] + ts) < (unsigned)a.W;
                load_both(in ? xoff[j] + toff : kOutOfRange, xh_rsrc, xl_rsrc, base + (unsigned)j * 1024u);
            }
        } else {
#pragma unroll
            for (int o = 0; o < 2; o++) {
                const int kb = (int)skb + (o ? lpo : lpe) * 16;                // past the last tap: tr >= R
                const int tap = fastdiv(kb, prm.div_c);
                const int tr = fastdiv(tap, prm.div_s), ts = tap - tr * a.S;
                const unsigned toff = (unsigned)((tr * a.W + ts) * a.C + kb - tap * a.C);
#pragma unroll
                for (int j = o; j < 2 * PT; j += 2) {
                    const bool in = (unsigned)(ih0[j] + tr) < (unsigned)a.H && (unsigned)(iw0[j] + ts) < (unsigned)a.W && tr < a.R;
                    load_both(in ? xoff[j] + toff : kOutOfRange, xh_rsrc, xl_rsrc, base + (unsigned)j * 1024u);
                }
            }
        }
        // (weights past R*S*C of their row are those of the next one, or zeros past the tensor, and meet zeros)
#pragma unroll
        for (int j = 0; j < 2 * CT; j++) load_both(woff[j] + skb, wh_rsrc, wl_rsrc, base + (unsigned)(2 * PT + j) * 1024u);
    };
    const int nst = prm.nst;
    for (int i = 0; i < min(nmine, nst); i++) issue(i, i);

    v4i accA[CT][PT], accB[CT][PT], accC[CT][PT];
#pragma unroll
    for (int c = 0; c < CT; c++)
#pragma unroll
        for (int p = 0; p < PT; p++) accA[c][p] = accB[c][p] = accC[c][p] = v4i{0, 0, 0, 0};

    const int swz = l16 >> 1;
    int stage = 0;
    for (int i = 0; i < nmine; i++) {
        wait_steps<LPW, NST - 1>(min(nmine - 1 - i, nst - 1));
        const v4i *sh = (const v4i *)((const char *)lds + wave * prm.region + stage * kStage), *sl = sh + ROWS * (kRow / 16);
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int g = (4 * h + lq) ^ swz;
            v4i xh[PT], xl[PT], wh[CT], wl[CT];
#pragma unroll
            for (int p = 0; p < PT; p++) {
                xh[p] = sh[(16 * p + l16) * (kRow / 16) + g];
                xl[p] = sl[(16 * p + l16) * (kRow / 16) + g];
            }
#pragma unroll
            for (int c = 0; c < CT; c++) {
                wh[c] = sh[(16 * (PT + c) + l16) * (kRow / 16) + g];
                wl[c] = sl[(16 * (PT + c) + l16) * (kRow / 16) + g];
            }
#pragma unroll
            for (int c = 0; c < CT; c++)
#pragma unroll
                for (int p = 0; p < PT; p++) {
                    accA[c][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh[c], xh[p], accA[c][p], 0, 0, 0);
                    accC[c][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wl[c], xl[p], accC[c][p], 0, 0, 0);
                    accB[c][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh[c], xl[p], accB[c][p], 0, 0, 0);
                    accB[c][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wl[c], xh[p], accB[c][p], 0, 0, 0);
                }
        }
        // the stage is free once its operands are in registers
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + nst < nmine) issue(i + nst, stage);
        stage = stage + 1 == nst ? 0 : stage + 1;
    }

    // ---- the partial sums go to the start of the wavefronts' own LDS regions (every load into them has been awaited)
    const int nactive = min(NW, prm.nsteps);
    if (wave < nactive) {
        v4i *part = (v4i *)((char *)lds + wave * prm.region);
#pragma unroll
        for (int c = 0; c < CT; c++)
#pragma unroll
            for (int p = 0; p < PT; p++) {
                part[64 * (3 * (c * PT + p) + 0) + lane] = accA[c][p];
                part[64 * (3 * (c * PT + p) + 1) + lane] = accB[c][p];
                part[64 * (3 * (c * PT + p) + 2) + lane] = accC[c][p];
            }
    }
    __syncthreads();

    double mx = 0.0;
    const int shift = a.amax ? 0 : a.oh ? a.shift : np_layer_shift(a);
    const NpRound rnd = {shift, a.p_y, (float)a.beta_max, a.relu};
    const NpFast fr = {(unsigned)(1023 + a.p_y + shift), (unsigned)(1023 + shift + 11), ((unsigned)(52 - a.p_y) << 20) | 0x80000u, a.beta_max};
    const NpFast fr2 = {(unsigned)(1023 + a.p_y + a.add_shift), (unsigned)(1023 + a.add_shift + 11), ((unsigned)(52 - a.p_y) << 20) | 0x80000u, a.beta_max};
    const bool fast = shift >= 7 && shift <= 36;
#pragma unroll
    for (int i = 0; i < NQ; i++) {
        const int b = wave + i * NW;
        const int m = m0 + 16 * (b % PT) + l16, kc = k0 + 16 * (b / PT) + 4 * lq;
        if (b >= PT * CT || m >= prm.M || kc >= a.K) continue;
        const int bv[4] = {bias[i].x, bias[i].y, bias[i].z, bias[i].w};
        int A[4], Bm[4], Cc[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            A[e] = 0;
            Bm[e] = bv[e] >> 6;
            Cc[e] = bv[e] & 63;
        }
        for (int u = 0; u < nactive; u++) {
            const v4i *part = (const v4i *)((const char *)lds + u * prm.region) + 64 * 3 * b + lane;
            const v4i ta = part[0], tb = part[64], tc = part[128];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                A[e] += ta[e];
                Bm[e] += tb[e];
                Cc[e] += tc[e];
            }
        }
        if (a.amax) {
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const double v = __builtin_fma((double)((A[e] << 6) + Bm[e]), 64.0, (double)Cc[e]);
                mx = __builtin_fmax(mx, a.relu ? v : __builtin_fabs(v));
            }
            continue;
        }
        uint32_t wc = 0, wh = 0, wl = 0;
        if (a.oh) {
            const int lo1 = a.relu ? 0 : -a.beta_max;
            if (a.add_relu) {
                np_finish_add_one<true, 0>(A[0], Cc[0], Bm[0], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
                np_finish_add_one<true, 1>(A[1], Cc[1], Bm[1], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
                np_finish_add_one<true, 2>(A[2], Cc[2], Bm[2], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
                np_finish_add_one<true, 3>(A[3], Cc[3], Bm[3], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
            } else {
                np_finish_add_one<false, 0>(A[0], Cc[0], Bm[0], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
                np_finish_add_one<false, 1>(A[1], Cc[1], Bm[1], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
                np_finish_add_one<false, 2>(A[2], Cc[2], Bm[2], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
                np_finish_add_one<false, 3>(A[3], Cc[3], Bm[3], oh4[i], ol4[i], lo1, a.add_sa, a.add_sb, fr, fr2, wh, wl);
            }
        } else {
            auto finish = [&](auto f, auto r) __attribute__((always_inline)) {
                constexpr bool F = decltype(f)::value, R = decltype(r)::value;
                np_finish_one<F, R, true, 0>(A[0], Cc[0], Bm[0], rnd, fr, a.p_y, wc, wh, wl);
                np_finish_one<F, R, true, 1>(A[1], Cc[1], Bm[1], rnd, fr, a.p_y, wc, wh, wl);
                np_finish_one<F, R, true, 2>(A[2], Cc[2], Bm[2], rnd, fr, a.p_y, wc, wh, wl);
                np_finish_one<F, R, true, 3>(A[3], Cc[3], Bm[3], rnd, fr, a.p_y, wc, wh, wl);
            };
            if (!fast) finish(std::false_type{}, std::false_type{});
            else if (a.relu) finish(std::true_type{}, std::true_type{});
            else finish(std::true_type{}, std::false_type{});
        }
        const size_t o = (size_t)m * a.K + kc;
        if (a.y) *(uint32_t *)(a.y + o) = wc;
        if (a.yh) *(uint32_t *)(a.yh + o) = wh;
        if (a.yl) *(uint32_t *)(a.yl + o) = wl;
    }
    if (a.amax) block_max_to(a.amax, (unsigned long long)mx, a.amax_words);
}

template <int PT, int CT, int NW, int NST>
hipError_t launch_cfg(const NpConvArgs &a, hipStream_t st)
{
    NpSkParams prm;
    prm.a = a;
    prm.M = a.N * a.P * a.Q;
    prm.Kgemm = a.R * a.S * a.C;
    prm.nsteps = (prm.Kgemm + kRow - 1) / kRow;
    prm.csteps = a.C / kRow;
    prm.tiles_p = (prm.M + 16 * PT - 1) / (16 * PT);
    prm.x_bytes = (unsigned)((long long)a.N * a.H * a.W * a.C);
    prm.w_bytes = (unsigned)((long long)a.K * prm.Kgemm);
    prm.div_tp = make_fastdiv(prm.tiles_p);
    prm.div_pq = make_fastdiv(a.P * a.Q);
    prm.div_q = make_fastdiv(a.Q);
    prm.div_c = make_fastdiv(a.C);
    prm.div_s = make_fastdiv(a.S);
    prm.div_cs = make_fastdiv(prm.csteps > 0 ? prm.csteps : 1);
    const int per_wave = (prm.nsteps + NW - 1) / NW;
    prm.nst = per_wave < NST ? per_wave : NST;
    constexpr int kStage = 2 * 16 * kRow * (PT + CT), kRegionMax = NST * kStage;
    static_assert(3 * PT * CT * 1024 <= kStage, "the partial sums take the place of a stage");
    static_assert(NW * kRegionMax <= kLdsBytes, "the rings do not fit the LDS");
    prm.region = prm.nst * kStage;
    const long long grid = (long long)prm.tiles_p * ((a.K + 16 * CT - 1) / (16 * CT));
    if (grid <= 0) return hipSuccess;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    using K = void (*)(NpSkParams);
    static const K kernels[3] = {conv_np_sk_kernel<PT, CT, NW, NST, 0>, conv_np_sk_kernel<PT, CT, NW, NST, 1>, conv_np_sk_kernel<PT, CT, NW, NST, 2>};
    auto attr_of = [](K k) { return hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, NW * kRegionMax); };
    static const hipError_t attr[3] = {attr_of(kernels[0]), attr_of(kernels[1]), attr_of(kernels[2])};
    const int mode = a.C % kRow ? 0 : (a.R == 1 && a.S == 1 && a.stride == 1 && a.pad == 0) ? 2 : 1;
    if (attr[mode] != hipSuccess) return attr[mode];
    kernels[mode]<<<(unsigned)grid, NW * 64, (size_t)NW * prm.region, st>>>(prm);
    return hipGetLastError();
}

// Fitted to 420 layers of a residual network (1 to 64 images of 96 to 224 pixels), each under every shape and conv_np_mfma_kernel: where
// this kernel is taken the layers take 0.45 of the time in the mean; four are more than 3 % slower, by 13 % at most.
//   up to one 16 x 16 tile per compute unit: those (3x3 512 -> 512 at 7 x 7, one image 38.4 us -> 6.3; 1x1 512 -> 1024, 36 pixels 7.8 -> 4.2);
//   up to one 32 x 32 tile: those with eight wavefronts if the chain is worth splitting (the same layer, eight images 39.2 -> 10.8);
//   else 32 x 32 with four while 6 + n/2 per tile (n steps of 128 bytes) stay below what the other kernel's chain costs, 100 (20 + 6 n):
//   3x3 512 -> 512, sixteen images 40.1 -> 17.2; at the line 3x3 256 -> 256 at 14 x 14, sixteen images 22.0 -> 20.1 and 1x1 512 -> 1024,
//   676 pixels 8.7, here 9.3.
// A calibration's maximum into a single word costs more per workgroup than it saves (one image, 512 -> 2048: 9.6, here 11.7).
enum class Shape { none, t16, t32x8, t32x4 };

Shape choose(const NpConvArgs &a)
{
    if (a.amax && a.amax_words == 1) return Shape::none;
    const long long M = (long long)a.N * a.P * a.Q;
    const long long t16 = ((M + 15) / 16) * ((a.K + 15) / 16), t32 = ((M + 31) / 32) * ((a.K + 31) / 32);
    const int n = (a.R * a.S * a.C + kRow - 1) / kRow;
    if (t16 <= kNumCU && n > 1) return Shape::t16;
    if (t32 <= kNumCU && n > 4) return Shape::t32x8;
    return t32 * (12 + n) <= 200LL * (20 + 6 * n) ? Shape::t32x4 : Shape::none;
}

}  // namespace

bool conv_np_sk_pays(const NpConvArgs &a) { return choose(a) != Shape::none; }

hipError_t launch_conv_np_sk(const NpConvArgs &a, hipStream_t st)
{
    switch (choose(a)) {
        case Shape::t16: return launch_cfg<1, 1, 8, 2>(a, st);
        case Shape::t32x8: return launch_cfg<2, 2, 8, 1>(a, st);
        default: return launch_cfg<2, 2, 4, 1>(a, st);
    }
}

}  // namespace dfq
