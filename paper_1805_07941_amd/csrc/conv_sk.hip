// Dense layers whose result is too small to fill the chip with the tiles of the general kernel (a few images, the late
// stages, fully connected layers) on the gfx950 int8 matrix cores: the reduction is split inside a workgroup.
//
// The sum of Eq. 6 for groups == 1 is the matrix product acc[k][m] = sum_j W[k][j] * X[m][j], j over the R*S*C (tap,
// channel) pairs.  For a 14 x 14 image and 256 channels that is 0.2 GOP over less than 1 MB: a microsecond of anything.
// What decides the time is how many compute units take part, how long the serial chain of steps is that each of them walks,
// and how fast one compute unit can fetch: with 64 x 64 tiles and four wavefronts that share every 64-byte step such a 3x3
// layer had 16 workgroups walking 36 steps with a barrier in each.  Here a workgroup owns one tile of 16*PT pixels x 16*CT
// channels, and its NW wavefronts split the reduction axis: wavefront v takes the 128-byte steps v, v + NW, ... of the whole
// tile alone, with a private LDS ring filled by direct loads and awaited by the count of younger loads, so that nothing is
// shared until the end, when the partial sums meet in LDS (integer sums: exact in any order) behind the only barrier.  All
// threads then add, rescale and store four consecutive channels each; what they need for that (bias, formats, the operand of
// a fused add) was fetched before the ring was started.  Steps of whole 128-byte lines: a compute unit draws twice as much
// from L2 as in 64-byte rows.
// The epilogue takes any shift, ragged channel tail, pitch, accumulator dump, one weight format per channel and the add.
//
// Measured (one layer among others, weights not in L2): 3x3 256 -> 256 at 14 x 14, one image 10.3 -> 4.1 us; 3x3 512 -> 512
// at 7 x 7, one image 17.0 -> 5.0, twelve images 17.0 -> 9.7; 1x1 2048 -> 512 at 7 x 7, twelve images 11.3 -> 6.5; fully
// connected 2048 -> 1000, one image 7.5 -> 4.0, 32 images 8.0 -> 4.2.
#include "conv_ring.hpp"

namespace dfq {

namespace {

constexpr int kRow = 128;        // bytes of the reduction axis per step: a whole cache line of every row

struct SkParams {
    ConvArgs a;
    int M;            // N*P*Q
    int Kgemm;        // R*S*C
    int nsteps;       // ceil(Kgemm / 128)
    int csteps;       // C / 128 (whole steps per tap)
    int nst;          // ring stages in use, 1 .. NST
    int region;       // bytes of LDS per wavefront
    unsigned x_bytes, w_bytes;
    FastDiv div_tp, div_pq, div_q, div_c, div_s, div_cs;
    int tiles_p;      // pixel tiles
    int words;        // four channels of an output pixel are one aligned word of y
};

// wait until only the loads of the next `ahead` (0 .. MAX) steps, LP each, are outstanding
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

// MODE 0: C a multiple of 16, a step may straddle taps; 1: C a multiple of 128, one tap per step; 2: additionally unpadded
// 1x1 at stride 1, output pixel m reads input pixel m.
template <int PT, int CT, int NW, int NST, int MODE>
__global__ void __launch_bounds__(NW * 64) conv_sk_kernel(SkParams prm)
{
    constexpr int LPW = 2 * (PT + CT);                 // loads per wavefront and step
    constexpr int kStage = 16 * kRow * (PT + CT);
    constexpr int NQ = (PT * CT * 64 + NW * 64 - 1) / (NW * 64);   // groups of four outputs per thread
    static_assert(NST * LPW < 64, "outstanding loads must fit the 6-bit counter");
    extern __shared__ uint4 lds[];
    const ConvArgs &a = prm.a;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int nmine = prm.nsteps > wave ? (prm.nsteps - wave + NW - 1) / NW : 0;    // steps wave, wave + NW, ...

    // Workgroup ids are dealt round-robin to the 8 XCDs; renumbered so that each XCD owns a contiguous range, the pixel
    // tiles of one channel tile - which read the same weight rows - share an L2.
    const int G = gridDim.x;
    int lb = blockIdx.x;
    {
        const int per = G / 8, rem = G % 8, xcd = lb % 8, idx = lb / 8;
        lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
    }
    const int ct = fastdiv(lb, prm.div_tp);
    const int m0 = (lb - ct * prm.tiles_p) * (16 * PT), k0 = ct * (16 * CT);

    const v4i xrsrc = make_rsrc(a.x, prm.x_bytes);
    const v4i wrsrc = make_rsrc(a.w, prm.w_bytes);
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char *)(char *)&lds[0];
    const unsigned ring_base = lds_base + (unsigned)(wave * prm.region);

    // ---- what the epilogue of this thread will need.  Group g of the tile: the four accumulator registers of lane g % 64 of
    // 16x16 block b = g / 64 = c * PT + p, i.e. channels kc .. kc+3 of pixel m.
    int bias[NQ][4], fw[NQ][4];
    uint32_t other[NQ];
#pragma unroll
    for (int i = 0; i < NQ; i++) {
        const int b = wave + i * NW;
        const int m = m0 + 16 * (b % PT) + l16, kc = k0 + 16 * (b / PT) + 4 * lq;
        const bool live = b < PT * CT && m < prm.M;
        other[i] = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const bool on = live && kc + e < a.K;
            bias[i][e] = (on && a.b) ? a.b[kc + e] : 0;
            fw[i][e] = (on && a.frac_w) ? a.frac_w[kc + e] : 0;
        }
        if (live && a.add && kc < a.K) other[i] = *(const uint32_t *)(a.add + (size_t)m * a.ldadd + kc);   // words: conv_sk_supports()
    }

    // ---- producer.  A wavefront-wide load covers 8 rows of a stage: lane l supplies row l/8, physical piece l%8, which holds
    // logical piece (l%8) ^ ((row>>1)&7), so that 16 consecutive rows put any one logical piece on 16 different bank groups.
    // Chunk j holds rows 8j .. 8j+7, so the bits of the row are those of lane/8 and j.
    const int lrow = lane >> 3;
    const int lpe = (lane & 7) ^ (lrow >> 1), lpo = (lane & 7) ^ (4 + (lrow >> 1));    // logical piece in even and odd chunks
    unsigned xoff[2 * PT], woff[2 * CT];      // byte offset of the lane's row (+ piece where MODE > 0), or out of range: zeros arrive
    int ih0[2 * PT], iw0[2 * PT];             // input coordinates of tap (0, 0)
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
        ih0[j] = m < prm.M ? p * a.stride - a.pad : -0x10000000;              // rows past the last pixel: outside for every tap
        iw0[j] = q * a.stride - a.pad;
        xoff[j] = (unsigned)(((n * a.H + p * a.stride - a.pad) * a.W + iw0[j]) * a.C) + (MODE ? piece : 0u);
    }
#pragma unroll
    for (int j = 0; j < 2 * CT; j++) {
        const int k = k0 + 8 * j + lrow;
        woff[j] = k < a.K ? (unsigned)(k * prm.Kgemm) + (unsigned)((j & 1) ? lpo : lpe) * 16u : kOutOfRange;
    }
    // this wavefront's i-th step into stage `stage` of its ring
    auto issue = [&](int i, int stage) __attribute__((always_inline)) {
        const unsigned base = (unsigned)__builtin_amdgcn_readfirstlane((int)(ring_base + (unsigned)(stage * kStage)));
        const int step = wave + NW * i;
        const unsigned skb = (unsigned)step * kRow;
        if (MODE == 2) {
#pragma unroll
            for (int j = 0; j < 2 * PT; j++) load_piece_to_lds(xoff[j] + skb, xrsrc, base + (unsigned)j * 1024u);
        } else if (MODE == 1) {
            const int tap = fastdiv(step, prm.div_cs);
            const int tr = fastdiv(tap, prm.div_s), ts = tap - tr * a.S;
            const unsigned toff = (unsigned)((tr * a.W + ts) * a.C + (step - tap * prm.csteps) * kRow);
#pragma unroll
            for (int j = 0; j < 2 * PT; j++) {
                const bool in = (unsigned)(ih0[j] + tr) < (unsigned)a.H && (unsigned)(iw0[j] + ts) < (unsigned)a.W;
                load_piece_to_lds(in ? xoff[j] + toff : kOutOfRange, xrsrc, base + (unsigned)j * 1024u);
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
                    load_piece_to_lds(in ? xoff[j] + toff : kOutOfRange, xrsrc, base + (unsigned)j * 1024u);
                }
            }
        }
        // (weights past R*S*C of their row are those of the next one and meet zeros)
#pragma unroll
        for (int j = 0; j < 2 * CT; j++) load_piece_to_lds(woff[j] + skb, wrsrc, base + (unsigned)(2 * PT + j) * 1024u);
    };
    const int nst = prm.nst;
    for (int i = 0; i < min(nmine, nst); i++) issue(i, i);

    v4i acc[CT][PT];
#pragma unroll
    for (int c = 0; c < CT; c++)
#pragma unroll
        for (int p = 0; p < PT; p++) acc[c][p] = v4i{0, 0, 0, 0};

    const int swz = l16 >> 1;
    int stage = 0;
    for (int i = 0; i < nmine; i++) {
        wait_steps<LPW, NST - 1>(min(nmine - 1 - i, nst - 1));
        const v4i *st = (const v4i *)((const char *)lds + wave * prm.region + stage * kStage);
        v4i x[2][PT], w[2][CT];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int g = (4 * h + lq) ^ swz;
#pragma unroll
            for (int p = 0; p < PT; p++) x[h][p] = st[(16 * p + l16) * (kRow / 16) + g];
#pragma unroll
            for (int c = 0; c < CT; c++) w[h][c] = st[(16 * (PT + c) + l16) * (kRow / 16) + g];
        }
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int c = 0; c < CT; c++)
#pragma unroll
                for (int p = 0; p < PT; p++) acc[c][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[h][c], x[h][p], acc[c][p], 0, 0, 0);
        // the stage is free once its operands are in registers
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + nst < nmine) issue(i + nst, stage);
        stage = stage + 1 == nst ? 0 : stage + 1;
    }

    // ---- the partial sums go to the start of the wavefronts' own LDS regions (every load into them has been awaited), the
    // four registers of lane l of block b at 16-byte word 64*b + l
    const int nactive = min(NW, prm.nsteps);
    if (wave < nactive) {
        v4i *part = (v4i *)((char *)lds + wave * prm.region);
#pragma unroll
        for (int c = 0; c < CT; c++)
#pragma unroll
            for (int p = 0; p < PT; p++) part[64 * (c * PT + p) + lane] = acc[c][p];
    }
    __syncthreads();

    Requant rq2;
    rq2.init(a.add ? a.add_shift : 1, a.add_relu);
#pragma unroll
    for (int i = 0; i < NQ; i++) {
        const int b = wave + i * NW;
        const int m = m0 + 16 * (b % PT) + l16, kc = k0 + 16 * (b / PT) + 4 * lq;
        if (b >= PT * CT || m >= prm.M || kc >= a.K) continue;
        int v[4] = {bias[i][0], bias[i][1], bias[i][2], bias[i][3]};
        for (int u = 0; u < nactive; u++) {
            const v4i t = ((const v4i *)((const char *)lds + u * prm.region))[64 * b + lane];
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = (int)((unsigned)v[e] + (unsigned)t[e]);
        }
        if (a.acc_out) {
            if ((a.K & 3) == 0) {
                *(int4 *)(a.acc_out + (size_t)m * a.K + kc) = make_int4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (kc + e < a.K) a.acc_out[(size_t)m * a.K + kc + e] = v[e];
            }
        }
        if (!a.y) continue;
        int q[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            ChannelRequant cr;
            cr.init(a.shift + fw[i][e]);
            q[e] = cr.apply(v[e], a.relu);
        }
        if (a.add) {
            constexpr int kBound = (127 << 23) + (1 << 29);      // see add_tile_lane_lazy
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const unsigned mine = a.add_lazy ? (unsigned)max(-kBound, min(kBound, v[e])) : (unsigned)q[e] << a.add_sa;
                q[e] = rq2.fast_one((int)(mine + ((unsigned)byte_of(other[i], e) << a.add_sb)));
            }
        }
        int8_t *dst = a.y + (size_t)m * a.ldy + kc;
        const uint32_t word = pack4_clamped(q[0], q[1], q[2], q[3]);
        if (prm.words && kc + 4 <= a.K) {
            *(uint32_t *)dst = word;
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++)
                if (kc + e < a.K) dst[e] = (int8_t)(word >> (8 * e));
        }
    }
}

template <int PT, int CT, int NW, int NST>
hipError_t launch_cfg(const ConvArgs &a, hipStream_t st)
{
    SkParams prm;
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
    prm.words = (a.ldy & 3) == 0 && ((uintptr_t)a.y & 3) == 0;
    const int per_wave = (prm.nsteps + NW - 1) / NW;
    prm.nst = per_wave < NST ? per_wave : NST;
    constexpr int kStage = 16 * kRow * (PT + CT), kRegionMax = NST * kStage;
    static_assert(PT * CT * 1024 <= kStage, "the partial sums take the place of a stage");
    static_assert(NW * kRegionMax <= kLdsBytes, "the rings do not fit the LDS");
    prm.region = prm.nst * kStage;
    const long long grid = (long long)prm.tiles_p * ((a.K + 16 * CT - 1) / (16 * CT));
    if (grid <= 0) return hipSuccess;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    using K = void (*)(SkParams);
    static const K kernels[3] = {conv_sk_kernel<PT, CT, NW, NST, 0>, conv_sk_kernel<PT, CT, NW, NST, 1>, conv_sk_kernel<PT, CT, NW, NST, 2>};
    auto attr_of = [](K k) { return hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, NW * kRegionMax); };
    static const hipError_t attr[3] = {attr_of(kernels[0]), attr_of(kernels[1]), attr_of(kernels[2])};
    const int mode = a.C % kRow ? 0 : (a.R == 1 && a.S == 1 && a.stride == 1 && a.pad == 0) ? 2 : 1;
    if (attr[mode] != hipSuccess) return attr[mode];
    kernels[mode]<<<(unsigned)grid, NW * 64, (size_t)NW * prm.region, st>>>(prm);
    return hipGetLastError();
}

}  // namespace

namespace {

// The shapes that were measured best: 16 x 16 tiles while they are at most two per compute unit, else 32 x 32 with a ring of
// one stage (several workgroups share a compute unit and cover each other's latency), eight wavefronts while there is at most
// one such tile per compute unit and a chain long enough to split, four otherwise.  (Larger tiles lost everywhere: 64 x 64
// took 6 us where these take 3 to 4, and more where there are many.)
enum class Shape { none, t16, t32x8, t32x4 };

Shape t32_shape(long long t32, int n) { return t32 <= kNumCU && n > 4 ? Shape::t32x8 : Shape::t32x4; }

Shape choose(const ConvArgs &a)
{
    if (!conv_sk_supports(a)) return Shape::none;
    const long long M = (long long)a.N * a.P * a.Q;
    const long long t16 = ((M + 15) / 16) * ((a.K + 15) / 16), t32 = ((M + 31) / 32) * ((a.K + 31) / 32);
    if (t16 <= 512) return Shape::t16;
    const int n = (a.R * a.S * a.C + kRow - 1) / kRow;
    // Fitted to 1300 layer sizes: this kernel takes 3 us + (2 + 0.4 n) ns per 32 x 32 tile; the general one, while its tiles do not
    // fill the chip, 3 us + 0.28 us per 128 bytes of the reduction in steps of that length, 0.7 us in steps of 64, 0.8 where K, a
    // multiple of 16, leaves its last channel tile partly empty (3x3 448 -> 224 at 31 x 27, 15 images 23.1, here 38.3), and up to 22 us
    // more where a ragged K takes its general epilogue (5x5 448 -> 832 at 45 x 77, one image, a format per channel: 72.7, here 94.7; 3x3
    // 528 -> 248 at 43 x 7, 16 images 37.7, here 26.4).  Of 506 layers whose K is no whole tile but a multiple of 16 the choice is 1.005
    // of the better in the mean, 10 of them more than 8 % off (priced as a ragged K 1.015 and 27); of 117 ragged ones 1.003 and 1; with
    // sums, where every K takes the general epilogue, 1.011 and 14 of 373.  Its 64 x 64 tiles for at most 1024 pixels, six stages
    // in flight, do as well as the long steps (96 -> 576, 980 pixels 4.1, here 4.9; 320 -> 320 4.3, 4.8), and so does any of its
    // tiles where the reduction is a single step (64 -> 64 at 56 x 56, one image 3.9, 4.4).  At the line: 3x3 256 -> 256 at 14 x 14, four images 8.4 -> 5.8 us, twelve
    // (592 tiles) 8.45 against 8.0; 1x1 512 -> 256 at 28 x 28, one image 4.4 -> 4.3, four 4.7 against 6.2; 3x3 64 -> 64 at
    // 56 x 56, four images 7.6 -> 6.7, twelve 8.7 against 14.4.
    long long price = 280LL * n;
    if (!conv_mfma_wide(a)) {
        // the input-resident kernel has no chain and is faster at once where C is no multiple of 128 (64 -> 448 at 35 x 35, two
        // images: 4.0 against 6.8)
        if (conv_pw_supports(a) && a.C % kRow) return Shape::none;
        if (!(conv_mfma_lean(a) && a.K % 64 == 0 && (M <= 1024 || n == 1)))
            price = a.K % (a.K <= 64 ? 64 : 128) == 0 ? 700LL * n
                    : conv_mfma_lean(a) && !a.frac_w && a.K % 16 == 0 ? 800LL * n
                                                                     : 700LL * n + 700LL * (n < 32 ? n : 32);
    }
    if (t32 * (20 + 4 * n) > price * 10) return Shape::none;
    return t32_shape(t32, n);
}

}  // namespace

bool conv_sk_supports(const ConvArgs &a)
{
    if (!conv_mfma_supports(a)) return false;
    if (a.add && (((uintptr_t)a.add & 3) || (a.ldadd & 3) || (a.K & 3))) return false;           // operand read in words
    return true;
}

bool conv_sk_pays(const ConvArgs &a) { return choose(a) != Shape::none; }

hipError_t launch_conv_sk(const ConvArgs &a, hipStream_t st)
{
    Shape s = choose(a);
    if (s == Shape::none)                          // asked for by name where another kernel is faster
        s = t32_shape(((long long)a.N * a.P * a.Q + 31) / 32 * ((a.K + 31) / 32), (a.R * a.S * a.C + kRow - 1) / kRow);
    switch (s) {
        case Shape::t16: return launch_cfg<1, 1, 8, 2>(a, st);
        case Shape::t32x8: return launch_cfg<2, 2, 8, 1>(a, st);
        default: return launch_cfg<2, 2, 4, 1>(a, st);
    }
}

}  // namespace dfq
