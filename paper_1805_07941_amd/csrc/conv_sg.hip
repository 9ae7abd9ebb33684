// Grouped quantized convolution (1 < groups, C/groups = K/groups in {4, 8, 16, 32, 64}) on the int8 matrix cores.
//
// A group's reduction (Eq. 6 over R * S * C/groups terms) is far shorter than a 64-byte step of the matrix
// instructions, but 64 consecutive channels hold whole groups, and the sum over a group equals the sum over those 64
// channels with the weights of the other groups' channels set to zero: the layer is C/64 independent dense 64 -> 64
// convolutions with block-diagonal weights.  The zeros cost matrix work (16x for groups of 4), which this chip has to
// spare: measured 3-4x faster than one output per lane with dot products on the vector ALU.
//
// Four wavefronts own 64 pixels x 32 channels each: 64 pixels x 128 channels of the layer where C is a multiple of 128 (a step is a whole
// cache line of every input row: 52 bytes a clock into LDS and not 29), else 128 pixels x 64 channels.  32 output channels are whole
// groups of up to 32, so of the wavefront's input only the same 32 channels count: one k-step of 32 bytes per kernel tap (NK = 1; groups
// of 64 take two).  Its weights - for every tap 32 rows x 32 bytes, zeros included - stay in registers (4 per tap and lane, the zeros
// never loaded) while the workgroup walks tiles of its channel block; the input streams through a ring of LDS stages filled by
// direct global -> LDS loads, one step per tap, on into the next tile under the epilogue (rows XOR-swizzled as in the dense
// kernels).  Epilogue in registers: bias as start value, ReLU, rounding shift, clamp (the lean form only; the launcher falls back
// otherwise).
// Bound by the feed of LDS: 64 x 28 x 28, 256 channels in 32 groups, 3x3 (115 MB through L1).  One tile of 64-channel blocks per
// workgroup, both halves multiplied, weights gathered for 128 pixels: 18.0 us; here 15.1.
#include "conv_ring.hpp"

namespace dfq {

namespace {

struct SgParams {
    ConvArgs a;
    int M;                  // N * P * Q output pixels
    int Cg;                 // channels per group
    int blocks_c;           // C / BLK
    int tiles;              // pixel tiles x channel blocks
    unsigned x_bytes;
    FastDiv div_q, div_p, div_bc;
};

template <int NTAPS, int NSTAGES, int BLK, int NK, int OCC>
__global__ void __launch_bounds__(256, OCC) conv_sg_kernel(SgParams prm)
{
    static_assert(NTAPS % NSTAGES == 0, "a tap's stage is the same in every tile");
    constexpr int BP = BLK == 128 ? 64 : 128;
    constexpr int PIECES = BLK / 16, RPC = 64 / PIECES;    // 16-byte pieces of a row; rows a wavefront-wide load fills
    constexpr int XJ = BP / (4 * RPC);                     // loads per wavefront and step
    constexpr int PT = 2;                                  // 32-pixel tiles per wavefront (64 pixels x 32 channels)
    extern __shared__ uint4 lds[];                         // [NSTAGES * BP input rows]
    const ConvArgs &a = prm.a;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // tiles of this workgroup: lb, lb + G, ...  Ids are dealt round-robin to the 8 XCDs; renumbered so that each XCD owns a contiguous
    // range (the channel blocks of one pixel tile and neighbouring pixel tiles read the same input lines).  G is a multiple of the number of
    // channel blocks, so the block never changes.
    const int G = gridDim.x;
    int lb = blockIdx.x;
    {
        const int per = G / 8, rem = G % 8, xcd = lb % 8, idx = lb / 8;
        lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
    }
    const int cb = lb - fastdiv(lb, prm.div_bc) * prm.blocks_c;
    const int ntiles = (prm.tiles - lb + G - 1) / G;       // lb < G <= tiles

    const v4i x_rsrc = make_rsrc(a.x, prm.x_bytes);
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char *)(char *)&lds[0];

    // ---- input producer: lane l of a wavefront-wide load supplies row l/PIECES of a chunk, physical piece l%PIECES, which holds logical
    // piece (l%4) ^ ((row>>2)&3) of 4, or (l%8) ^ ((row>>1)&7) of 8 (bit 3 of the row being that of the chunk's number, the wavefront's)
    const int lrow = lane / PIECES;
    const int lp = BLK == 64 ? (lane & 3) ^ ((lane >> 4) & 3) : (lane & 7) ^ ((lane >> 4) | ((wave & 1) << 2));
    int ih0[XJ], iw0[XJ], xbase[XJ];
    int p_r = 0, p_s = 0, p_tile = lb;                     // kernel row, column and tile of the step fetched next
    auto begin_tile = [&]() __attribute__((always_inline)) {
        const int m0 = fastdiv(p_tile, prm.div_bc) * BP;
#pragma unroll
        for (int j = 0; j < XJ; j++) {
            const int m = m0 + RPC * (wave + 4 * j) + lrow;
            const int mi = min(m, prm.M - 1);
            const int t = fastdiv(mi, prm.div_q);
            const int oq = mi - t * a.Q;
            const int n = fastdiv(t, prm.div_p);
            const int op = t - n * a.P;
            ih0[j] = m < prm.M ? op * a.stride - a.pad : -(1 << 28);      // past the last pixel: no kernel row is inside the image
            iw0[j] = oq * a.stride - a.pad;
            xbase[j] = ((n * a.H + op * a.stride - a.pad) * a.W + iw0[j]) * a.C + cb * BLK + lp * 16;
        }
        p_r = p_s = 0;
    };
    auto issue = [&](int stage) __attribute__((always_inline)) {
        const int tap_off = (p_r * a.W + p_s) * a.C;
        const unsigned sbase = lds_base + (unsigned)(stage * BP * BLK) + (unsigned)wave * 1024u;
#pragma unroll
        for (int j = 0; j < XJ; j++) {
            const bool ok = (unsigned)(ih0[j] + p_r) < (unsigned)a.H && (unsigned)(iw0[j] + p_s) < (unsigned)a.W;
            const unsigned off = ok ? (unsigned)(xbase[j] + tap_off) : kOutOfRange;
            load_piece_to_lds(off, x_rsrc, (unsigned)__builtin_amdgcn_readfirstlane((int)(sbase + (unsigned)(j * 4096))));
        }
        if (++p_s == a.S) {
            p_s = 0;
            ++p_r;
        }
    };
    begin_tile();
#pragma unroll
    for (int i = 0; i < NSTAGES; i++) issue(i);

    // ---- consumer
    const int wp0 = BLK == 128 ? 0 : (wave & 1) * 64, wc0 = BLK == 128 ? wave * 32 : (wave >> 1) * 32;
    const int l32 = lane & 31, lh = lane >> 5;
    const int swz = BLK == 64 ? (l32 >> 2) & 3 : (l32 >> 1) & 7;
    const int kc = cb * BLK + wc0 + 16 * lh;               // the lane's 16 output channels
    const int in0 = NK == 1 ? wc0 : wc0 & ~63;             // first input channel that counts, within the block
    int bias[16];
#pragma unroll
    for (int r4 = 0; r4 < 4; r4++) {
        const int4 bv = a.b ? *(const int4 *)(a.b + kc + 4 * r4) : make_int4(0, 0, 0, 0);
        bias[4 * r4 + 0] = bv.x;
        bias[4 * r4 + 1] = bv.y;
        bias[4 * r4 + 2] = bv.z;
        bias[4 * r4 + 3] = bv.w;
    }
    // ---- weights: the matrix instruction's first operand for tap t and k-step kk is, in lane (l32, lh), bytes 32 kk + 16 lh .. + 15 of row
    // l32 of the wavefront's slab.  Row i = 8g + 4h + e holds channel 16h + 4g + e (so that the instruction leaves 16 consecutive channels
    // in each lane); of its bytes only the channels of that output channel's own group are weights, the rest zeros.
    v4i wreg[NTAPS][NK];
    {
        const int kl = wc0 + 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);        // channel within the block
        const int c_lo = (kl / prm.Cg) * prm.Cg - in0;                                 // first channel of its group, from in0 on
        const uint32_t *wk = (const uint32_t *)(a.w + (size_t)(cb * BLK + kl) * NTAPS * prm.Cg);
#pragma unroll
        for (int t = 0; t < NTAPS; t++)
#pragma unroll
            for (int kk = 0; kk < NK; kk++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int c = 32 * kk + 16 * lh + 4 * e - c_lo;                    // channel within the group, if inside
                    wreg[t][kk][e] = (c >= 0 && c < prm.Cg) ? (int)wk[(t * prm.Cg + c) >> 2] : 0;
                }
    }
    v4i f[NK][PT];
    auto read_step = [&](int kk, int stage) __attribute__((always_inline)) {
        const char *base = (const char *)lds + stage * BP * BLK;
        const int g = (in0 / 16 + kk * 2 + lh) ^ swz;
#pragma unroll
        for (int p = 0; p < PT; p++) f[kk][p] = *(const v4i *)(base + (wp0 + p * 32 + l32) * BLK + g * 16);
    };
    auto ring_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    Requant rq;
    rq.init(a.shift, a.relu);
    // step 0 has landed when at most the loads of the steps issued after it are outstanding
    wait_ahead<XJ>(NSTAGES - 1);
    ring_barrier();
#pragma unroll
    for (int kk = 0; kk < NK; kk++) read_step(kk, 0);
    int c_tile = lb;
    for (int i = 0; i < ntiles; i++) {
        const bool last = i + 1 == ntiles;
        v16i acc[PT];
#pragma unroll
        for (int p = 0; p < PT; p++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[p][r] = bias[r];
#pragma unroll
        for (int it = 0; it < NTAPS; it++) {
            const int stage = it % NSTAGES, next = (it + 1) % NSTAGES;
#pragma unroll
            for (int kk = 0; kk < NK; kk++)
#pragma unroll
                for (int p = 0; p < PT; p++) acc[p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wreg[it][kk], f[kk][p], acc[p], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NSTAGES > 1) {
                if (it + 1 < NTAPS || !last) {
                    // the next step has landed when only younger ones are on their way (a tile's stores may be among them: a longer wait)
                    if (last) wait_ahead<XJ>(max(min(NSTAGES - 2, NTAPS - it - 2), 0));
                    else wait_loads<(NSTAGES - 2) * XJ>();
                    ring_barrier();                        // every wavefront has read this step: its stage may be refilled
                    if (it + NSTAGES == NTAPS && !last) {
                        p_tile += G;
                        begin_tile();
                    }
                    if (it + NSTAGES < NTAPS || !last) issue(stage);
#pragma unroll
                    for (int kk = 0; kk < NK; kk++) read_step(kk, next);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- epilogue: register r of a lane belongs to channel kc + r of pixel m
        settle_accumulators<PT>(&acc[0]);
        const int m0 = fastdiv(c_tile, prm.div_bc) * BP;
#pragma unroll
        for (int p = 0; p < PT; p++) {
            const int m = m0 + wp0 + p * 32 + l32;
            const uint4 out = requant_tile_lane_fast(acc[p], rq);
            if (m < prm.M) *(uint4 *)(a.y + (size_t)m * a.ldy + kc) = out;
        }
        c_tile += G;
    }
}

template <int NTAPS, int NSTAGES, int BLK, int NK>
hipError_t launch_blk(SgParams &prm, hipStream_t st)
{
    constexpr int BP = BLK == 128 ? 64 : 128, OCC = NK == 1 ? 4 : 3;
    constexpr size_t lds_bytes = (size_t)NSTAGES * BP * BLK;
    static_assert(lds_bytes * OCC <= (size_t)kLdsBytes, "the workgroups of a compute unit share its LDS");
    prm.blocks_c = prm.a.C / BLK;
    prm.div_bc = make_fastdiv(prm.blocks_c);
    const long long tiles = ((prm.M + (long long)BP - 1) / BP) * prm.blocks_c;
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    prm.tiles = (int)tiles;
    // one tap: its weights are no reason to stay, and one stage has nothing on its way into the next tile (116 x 17 x 82, 64 channels in 4 groups
    // 9.8 us persistent, 7.7 a tile to a workgroup)
    long long grid = NTAPS == 1 ? tiles : OCC * kNumCU / prm.blocks_c * prm.blocks_c;
    if (grid < prm.blocks_c) grid = prm.blocks_c;
    if (grid > tiles) grid = tiles;                        // a multiple of the blocks, too
    conv_sg_kernel<NTAPS, NSTAGES, BLK, NK, OCC><<<(unsigned)grid, 256, lds_bytes, st>>>(prm);
    return hipGetLastError();
}

template <int NTAPS, int NSTAGES>
hipError_t launch_sg(SgParams &prm, hipStream_t st)
{
    const bool wide = prm.a.C % 128 == 0;
    if (prm.Cg == 64) {        // at most 64 KB of weights (conv_grouped_supports): six taps in 128 channels, four in 192
        if constexpr (NTAPS <= 6) {
            if (wide) return launch_blk<NTAPS, NSTAGES, 128, 2>(prm, st);
        }
        if constexpr (NTAPS <= 4) {
            if (!wide) return launch_blk<NTAPS, NSTAGES, 64, 2>(prm, st);
        }
        return hipErrorInvalidValue;
    }
    return wide ? launch_blk<NTAPS, NSTAGES, 128, 1>(prm, st) : launch_blk<NTAPS, NSTAGES, 64, 1>(prm, st);
}

}  // namespace

bool conv_sg_supports(const ConvArgs &a)
{
    if (a.groups < 2 || a.C % 64 || a.K != a.C) return false;
    const int Cg = a.C / a.groups;
    if (Cg != 4 && Cg != 8 && Cg != 16 && Cg != 32 && Cg != 64) return false;
    const int taps = a.R * a.S;
    if ((taps != 1 && taps != 4 && taps != 6 && taps != 9) || a.stride < 1) return false;      // the tap counts the kernel is built for
    if (a.frac_w || a.add || a.acc_out || !a.y) return false;
    if (a.shift < 0 || a.shift > 23) return false;                                  // the lean epilogue
    if ((a.ldy & 15) || ((uintptr_t)a.y & 15) || ((uintptr_t)a.x & 15) || ((uintptr_t)a.w & 3) || (a.b && ((uintptr_t)a.b & 15))) return false;
    if ((long long)a.N * a.H * a.W * a.C >= (1LL << 31) - (1 << 24)) return false;   // 31-bit byte offsets into the input
    if ((long long)a.N * a.P * a.Q >= (1LL << 31) - 512) return false;
    if ((long long)a.N * a.P * a.Q * a.ldy >= (1LL << 40)) return false;
    return (((long long)a.N * a.P * a.Q + 63) / 64) * (a.C / 64) <= 0x7fffffffLL;
}

hipError_t launch_conv_sg(const ConvArgs &a, hipStream_t st)
{
    SgParams prm;
    prm.a = a;
    const long long M = (long long)a.N * a.P * a.Q;
    prm.M = (int)M;
    prm.Cg = a.C / a.groups;
    prm.x_bytes = (unsigned)((long long)a.N * a.H * a.W * a.C);
    prm.div_q = make_fastdiv(a.Q);
    prm.div_p = make_fastdiv(a.P);
    switch (a.R * a.S) {
        case 1: return launch_sg<1, 1>(prm, st);
        case 4: return launch_sg<4, 4>(prm, st);
        case 6: return launch_sg<6, 3>(prm, st);
        default: return launch_sg<9, 3>(prm, st);
    }
}

}  // namespace dfq
