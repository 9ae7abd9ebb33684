// Grouped convolutions with any number of channels in a group and any alignment on the gfx950 int8 matrix cores, several groups at a time.
//
// A block is 32 output channels (or fewer) that are whole groups, with all the input channels of those groups: Kg = 12 gives blocks of two
// groups, 24 outputs and 2 * Cg inputs; more than 32 outputs in a group give several blocks with the same inputs.  Inside a block the
// layer is an ungrouped convolution whose weights are zero outside the group's own columns, and the zeros cost matrix work that this chip
// has to spare.  A workgroup of four wavefronts walks tiles of 128 or 256 output pixels of one block:
//   weights: once per workgroup, 16-byte pieces (tap, piece of the block's channels) cut out at any byte address, masked to the group's
//            columns, in the order the matrix instruction reads them;
//   input:   per tile the image rows it reads, only the block's channels of each pixel, cut out at any byte address and left at an odd number
//            of 16-byte pieces per pixel (one bank conflict in two reads would follow from an even one), padding as zeros;
//   sum:     two pieces per matrix instruction, a lane half each, at offsets that a table in LDS holds for every piece (kernel rows and
//            taps that skip are then no different from others).
// conv_rag_kernel, one group at a time, fetches and shifts every piece of the input once per tap and group and fills 32 rows of the matrix
// instruction with a group's few outputs.  203 x 16 x 29, 32 groups of 5 -> 5, 5x5: 335 us there, here 33; 19 x 45 x 69, 8 groups of 6 -> 6, 5x5 51,
// 12; depthwise with a channel count that is no multiple of four, 8 x 44 x 70 x 382, 3x3, formats per channel 103 (conv_direct.hip), 27.  Code
// size counts for small layers: divisions with a branch for 1 and both shifts of a piece in all their copies were 24 KB and 2 us on a layer of one tile (5.3 us).
// Bound by the tiles' chain of load, LDS, barrier, products and store: 1.4 us of a unit for each.
#include "conv_epilogue.hpp"
#include "dfq_host.hpp"
#include "input_piece.hpp"

namespace dfq {

namespace {

constexpr int kGroupsThreads = 256;
constexpr int kGroupsLds = 160 * 1024;
constexpr int kGroupsUnits = 256;

// exact n / d for 0 <= n < 2^31 without a branch (the code of this kernel is fetched anew for every small layer): n itself is kept for d = 1
struct GroupsDiv {
    uint32_t mul, keep;
    int s, d;
};

GroupsDiv groups_div(int d)
{
    const FastDiv f = make_fastdiv(d);
    return {f.mul, d == 1 ? ~0u : 0u, d == 1 ? 0 : f.s - 1, d};
}

__device__ __forceinline__ int operator/(int n, const GroupsDiv &f) { return (int)((__umulhi((uint32_t)n, f.mul) + ((uint32_t)n & f.keep)) >> f.s); }

struct GroupsParams {
    ConvArgs a;
    int M;                       // N*P*Q
    int Cg, Kg;
    int per_block;               // groups of a block
    int blocks, tiles_k;         // blocks; blocks of one group (1: whole groups)
    int np, pitch;               // pieces of a block's channels; LDS bytes of a pixel
    int wp;                      // LDS pixels of an image row
    int npieces, chunks;         // taps * np; matrix instructions per 32 x 32 tile
    int vs, slots;               // LDS rows an output row advances by; LDS rows of an image
    int tiles_p;
    int row_bytes, x_last, w_row, w_last;
    int w_at, tab_at;            // LDS bytes of the weights and of the table
    GroupsDiv div_pq, div_q, div_slots, div_r, div_row, div_np, div_blocks, div_tk, div_kg, div_s;
};

struct __attribute__((packed, aligned(1))) GroupsPiece {
    unsigned long long lo, hi;
};

typedef unsigned __int128 u128;

// How a tile goes out: one shift within [0, 23]; a shift within it for every channel; sums, or any shift.
enum { kOutLean, kOutChannel, kOutAny };

// PT: 32-pixel tiles of a wavefront
template <int PT, int OUT>
__global__ void __launch_bounds__(kGroupsThreads, 4) conv_rag_kernel_groups(GroupsParams prm)
{
    constexpr int BM = 128 * PT;
    constexpr int kRuns = 4;                         // pieces of the input in flight per lane
    extern __shared__ uint4 lds[];
    const ConvArgs &a = prm.a;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int G = gridDim.x;
    int lb = blockIdx.x;
    {   // ids are dealt round-robin to the 8 XCDs: neighbours, which read the same pixels, on one XCD
        const int per = G / 8, rem = G % 8, xcd = lb % 8, idx = lb / 8;
        lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
    }
    const int pt0 = lb / prm.div_blocks, block = lb - pt0 * prm.blocks, pt_step = G / prm.blocks;
    int g0, k0, kcount;
    if (prm.tiles_k == 1) {
        g0 = block * prm.per_block;
        k0 = g0 * prm.Kg;
        kcount = min(prm.per_block, a.groups - g0) * prm.Kg;
    } else {
        g0 = block / prm.div_tk;
        const int t = block - g0 * prm.tiles_k;
        k0 = g0 * prm.Kg + 32 * t;
        kcount = min(32, prm.Kg - 32 * t);
    }
    const int c0 = g0 * prm.Cg;
    char *const base = (char *)lds;

    // ---- weights: LDS row i = 8g + 4h + e of a piece receives channel 16h + 4g + e, so that a lane ends up with 16 consecutive channels
    auto weights = [&](int i0) __attribute__((always_inline)) {
        constexpr int kAtOnce = 2;
        unsigned long long v[kAtOnce][2];
        int d[kAtOnce], lo[kAtOnce];
#pragma unroll
        for (int e = 0; e < kAtOnce; e++) {
            const int i = i0 + e * kGroupsThreads;
            const int row = i & 31, piece = i >> 5, ch = 16 * ((row >> 2) & 1) + 4 * (row >> 3) + (row & 3);
            const int tap = piece / prm.div_np, o = 16 * (piece - tap * prm.np);
            lo[e] = (prm.tiles_k == 1 ? ch / prm.div_kg * prm.Cg : 0) - o;                   // the group's first column inside the piece
            const bool any = piece < prm.npieces && ch < kcount && lo[e] < 16 && lo[e] + prm.Cg > 0;
            const int b = (k0 + ch) * prm.w_row + tap * prm.Cg - min(lo[e], 0), from = any ? min(b, prm.w_last) : 0;
            if (!any) lo[e] = -(1 << 30);
            d[e] = any ? b - from : 0;
            const GroupsPiece t = *(const GroupsPiece *)(a.w + (unsigned)from);
            v[e][0] = t.lo;
            v[e][1] = t.hi;
        }
#pragma unroll
        for (int e = 0; e < kAtOnce; e++) {
            const int i = i0 + e * kGroupsThreads, hi = lo[e] + prm.Cg;
            if (__builtin_amdgcn_ballot_w64(d[e] != 0)) {                // the end of the weights
                const u128 t = (((u128)v[e][1] << 64) | v[e][0]) >> (8 * d[e]);
                v[e][0] = (unsigned long long)t;
                v[e][1] = (unsigned long long)(t >> 64);
            }
            if (__builtin_amdgcn_ballot_w64(lo[e] > 0)) {
                const u128 t = (((u128)v[e][1] << 64) | v[e][0]) << (8 * max(lo[e], 0));
                v[e][0] = (unsigned long long)t;
                v[e][1] = (unsigned long long)(t >> 64);
            }
#pragma unroll
            for (int h = 0; h < 2; h++) {                                // the columns behind the group's: half of the shift twice, 8 bytes make a zero
                const int keep = 4 * min(max(hi - 8 * h, 0), 8);
                v[e][h] &= ~((~0ull << keep) << keep);
            }
            if (i < prm.chunks * 64) {
                unsigned long long *to = (unsigned long long *)(base + prm.w_at + 16 * i);
                to[0] = v[e][0];
                to[1] = v[e][1];
            }
        }
    };
    for (int i = tid; i < prm.chunks * 2; i += kGroupsThreads) {
        const int tap = i / prm.div_np, r = tap / prm.div_s, s = tap - r * a.S;
        *(int *)(base + prm.tab_at + 4 * i) = i < prm.npieces ? (r * prm.wp + s) * prm.pitch + 16 * (i - tap * prm.np) : 0;
    }
    int bv[16];
    const int kc = k0 + 16 * lh, count = min(16, kcount - 16 * lh);
#pragma unroll
    for (int i = 0; i < 16; i++) bv[i] = a.b ? a.b[kc + min(i, count - 1)] : 0;        // (a channel past the last is never stored)
    int sv[OUT == kOutChannel ? 16 : 1];
    if constexpr (OUT == kOutChannel) {
#pragma unroll
        for (int i = 0; i < 16; i++) sv[i] = a.shift + a.frac_w[kc + min(i, count - 1)];
    }
    Requant rq;
    rq.init(a.shift, a.relu);

    auto slot_of = [&](int m, int &q) {
        const int n = m / prm.div_pq, pq = m - n * prm.div_pq.d;
        const int p = pq / prm.div_q;
        q = pq - p * a.Q;
        return n * prm.slots + p * prm.vs;
    };
    const int *const tab = (const int *)(base + prm.tab_at) + lh;
    const v4i *const wl = (const v4i *)(base + prm.w_at) + 32 * lh + l32;
    const int pieces_row = prm.div_row.d;

    // ---- the rows of a tile: kRuns pieces per lane on their way
    int u0, total, q;
    u128 xv[kRuns];
    int xd[kRuns], xto[kRuns];
    auto rows_of = [&](int pt) __attribute__((always_inline)) {
        const int m0 = pt * BM, m_last = min(m0 + BM, prm.M) - 1;
        u0 = __builtin_amdgcn_readfirstlane(slot_of(m0, q));
        total = __builtin_amdgcn_readfirstlane((slot_of(m_last, q) + a.R - u0) * pieces_row);
    };
    auto fetch = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < kRuns; e++) {
            const int i = i0 + e * kGroupsThreads;
            const int u = i / prm.div_row, left = i - u * pieces_row;
            const int c = left / prm.div_np, j = left - c * prm.np;
            const int us = u0 + u, n = us / prm.div_slots, s = us - n * prm.slots;
            const int p = a.stride >= a.R ? s / prm.div_r : s;             // kernels that skip rows have no slots for them
            const int ih = (a.stride >= a.R ? p * a.stride + s - p * a.R : s) - a.pad, iw = c - a.pad;
            const bool in = i < total && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            const unsigned b = in ? (unsigned)(n * a.H + ih) * (unsigned)prm.row_bytes + (unsigned)(iw * a.C + c0 + 16 * j) : 0u;
            const unsigned from = min(b, (unsigned)prm.x_last);
            xd[e] = piece_move(in, b, from);
            xto[e] = i < total ? (u * prm.wp + c) * prm.pitch + 16 * j : -1;
            const GroupsPiece t = *(const GroupsPiece *)(a.x + from);
            xv[e] = ((u128)t.hi << 64) | t.lo;
        }
    };
    auto deposit = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < kRuns; e++) {
            if (__builtin_amdgcn_ballot_w64(xd[e] > 0)) xv[e] >>= 8 * max(xd[e], 0);         // the end of the input
            if (xd[e] < 0) xv[e] = 0;
            if (xto[e] >= 0) *(u128 *)(base + xto[e]) = xv[e];
        }
    };
    rows_of(pt0);
    fetch(tid);
    for (int i0 = tid; i0 < prm.chunks * 64; i0 += 2 * kGroupsThreads) weights(i0);

    for (int pt = pt0; pt < prm.tiles_p; pt += pt_step) {
        const int m0 = pt * BM, m_last = min(m0 + BM, prm.M) - 1, u_first = u0;
        deposit();
        for (int i0 = tid + kRuns * kGroupsThreads; i0 < total; i0 += kRuns * kGroupsThreads) {
            fetch(i0);
            deposit();
        }
        int m[PT];
        const char *xp[PT];
#pragma unroll
        for (int p = 0; p < PT; p++) {
            m[p] = m0 + 32 * (wave * PT + p) + l32;
            const int row = slot_of(min(m[p], m_last), q) - u_first;
            xp[p] = base + (row * prm.wp + q * a.stride) * prm.pitch;
        }
        v16i acc[PT];
#pragma unroll
        for (int p = 0; p < PT; p++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[p][i] = bv[i];
        __syncthreads();
        if (pt + pt_step < prm.tiles_p) {            // the first pieces of the next tile, under the products of this one
            rows_of(pt + pt_step);
            fetch(tid);
        }
#pragma unroll 4
        for (int i = 0; i < prm.chunks; i++) {
            const int off = tab[2 * i];
            const v4i wf = wl[64 * i];
#pragma unroll
            for (int p = 0; p < PT; p++) acc[p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf, *(const v4i *)(xp[p] + off), acc[p], 0, 0, 0);
        }
        if (pt + pt_step < prm.tiles_p) __syncthreads();        // this tile's rows have been read
        settle_accumulators<PT>(&acc[0]);
        if (count > 0) {
#pragma unroll
            for (int p = 0; p < PT; p++) {
                if (m[p] >= prm.M) continue;
                int8_t *dst = a.y + (size_t)m[p] * a.ldy + kc;
                if constexpr (OUT == kOutLean) {
                    const uint4 r = requant_tile_lane_fast(acc[p], rq);
                    store_bytes(Bytes16{{r.x, r.y, r.z, r.w}}, dst, count);
                } else if constexpr (OUT == kOutChannel) {
                    Bytes16 r;
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        int4 s, hi, badd;
#pragma unroll
                        for (int i = 4 * j; i < 4 * j + 4; i++) asm volatile("" : "+v"(sv[i]));      // what follows is cheaper than registers for it
                        s = make_int4(sv[4 * j], sv[4 * j + 1], sv[4 * j + 2], sv[4 * j + 3]);
                        hi = make_int4(127 << s.x, 127 << s.y, 127 << s.z, 127 << s.w);
                        badd = make_int4(max((1 << s.x) >> 1, 1) - 1, max((1 << s.y) >> 1, 1) - 1, max((1 << s.z) >> 1, 1) - 1, max((1 << s.w) >> 1, 1) - 1);
                        r.w[j] = requant_four_per_channel(acc[p][4 * j], acc[p][4 * j + 1], acc[p][4 * j + 2], acc[p][4 * j + 3], s, hi, badd, a.relu);
                    }
                    store_bytes(r, dst, count);
                } else {
                    store_tile_lane_ragged(acc[p], a, m[p], kc, count);
                }
            }
        }
    }
}

// LDS bytes of the rows that `bm` output pixels read, at worst, at `pitch` bytes per pixel
long long groups_rows(const ConvArgs &a, int bm, int pitch)
{
    const int vs = a.stride < a.R ? a.stride : a.R;
    const long long out_rows = (bm - 2) / a.Q + 2, images = (out_rows - 2) / a.P + 1;
    const long long rows = (out_rows - 1) * vs + a.R + images * (a.R - vs);
    return rows * ((long long)(a.Q - 1) * a.stride + a.S) * pitch;
}

bool out_any(const ConvArgs &a)
{
    return a.acc_out || !a.y || a.shift + (a.frac_w ? a.frac_w_lo : 0) < 0 || a.shift + (a.frac_w ? a.frac_w_hi : 0) > 23;
}

struct GroupsForm {
    int pt, per_block, np, pitch;
    long long rows, lds;
};

GroupsForm groups_form(const ConvArgs &a, int pt, int per_block)
{
    GroupsForm f;
    f.pt = pt;
    f.per_block = per_block;
    f.np = (per_block * (a.C / a.groups) + 15) / 16;
    f.pitch = 16 * (f.np | 1);
    f.rows = groups_rows(a, 128 * pt, f.pitch);
    const long long chunks = ((long long)a.R * a.S * f.np + 1) / 2;
    f.lds = f.rows + chunks * (1024 + 8);
    return f;
}

// The form for a call, or pt = 0: 256 pixels to a workgroup, the weights read once for two products, while that fills the chip and leaves four
// workgroups to a unit (19 x 45 x 69, 8 groups of 6 -> 6, 5x5 14.1 us with 128, 12.0; 2 x 77 x 76, 16 groups of 8 -> 7, 3x3 / 2 7.2, 8.4); fewer
// groups to a block where the rows would take more than half of the LDS.
GroupsForm groups_choose(const ConvArgs &a)
{
    const int Kg = a.K / a.groups;
    int per = Kg <= 32 ? 32 / Kg : 1;
    if (per > a.groups) per = a.groups;
    const long long blocks = Kg <= 32 ? (a.groups + per - 1) / per : (long long)a.groups * ((Kg + 31) / 32);
    GroupsForm f = groups_form(a, 2, per);
    if (out_any(a) || (long long)a.N * a.P * a.Q / 256 * blocks < 512 || f.lds > 40 * 1024) f = groups_form(a, 1, per);
    while (f.lds > 80 * 1024 && f.per_block > 1) f = groups_form(a, f.pt, (f.per_block + 1) / 2);
    if (f.lds > kGroupsLds - 512) f.pt = 0;
    return f;
}

template <int PT, int OUT>
hipError_t launch_out(const GroupsParams &prm, long long grid, long long lds, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute((const void *)conv_rag_kernel_groups<PT, OUT>, hipFuncAttributeMaxDynamicSharedMemorySize, kGroupsLds);
    if (attr != hipSuccess) return attr;
    conv_rag_kernel_groups<PT, OUT><<<(unsigned)grid, kGroupsThreads, (size_t)lds, st>>>(prm);
    return hipGetLastError();
}

template <int PT>
hipError_t launch_form(GroupsParams &prm, const GroupsForm &f, hipStream_t st)
{
    const ConvArgs &a = prm.a;
    prm.tiles_p = (int)((prm.M + 128LL * PT - 1) / (128 * PT));
    int occ = (int)(kGroupsLds / (f.lds + 512));
    if (occ > 4) occ = 4;
    long long grid = (long long)prm.tiles_p * prm.blocks;
    const long long most = (long long)occ * kGroupsUnits;
    if (grid > most) grid = most / prm.blocks * prm.blocks;
    if (grid < prm.blocks) grid = prm.blocks;
    if (out_any(a)) return launch_out<1, kOutAny>(prm, grid, f.lds, st);
    return a.frac_w ? launch_out<PT, kOutChannel>(prm, grid, f.lds, st) : launch_out<PT, kOutLean>(prm, grid, f.lds, st);
}

}  // namespace

// Nanoseconds of three kernels on grouped layers, each fitted to what 2700 to 4100 layers of a random mix took (2 to 640 groups of 1 .. 64 -> 1 .. 64
// channels, 1x1 to 5x5, strides to 3, images from 1 x 3 to 90 x 90; plain, formats per channel, sums, shifts beyond the packed rounding), to 7 to 10 % in
// the mean.  This kernel: matrix instructions of a tile, and for every tile of a unit the pieces a lane brings in, the instructions, 1.1 us and
// what its end takes; alone on a unit a tile hides less.  A layer it does not take costs more than any.
double conv_rag_groups_time(const ConvArgs &a)
{
    if (a.groups < 2 || !conv_rag_supports(a)) return 1e30;
    const GroupsForm f = groups_choose(a);
    if (!f.pt) return 1e30;
    const int Kg = a.K / a.groups, outputs = Kg <= 32 ? f.per_block * Kg : 32;
    const double blocks = Kg <= 32 ? (a.groups + f.per_block - 1) / f.per_block : (double)a.groups * ((Kg + 31) / 32);
    const double tiles = (double)(((long long)a.N * a.P * a.Q + 128 * f.pt - 1) / (128 * f.pt)) * blocks;
    const double load = tiles > kGroupsUnits ? tiles / kGroupsUnits : 1.0;
    const double pieces = (double)f.rows / f.pitch * f.np / kGroupsThreads, products = (double)((a.R * a.S * f.np + 1) / 2) * f.pt;
    double tile = 159.0 * pieces + (2 * (f.lds + 512) > kGroupsLds ? 42.0 : 22.0) * products + 1082.0, once = 4454.0 + 86.0 * products;
    // sums go out a dword at a time unless a group's channels start and end on four (6 x 67 x 83 x 638, 1x1 / 2: 50.1 us, one output per lane 27.4)
    if (a.acc_out) {
        const bool words = a.K % 4 == 0 && (Kg <= 32 ? outputs : Kg) % 4 == 0;
        tile += (words ? 1170.0 : 3770.0) * outputs / 32;
    } else if (out_any(a)) {
        tile += 326.0;
        once += 1915.0;
    } else if (a.frac_w) {
        tile += 437.0 * f.pt;
    }
    return once + load * tile;
}

namespace {

// conv_rag_kernel, one group at a time
double one_group_time(const ConvArgs &a)
{
    const long long Cg = a.C / a.groups, Kg = a.K / a.groups, M = (long long)a.N * a.P * a.Q;
    const double steps = (double)(((long long)a.R * a.S * ((Cg + 15) / 16) + 3) / 4);
    const long long wide = (M + 127) / 128 * a.groups * ((Kg + 63) / 64);
    const bool narrow = Kg <= 32, large = !narrow && wide >= 512;                          // 128 x 32, 128 x 64 or 64 x 64 tiles
    const double tiles = narrow ? (double)((M + 127) / 128 * a.groups) : large ? (double)wide : (double)((M + 63) / 64 * a.groups * ((Kg + 63) / 64));
    const double load = tiles > kGroupsUnits ? tiles / kGroupsUnits : 1.0;
    double tile = narrow ? 351.0 * steps + 804.0 : large ? 332.0 * steps + 1253.0 : 310.0 * steps + 294.0;
    double once = 4261.0 + (narrow ? 298.0 : large ? 222.0 : 236.0) * steps;
    if (a.acc_out || a.frac_w || out_any(a)) {
        const double part = (Kg < 16 ? Kg : 16) / 16.0;
        tile += part * (a.acc_out ? (large ? 5027.0 : 883.0) : out_any(a) ? 488.0 : 899.0);
        once += 1176.0 * part;
    }
    return once + load * tile;
}

// conv_direct_kernel, one output per lane; taps outside the image cost nothing
double one_output_time(const ConvArgs &a)
{
    const double Cg = a.C / a.groups, outputs = (double)a.N * a.P * a.Q * a.K;
    const double taps = (double)(a.R < a.H ? a.R : a.H) * (a.S < a.W ? a.S : a.W);
    return 3821.0 + taps * (92.7 + 76.8 * Cg) + outputs * (4.12e-3 + taps * (3.55e-5 + 5.76e-4 * Cg));
}

}  // namespace

bool conv_rag_groups_faster(const ConvArgs &a) { return a.groups > 1 && conv_rag_groups_time(a) < 0.9 * one_group_time(a); }

// A tenth is for the fit.  203 x 16 x 29, 32 groups of 5 -> 5, 5x5 335 us (one group at a time), here 33; 207 x 59 x 14, 4 groups of 4 -> 16, 5x5 59.3
// (conv_grouped.hip), 18.4; 84 x 37 x 15, 32 groups of 2 -> 3, 3x3 / 2 20.1 (conv_direct.hip), 8.5.  On the other side 51 x 25 x 11, 8 groups of
// 12 -> 4, 3x3 6.3 (conv_grouped.hip), here 9.3; 217 x 53 x 16, 4 groups of 64 -> 64, 3x3 / 3 16.4 (one group at a time), 38.4.  (Depthwise layers
// that conv_depthwise.hip takes - 3x3, C a multiple of four, words aligned - are not asked about: that kernel's time is not fitted.)
bool conv_rag_groups_pays(const ConvArgs &a)
{
    if (a.groups < 2) return false;
    const bool few = a.C / a.groups <= 2 && a.K > a.C;
    double other;
    if (conv_grouped_supports(a)) {
        if (conv_sg_supports(a)) return false;
        other = conv_grouped_time(a);
    } else {
        // one or two inputs to several outputs: conv_direct_time() is the fit that holds there (251 such layers took 1.00 of it in the mean,
        // 1x1 to 5x5, but 0.83 of one_output_time(), which sent 8 x 28 x 28, 32 groups of 2 -> 3, 3x3 here; 11.9 us measured, 12.0 and 15.0 by the two).
        // Half of it is a cautious line: it keeps that layer at 11.9 us where this kernel takes 6.1; of 329 others behind it 117 would be a tenth faster.
        other = conv_rag_pays(a) ? one_group_time(a) : few ? conv_direct_time(a) : one_output_time(a);
    }
    return conv_rag_groups_time(a) < (few ? 0.5 : 0.9) * other;
}

// (the caller has cut the batch to 31-bit offsets and pixel numbers, and the weights and a row hold a whole piece)
hipError_t launch_conv_rag_groups(const ConvArgs &a, hipStream_t st)
{
    const GroupsForm f = groups_choose(a);
    GroupsParams prm{};
    prm.a = a;
    prm.M = a.N * a.P * a.Q;
    prm.Cg = a.C / a.groups;
    prm.Kg = a.K / a.groups;
    prm.per_block = f.per_block;
    prm.tiles_k = (prm.Kg + 31) / 32;
    prm.blocks = prm.tiles_k == 1 ? (a.groups + f.per_block - 1) / f.per_block : a.groups * prm.tiles_k;
    prm.np = f.np;
    prm.pitch = f.pitch;
    prm.wp = (a.Q - 1) * a.stride + a.S;
    prm.npieces = a.R * a.S * f.np;
    prm.chunks = (prm.npieces + 1) / 2;
    prm.vs = a.stride < a.R ? a.stride : a.R;
    prm.slots = (a.P - 1) * prm.vs + a.R;
    prm.row_bytes = a.W * a.C;
    prm.x_last = (int)((long long)a.N * a.H * a.W * a.C - 16);
    prm.w_row = a.R * a.S * prm.Cg;
    prm.w_last = a.K * prm.w_row - 16;
    prm.w_at = (int)f.rows;
    prm.tab_at = prm.w_at + prm.chunks * 1024;
    prm.div_pq = groups_div(a.P * a.Q);
    prm.div_q = groups_div(a.Q);
    prm.div_slots = groups_div(prm.slots);
    prm.div_r = groups_div(a.R);
    prm.div_row = groups_div(prm.wp * prm.np);
    prm.div_np = groups_div(prm.np);
    prm.div_blocks = groups_div(prm.blocks);
    prm.div_tk = groups_div(prm.tiles_k);
    prm.div_kg = groups_div(prm.Kg);
    prm.div_s = groups_div(a.S);
    return f.pt == 2 ? launch_form<2>(prm, f, st) : launch_form<1>(prm, f, st);
}

}  // namespace dfq
