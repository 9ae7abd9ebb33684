// Convolutions with any number of channels, any grouping and any alignment on the gfx950 int8 matrix cores: the layers the
// other matrix-core kernels decline because a tap's channels are no whole 16-byte pieces (pruned networks, 83 -> 131
// channels), because a pointer or a group starts at an odd byte, or because the kernel is larger than their masks.
//
// The reduction axis is cut into SEGMENTS whose bytes are contiguous in both operands, each padded to whole 16-byte pieces:
//   groups == 1: a kernel row - the S * C bytes of the S neighbouring pixels an output reads from one image row stand one
//                behind the other in NHWC, and so do those of w[k][r][.][.]; 83 channels x 3 taps are 249 bytes, 16 pieces
//                (2.7 % padding), where tap by tap they would be 18;
//   groups > 1 : one tap of the group, C/groups bytes.
// A weight piece is zero behind the end of its segment, so whatever the input piece holds there does not count; an input
// piece only has to be zero where it leaves the image row (padding), and both are made so in registers: a lane fetches its 16
// bytes at any byte address with one load that stays inside the row (inside the weights), shifts them into place if the row
// ended, and writes them to LDS.  This is vector work the direct-to-LDS kernels do not have (about 200 instructions
// per step and wavefront against four matrix instructions), and it bounds the kernel; it buys the whole shape range.
//
// A workgroup of four wavefronts owns BM pixels x BK channels of one group and walks the pieces four (64 bytes) at a time
// through two LDS stages: while one is multiplied, the loads of the step behind the next are in flight in registers.
// 24 KB of LDS let five or six workgroups share a compute unit, which is what hides the load latency.
// Measured on 16 x 57 x 43 x 83 -> 131, 3x3 (7.7 GOP): 9.2 ms with one output per lane (conv_direct.hip) -> 22.6 us, 340 TOP/s, the vector
// ALUs busy 60 % of the time and the matrix pipes 12 %; 20 x 28 x 28 x 250 -> 250, 1x1: 2.49 ms -> 10.5 us; 19 x 14 x 13 in 32 groups of
// 13 -> 3, 3x3: 63 -> 11 us.
#include "conv_epilogue.hpp"
#include "rag_images.hpp"

namespace dfq {

namespace {

constexpr int kRagThreads = 256;
constexpr int kLdsMost = 160 * 1024;
constexpr int kNumUnits = 256;

struct RagParams {
    ConvArgs a;
    int M;                 // N*P*Q
    int Cg, Kg;
    int segs_row;          // segments per kernel row: 1 (groups == 1) or S
    int seglen;            // bytes of a segment: S*C or Cg
    int seg_end;           // pieces of a segment times 16
    int nsteps;            // ceil(R * segs_row * pieces / 4)
    int tiles_k;           // channel tiles per group
    int row_bytes;         // W*C
    int w_row;             // R*S*Cg: bytes of a weight row
    int w_bytes;           // bytes of the whole weight tensor
    FastDiv div_kt, div_tk, div_pq, div_q;
};

struct __attribute__((packed, aligned(1))) Piece16 {
    unsigned long long lo, hi;
};

typedef unsigned __int128 u128;

// 16 bytes at base + off (a scalar base and a 32-bit offset: one address register)
__device__ __forceinline__ u128 load16(const int8_t *base, unsigned off)
{
    const Piece16 v = *(const Piece16 *)(base + off);
    return ((u128)v.hi << 64) | v.lo;
}

// v moved by d bytes: out[i] = v[i + d], zeros from outside (|d| < 16; d of 16 and more, either sign, gives zeros)
__device__ __forceinline__ u128 shift_bytes(u128 v, int d)
{
    if (d >= 16 || d <= -16) return 0;
    return d >= 0 ? v >> (8 * d) : v << (-8 * d);
}

// The end of a tile for formats per channel that all lie within the four-instruction rounding: no branch in a channel, and the formats
// fetched anew for each of a lane's pixels (48 registers otherwise).
__device__ __forceinline__ void store_lane_formats(const v16i &v, const ConvArgs &a, int m, int kc, int count)
{
    const int *f = a.frac_w + kc;
    Bytes16 o;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        asm volatile("" : "+v"(f));
        int4 s = make_int4(f[min(4 * j, count - 1)], f[min(4 * j + 1, count - 1)], f[min(4 * j + 2, count - 1)], f[min(4 * j + 3, count - 1)]);
        s = make_int4(s.x + a.shift, s.y + a.shift, s.z + a.shift, s.w + a.shift);
        const int4 hi = make_int4(127 << s.x, 127 << s.y, 127 << s.z, 127 << s.w);
        const int4 badd = make_int4(max((1 << s.x) >> 1, 1) - 1, max((1 << s.y) >> 1, 1) - 1, max((1 << s.z) >> 1, 1) - 1, max((1 << s.w) >> 1, 1) - 1);
        o.w[j] = requant_four_per_channel(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3], s, hi, badd, a.relu);
    }
    store_bytes(o, a.y + (size_t)m * a.ldy + kc, count);
}

__device__ __forceinline__ bool formats_are_fast(const ConvArgs &a)
{
    return a.frac_w && !a.acc_out && a.y && a.shift + a.frac_w_lo >= 0 && a.shift + a.frac_w_hi <= 23;
}

// CONTIG: groups == 1, a segment is a whole kernel row
template <int BM, int BK, bool CONTIG>
__global__ void __launch_bounds__(kRagThreads) conv_rag_kernel(RagParams prm)
{
    constexpr int XS = BM * 4 / kRagThreads;                  // input pieces per lane and step
    constexpr int WS = (BK * 4 + kRagThreads - 1) / kRagThreads;
    constexpr bool kPartialW = BK * 4 < kRagThreads;
    constexpr int WAVES_P = BM / 32 < 4 ? BM / 32 : 4, WAVES_C = 4 / WAVES_P;
    constexpr int PT = BM / WAVES_P / 32, CT = BK / WAVES_C / 32;
    static_assert(PT >= 1 && CT >= 1 && XS >= 1, "tile shape");
    constexpr int STAGE = (BM + BK) * 4;                      // 16-byte pieces of a stage
    __shared__ uint4 lds[2 * STAGE];
    const ConvArgs &a = prm.a;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;

    // tile numbers run over the channel tiles of all groups first: the tiles that read the same pixels are neighbours, and the
    // renumbering keeps neighbours on one XCD
    const int G = gridDim.x;
    int lb = blockIdx.x;
    {
        const int per = G / 8, rem = G % 8, xcd = lb % 8, idx = lb / 8;
        lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
    }
    const int pt = fastdiv(lb, prm.div_kt);
    const int kt = lb - pt * prm.div_kt.d;
    const int g = fastdiv(kt, prm.div_tk);
    const int m0 = pt * BM, kg0 = (kt - g * prm.tiles_k) * BK;    // kg0: first channel inside the group
    const int k_base = g * prm.Kg, goff = g * prm.Cg;

    // ---- this lane's rows of a stage: row tid/4 (+ 64 per further piece), piece tid%4
    const int lrow = tid >> 2, lp = tid & 3;
    int xrow[XS];                     // byte of the image row that kernel row 0 of the lane's pixel reads (may lie outside the image)
    int ih0[XS], iwb[XS];             // that row; first byte the pixel's window reads inside a row, the group's offset included
    int iw0[XS];
#pragma unroll
    for (int j = 0; j < XS; j++) {
        const int m = m0 + 64 * j + lrow;
        const bool live = m < prm.M;
        const int mi = live ? m : 0;
        const int n = fastdiv(mi, prm.div_pq);
        const int pq = mi - n * (a.P * a.Q);
        const int p = fastdiv(pq, prm.div_q), q = pq - p * a.Q;
        ih0[j] = live ? p * a.stride - a.pad : -(1 << 30);        // a pixel past the last one: every row lies outside
        iw0[j] = q * a.stride - a.pad;
        iwb[j] = iw0[j] * a.C + goff;
        xrow[j] = live ? (n * a.H + ih0[j]) * prm.row_bytes : 0;
    }
    int woff[WS];                     // first byte of the lane's weight row
#pragma unroll
    for (int j = 0; j < WS; j++) {
        // LDS row i = 8g + 4h + e of a 32-row group receives channel 16h + 4g + e: the matrix instruction then leaves 16
        // consecutive channels in each lane
        const int rr = 64 * j + lrow, i32 = rr & 31;
        const int k = kg0 + (rr & ~31) + 16 * ((i32 >> 2) & 1) + 4 * (i32 >> 3) + (i32 & 3);
        woff[j] = (k_base + min(k, prm.Kg - 1)) * prm.w_row;
    }

    // position on the reduction axis: kernel row r, segment s of the row, byte o of the segment
    int r = 0, s = 0, o = 16 * lp;
    int wseg = 0, rline = 0;          // the segment's first byte inside a weight row; r * row_bytes
    auto next_segment = [&]() {
        o -= prm.seg_end;
        wseg += prm.seglen;
        if (CONTIG || ++s == prm.segs_row) { s = 0; r++; rline += prm.row_bytes; }
    };
    auto settle = [&]() {
        if (CONTIG && prm.seg_end >= 64) {
            if (o >= prm.seg_end) next_segment();
        } else {
            while (o >= prm.seg_end) next_segment();
        }
    };
    settle();

    u128 xv[XS], wv[WS];
    int xd[XS], wd[WS];
    int wvalid = 16;                  // bytes of the weight piece inside its segment
    const int wlast = prm.w_bytes - 16, xlast = prm.row_bytes - 16;
    // A piece that is not wanted at all is fetched from the tensor's start and shifted out: the loads need no branch.
    auto fetch = [&]() __attribute__((always_inline)) {
        const bool in_k = r < a.R;
        const int sc = CONTIG ? 0 : s * a.C;
#pragma unroll
        for (int j = 0; j < XS; j++) {
            bool ok = in_k && (unsigned)(ih0[j] + r) < (unsigned)a.H;
            if (!CONTIG) ok = ok && (unsigned)(iw0[j] + s) < (unsigned)a.W;
            const int b = iwb[j] + sc + o;                            // first wanted byte of the image row
            const int at = max(0, min(b, xlast));                     // the load stays inside the row
            xd[j] = ok ? b - at : 16;
            xv[j] = load16(a.x, ok ? (unsigned)(xrow[j] + rline + at) : 0u);
        }
        wvalid = prm.seglen - o;
#pragma unroll
        for (int j = 0; j < WS; j++) {
            // behind the last piece the input is zero, and a channel past the group's last is never stored: any bytes will do there
            const int b = min(woff[j] + wseg + o, prm.w_bytes), at = min(b, wlast);
            wd[j] = b - at;
            wv[j] = load16(a.w, (unsigned)at);
        }
        o += 64;
        settle();
    };
    // Uniform branches: most wavefronts have no lane at an image border, at a segment's end or at the end of the weights.
    auto any = [](bool c) { return __builtin_amdgcn_ballot_w64(c) != 0; };
    auto deposit = [&](int stage) __attribute__((always_inline)) {
        uint4 *xs = lds + stage * STAGE, *ws = xs + BM * 4;
        const int swz = (lrow >> 2) & 3;                              // 16 consecutive rows spread one logical piece over all banks
#pragma unroll
        for (int j = 0; j < XS; j++) {
            u128 v = xv[j];
            if (any(xd[j] != 0)) v = shift_bytes(v, xd[j]);
            *(u128 *)(xs + (64 * j + lrow) * 4 + (lp ^ swz)) = v;
        }
        if (!kPartialW || lrow < BK) {
#pragma unroll
            for (int j = 0; j < WS; j++) {
                u128 v = wv[j];
                if (any(wd[j] != 0)) v = shift_bytes(v, wd[j]);
                if (any(wvalid < 16)) {
                    const unsigned long long part = (1ull << (8 * (wvalid & 7))) - 1ull;
                    const unsigned long long lo = (unsigned long long)v, hi = (unsigned long long)(v >> 64);
                    if (wvalid < 16) v = wvalid < 8 ? (u128)(lo & part) : ((u128)(hi & part) << 64) | lo;
                }
                *(u128 *)(ws + (64 * j + lrow) * 4 + (lp ^ swz)) = v;
            }
        }
    };

    v16i acc[CT][PT];
#pragma unroll
    for (int c = 0; c < CT; c++)
#pragma unroll
        for (int p = 0; p < PT; p++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[c][p][i] = 0;

    const int wp0 = (wave % WAVES_P) * (BM / WAVES_P), wc0 = (wave / WAVES_P) * (BK / WAVES_C);
    const int swz = (l32 >> 2) & 3;
    fetch();
    deposit(0);
    if (prm.nsteps > 1) fetch();
    __syncthreads();
    for (int i = 0; i < prm.nsteps; i++) {
        const v4i *xs = (const v4i *)lds + (i & 1) * STAGE, *ws = xs + BM * 4;
#pragma unroll
        for (int kk = 0; kk < 2; kk++) {
            const int piece = (kk * 2 + lh) ^ swz;
            v4i wf[CT], xf[PT];
#pragma unroll
            for (int c = 0; c < CT; c++) wf[c] = ws[(wc0 + c * 32 + l32) * 4 + piece];
#pragma unroll
            for (int p = 0; p < PT; p++) xf[p] = xs[(wp0 + p * 32 + l32) * 4 + piece];
#pragma unroll
            for (int c = 0; c < CT; c++)
#pragma unroll
                for (int p = 0; p < PT; p++) acc[c][p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[c], xf[p], acc[c][p], 0, 0, 0);
        }
        if (i + 1 < prm.nsteps) {
            deposit((i + 1) & 1);                 // the stage read one step ago; its readers have met at the barrier below
            if (i + 2 < prm.nsteps) fetch();
            __syncthreads();
        }
    }
    settle_accumulators<CT * PT>(&acc[0][0]);

    Requant rq;
    rq.init(a.shift, a.relu);
    const bool lean = rq.fast && !a.frac_w && !a.acc_out;         // one shift for the launch, int8 result only
    const bool formats = formats_are_fast(a);
#pragma unroll
    for (int c = 0; c < CT; c++) {
        const int kl = kg0 + wc0 + c * 32 + 16 * lh;        // first of the lane's 16 channels, inside the group
        if (kl >= prm.Kg) continue;
        const int kc = k_base + kl, count = min(16, prm.Kg - kl);
        int bv[16];
#pragma unroll
        for (int i = 0; i < 16; i++) bv[i] = (a.b && i < count) ? a.b[kc + i] : 0;
#pragma unroll
        for (int p = 0; p < PT; p++) {
            const int m = m0 + wp0 + p * 32 + l32;
            if (m >= prm.M) continue;
#pragma unroll
            for (int i = 0; i < 16; i++) acc[c][p][i] += bv[i];
            if (lean) {
                const uint4 o = requant_tile_lane_fast(acc[c][p], rq);
                store_bytes(Bytes16{{o.x, o.y, o.z, o.w}}, a.y + (size_t)m * a.ldy + kc, count);
            } else if (formats) {
                store_lane_formats(acc[c][p], a, m, kc, count);
            } else {
                store_tile_lane_ragged(acc[c][p], a, m, kc, count);
            }
        }
    }
}

constexpr int kRowsBM = 128;

// ---- the input's rows in LDS -------------------------------------------------------------------------------------------
// groups == 1 and rows that fit: the image rows a tile of BM output pixels reads are brought to LDS once, padding columns and rows
// outside the image as zeros, each row at a 16-byte boundary - whatever the channel count and the base's alignment.  Every kernel
// row and every channel of the tile then reads its operands from there: an output pixel's window in a row is S*C contiguous
// bytes that start anywhere, so a lane takes five aligned words and cuts its 16 bytes out with four byte alignments by an amount that
// never changes (rows and pieces lie at multiples of 16).  What conv_rag_kernel does per 16 bytes, tap and channel tile - address,
// border test, shift, LDS write - happens here once per 16 bytes of the input.  The weights take conv_rag_kernel's route through two LDS
// stages.  The reduction runs in chunks of 32 bytes of a kernel row; behind the end of a row's S*C bytes the weights are zero.
// A workgroup owns 128 pixels, a wavefront 32 of them and all 32 * CT channels of the tile.
// Bound by the LDS: a lane's 16 bytes are five words wherever they start (34 LDS cycles per chunk and wavefront against 64 of the matrix
// pipe).  16 x 57 x 43 x 83 -> 131, 3x3 (rotating inputs): conv_rag_kernel 24.9 us, here 20.0 (without stores 16.9, without the input's
// rows 16.6, launch and addresses alone 4.2); 292 x 48 x 250 -> 9, 5x5 67.9, 38.0; 1950 pixels of 114 -> 292, 5x5 31.5, 21.1.
// Tried: 96 .. 160 channels per tile (fewer workgroups: 20.7 .. 22 us), tiles of 64 pixels (28 us: nearly the same rows), a ring of
// weights one step ahead (the same time).
struct RowsParams {
    ConvArgs a;
    int M;
    int seglen, seg_end;         // bytes of a window's row: S*C, and rounded up to whole chunks of 32
    int nsteps;                  // steps of two chunks
    int tiles_k;
    int row_bytes, w_row, w_bytes;
    int pitch;                   // LDS bytes of an image row
    int vs, slots;               // LDS rows an output row advances by; LDS rows of an image
    int stage_at;                // LDS byte of the weight stages
    FastDiv div_tk, div_pq, div_q, div_pieces, div_slots, div_r;
};

template <int CT>
__global__ void __launch_bounds__(kRagThreads) conv_rag_kernel_rows(RowsParams prm)
{
    constexpr int BM = kRowsBM, BK = 32 * CT;
    constexpr bool kPartialW = BK * 4 < kRagThreads;
    static_assert(BK * 4 <= kRagThreads, "one weight piece per lane and step");
    constexpr int kAhead = 4, kRuns = 6;             // steps of weights in flight; runs of the input in flight
    extern __shared__ uint4 lds[];
    const ConvArgs &a = prm.a;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int G = gridDim.x;
    int lb = blockIdx.x;
    {
        const int per = G / 8, rem = G % 8, xcd = lb % 8, idx = lb / 8;
        lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
    }
    const int pt = fastdiv(lb, prm.div_tk);
    const int k0 = (lb - pt * prm.tiles_k) * BK, m0 = pt * BM;

    // LDS row of output row p of image n: n * slots + p * vs (+ kernel row); the tile's first one is row 0
    auto slot_of = [&](int m, int &q) {
        const int n = fastdiv(m, prm.div_pq), pq = m - n * prm.div_pq.d;
        const int p = fastdiv(pq, prm.div_q);
        q = pq - p * a.Q;
        return n * prm.slots + p * prm.vs;
    };
    int q_first, q_last, q_mine;
    const int m_last = min(m0 + BM, prm.M) - 1;
    const int u0 = __builtin_amdgcn_readfirstlane(slot_of(m0, q_first)), nrows = __builtin_amdgcn_readfirstlane(slot_of(m_last, q_last) + a.R - u0);
    const int m = m0 + 32 * wave + l32;
    const unsigned at = (unsigned)((slot_of(min(m, m_last), q_mine) - u0) * prm.pitch + q_mine * a.stride * a.C + 16 * lh);
    const unsigned cut = at & 3u;
    const char *xbase = (const char *)lds + (at & ~3u);

    // ---- weights: lane's row tid/4 of a stage, piece tid%4.  Positions are scalars of the two chunks of a step: byte inside a weight
    // row, and how many bytes of the window's row are left there.
    const int lrow = tid >> 2, lp = tid & 3;
    // (row order as in conv_rag_kernel: 16 consecutive channels end in each lane)
    const int i32 = lrow & 31, k_mine = k0 + (lrow & ~31) + 16 * ((i32 >> 2) & 1) + 4 * (i32 >> 3) + (i32 & 3);
    const int woff = min(k_mine, a.K - 1) * prm.w_row + 16 * (lp & 1);
    int f_o = 0, f_seg = 0;                     // the next chunk: byte of the window's row; the row's first byte inside a weight row
    u128 wv[kAhead];                            // steps on their way
    int wd[kAhead], left0[kAhead], left1[kAhead];
    const int wlast = prm.w_bytes - 16;
    auto next_chunk = [&](int &byte, int &left) __attribute__((always_inline)) {
        byte = f_seg + f_o;
        left = f_seg < prm.w_row ? prm.seglen - f_o : 0;               // (past the last kernel row: nothing)
        f_o += 32;
        if (f_o == prm.seg_end) {
            f_o = 0;
            f_seg += prm.seglen;
        }
    };
    auto fetch = [&](int f) __attribute__((always_inline)) {
        int b0, b1;
        next_chunk(b0, left0[f]);
        next_chunk(b1, left1[f]);
        const int b = woff + (lp < 2 ? b0 : b1), from = min(b, wlast);
        wd[f] = b - from;
        wv[f] = load16(a.w, (unsigned)from);
    };
    auto any = [](bool c) { return __builtin_amdgcn_ballot_w64(c) != 0; };
    auto deposit = [&](int f, int stage) __attribute__((always_inline)) {
        if (kPartialW && lrow >= BK) return;
        uint4 *ws = lds + prm.stage_at / 16 + stage * (BK * 4);
        u128 v = wv[f];
        if (any(wd[f] != 0)) v = shift_bytes(v, wd[f]);
        if (min(left0[f], left1[f]) < 32) {
            const int valid = (lp < 2 ? left0[f] : left1[f]) - 16 * (lp & 1);
            const unsigned long long part = (1ull << (8 * (valid & 7))) - 1ull;
            const unsigned long long lo = (unsigned long long)v, hi = (unsigned long long)(v >> 64);
            if (valid <= 0) v = 0;
            else if (valid < 16) v = valid < 8 ? (u128)(lo & part) : ((u128)(hi & part) << 64) | lo;
        }
        *(u128 *)(ws + lrow * 4 + (lp ^ ((lrow >> 2) & 3))) = v;
    };
#pragma unroll
    for (int f = 0; f < kAhead; f++)
        if (f < prm.nsteps) fetch(f);

    // ---- the tile's image rows, 64 pieces of a row per wavefront and load: everything about the row is scalar
    {
        const int per_row = prm.div_pieces.d, runs = (per_row + 63) / 64, total = nrows * runs, pad_bytes = a.pad * a.C, xlast = prm.row_bytes - 16;
        int u = 0, run = wave;                  // wavefront v takes runs v, v + 4, ... of all rows together
        while (run >= runs) { run -= runs; u++; }
        for (int i0 = wave; i0 < total; i0 += 4 * kRuns) {
            u128 v[kRuns];
            int d[kRuns], to[kRuns];
#pragma unroll
            for (int e = 0; e < kRuns; e++) {
                const int us = u0 + u, n = fastdiv(us, prm.div_slots), s = us - n * prm.slots;
                const int p = a.stride >= a.R ? fastdiv(s, prm.div_r) : s;         // kernels that skip rows have no slots for them
                const int ih = (a.stride >= a.R ? p * a.stride + s - p * a.R : s) - a.pad;
                const bool row_in = i0 + 4 * e < total && (unsigned)ih < (unsigned)a.H;
                const unsigned row = row_in ? (unsigned)(n * a.H + ih) * (unsigned)prm.row_bytes : 0u;
                const int piece = run * 64 + lane, b = piece * 16 - pad_bytes, from = max(0, min(b, xlast));
                to[e] = i0 + 4 * e < total && piece < per_row ? u * prm.pitch + piece * 16 : -1;
                d[e] = row_in ? b - from : 16;
                v[e] = load16(a.x, row + (unsigned)from);
                run += 4;
                while (run >= runs) { run -= runs; u++; }
            }
#pragma unroll
            for (int e = 0; e < kRuns; e++) {
                if (any(d[e] != 0)) v[e] = shift_bytes(v[e], d[e]);
                if (to[e] >= 0) *(u128 *)((char *)lds + to[e]) = v[e];
            }
        }
    }
    deposit(0, 0);
    if (kAhead < prm.nsteps) fetch(0);

    v16i acc[CT];
#pragma unroll
    for (int c = 0; c < CT; c++)
#pragma unroll
        for (int i = 0; i < 16; i++) acc[c][i] = 0;
    const int swz = (l32 >> 2) & 3;
    int xo = 0, xr = 0;                          // byte of the window's row, the kernel row's LDS bytes
    const int xr_last = (a.R - 1) * prm.pitch;
    // (a barrier that waits for LDS alone: the weights on their way stay there)
    auto ring_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto step = [&](int i, int f) __attribute__((always_inline)) {           // f: where the next step's weights are
        const v4i *ws = (const v4i *)(lds + prm.stage_at / 16 + (f + 1 & 1) * (BK * 4));
#pragma unroll
        for (int kk = 0; kk < 2; kk++) {
            const uint32_t *src = (const uint32_t *)(xbase + xr + xo);
            uint32_t w5[5];
#pragma unroll
            for (int e = 0; e < 5; e++) w5[e] = src[e];
            v4i wf[CT], xf;
#pragma unroll
            for (int c = 0; c < CT; c++) wf[c] = ws[(c * 32 + l32) * 4 + ((kk * 2 + lh) ^ swz)];
#pragma unroll
            for (int e = 0; e < 4; e++) xf[e] = (int)__builtin_amdgcn_alignbyte(w5[e + 1], w5[e], cut);
#pragma unroll
            for (int c = 0; c < CT; c++) acc[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[c], xf, acc[c], 0, 0, 0);
            xo += 32;
            if (xo == prm.seg_end) {
                xo = 0;
                xr = min(xr + prm.pitch, xr_last);       // (an odd last chunk meets zero weights)
            }
        }
        if (i + 1 < prm.nsteps) {
            deposit(f, f & 1);                // the stage read one step ago; its readers have met at the barrier below
            if (i + 1 + kAhead < prm.nsteps) fetch(f);
            ring_barrier();
        }
    };
    static_assert(kAhead % 2 == 0, "a step's stage is its number's parity");
    ring_barrier();
    for (int i = 0; i < prm.nsteps; i += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; u++)
            if (i + u < prm.nsteps) step(i + u, (u + 1) % kAhead);
    }
    settle_accumulators<CT>(&acc[0]);

    Requant rq;
    rq.init(a.shift, a.relu);
    const bool lean = rq.fast && !a.frac_w && !a.acc_out, formats = formats_are_fast(a);
    if (m >= prm.M) return;
#pragma unroll
    for (int c = 0; c < CT; c++) {
        const int kc = k0 + c * 32 + 16 * lh;
        if (kc >= a.K) continue;
        const int count = min(16, a.K - kc);
        int bv[16];
        load_bias16(a, kc, bv);
#pragma unroll
        for (int i = 0; i < 16; i++) acc[c][i] += bv[i];
        if (lean) {
            const uint4 r = requant_tile_lane_fast(acc[c], rq);
            store_bytes(Bytes16{{r.x, r.y, r.z, r.w}}, a.y + (size_t)m * a.ldy + kc, count);
        } else if (formats) {
            store_lane_formats(acc[c], a, m, kc, count);
        } else {
            store_tile_lane_ragged(acc[c], a, m, kc, count);
        }
    }
}

// A tile's rows at worst: how many, the LDS bytes of one, and of all with the words behind the last window.
struct TileRows {
    long long rows, pitch, bytes;
};

TileRows tile_rows(const ConvArgs &a)
{
    constexpr int bm = kRowsBM;
    const int vs = a.stride < a.R ? a.stride : a.R;
    const long long out_rows = (bm - 2) / a.Q + 2, images = (out_rows - 2) / a.P + 1;
    const long long rows = (out_rows - 1) * vs + a.R + images * (a.R - vs);
    const long long pitch = ((long long)((a.Q - 1) * a.stride + a.S) * a.C + 15) / 16 * 16;
    return {rows, pitch, rows * pitch + 64};
}

// Channel tiles (of 32) of conv_rag_kernel_rows for a call, or 0: conv_rag_kernel.  Fitted to 726 layers (3x3 to 7x7, 3 to 400 channels,
// strides 1 and 2; plain, formats per channel, sums), each under both: 216 lie behind the line, 18 % faster in the mean, eight of them more
// than 4 % slower, by 12 % at most.  Below ten steps, or 16 where rows and columns are skipped, staging the rows costs what it saves
// (39456 pixels of 51 -> 63, 1x1: 7.4 us, with rows 9.9; 3072 of 63 -> 62, 3x3 / 2: 9.2, 13.4); rows of more than 72 KB leave one
// workgroup per unit (123200 pixels of 182 -> 12, 3x3: 36.0, 53.6).  Tiles of 32 channels while they are at most two per unit (1950 pixels of
// 114 -> 292, 5x5: 21.1 us, of 64 channels 23.9), else 64 (7670 of 164 -> 169, 5x5: 53.7, 33.5).
int rows_tile(const ConvArgs &a)
{
    const long long steps = ((long long)a.R * ((a.S * a.C + 31) / 32) + 1) / 2;
    const long long tiles_p = ((long long)a.N * a.P * a.Q + kRowsBM - 1) / kRowsBM, tiles = tiles_p * ((a.K + 31) / 32);
    // (with one tile for a unit more rows cost nothing: 2 x 76 x 51 of 181 -> 48, 3x3 19.1 us, with rows 14.9; 48 x 21 x 29 of 316 -> 11, 5x5 79.8,
    // 48.6; but 12 x 35 x 9 of 118 -> 16, 3x3 / 2 15.6, 18.5)
    const long long most = tiles <= kNumUnits && (a.stride == 1 || a.R * a.S >= 25) ? 148 * 1024 : 72 * 1024;
    const TileRows t = tile_rows(a);
    if (a.groups != 1 || steps < (a.stride > 1 ? 16 : 10) || a.R * a.S < 9 || t.bytes > most) return 0;
    // The rows come in runs of 64 pieces, 24 runs at a time; six steps pay for one such round, and images of a few columns or pixels have many
    // (117 x 51 x 3 of 61 -> 64, 5x5 / 3, 17 rounds and 25 steps: 19.7 us, with rows 55.3; 54 x 49 x 8 of 71 -> 180, 5x5 / 2, 6 and 30: 22.8, 38.2; 585
    // layers: 0.86 of the time in the mean with this line and without, 8 instead of 59 more than 8 % slower)
    const long long rounds = (t.rows * ((t.pitch / 16 + 63) / 64) + 23) / 24;
    if (6 * rounds > steps) return 0;
    // (a lane has one pixel for every format it fetches, or for every sum's address: many tiles with formats per channel or sums lose,
    // 81648 pixels of 86 -> 97, 3x3, per channel 34.0 us, here 38.4; 85500 of 58 -> 25, 5x5 / 2, 30.0, 41.5)
    if ((a.frac_w || a.acc_out) && tiles_p > 400) return 0;
    return a.K <= 32 || tiles <= 2 * kNumUnits ? 1 : 2;
}

template <int CT>
hipError_t launch_rows(const ConvArgs &a, hipStream_t st)
{
    constexpr int BM = kRowsBM, BK = 32 * CT;
    RowsParams prm{};
    prm.a = a;
    prm.M = a.N * a.P * a.Q;
    prm.seglen = a.S * a.C;
    prm.seg_end = (prm.seglen + 31) / 32 * 32;
    prm.nsteps = (a.R * (prm.seg_end / 32) + 1) / 2;
    prm.tiles_k = (a.K + BK - 1) / BK;
    prm.row_bytes = a.W * a.C;
    prm.w_row = a.R * prm.seglen;
    prm.w_bytes = a.K * prm.w_row;
    prm.pitch = (((a.Q - 1) * a.stride + a.S) * a.C + 15) / 16 * 16;
    prm.vs = a.stride < a.R ? a.stride : a.R;
    prm.slots = (a.P - 1) * prm.vs + a.R;
    prm.stage_at = (int)tile_rows(a).bytes;
    prm.div_tk = make_fastdiv(prm.tiles_k);
    prm.div_pq = make_fastdiv(a.P * a.Q);
    prm.div_q = make_fastdiv(a.Q);
    prm.div_pieces = make_fastdiv(prm.pitch / 16);
    prm.div_slots = make_fastdiv(prm.slots);
    prm.div_r = make_fastdiv(a.R);
    const size_t lds_bytes = (size_t)prm.stage_at + 2 * BK * 64;
    const long long grid = (prm.M + (long long)BM - 1) / BM * prm.tiles_k;
    if (grid > 0x7fffffffLL || lds_bytes > kLdsMost) return hipErrorInvalidValue;
    static const hipError_t attr = hipFuncSetAttribute((const void *)conv_rag_kernel_rows<CT>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMost);
    if (attr != hipSuccess) return attr;
    conv_rag_kernel_rows<CT><<<(unsigned)grid, kRagThreads, lds_bytes, st>>>(prm);
    return hipGetLastError();
}

template <int BM, int BK>
hipError_t launch_rag(RagParams &prm, hipStream_t st)
{
    prm.tiles_k = (prm.Kg + BK - 1) / BK;
    const long long kt = (long long)prm.a.groups * prm.tiles_k;
    const long long grid = (prm.M + (long long)BM - 1) / BM * kt;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    prm.div_kt = make_fastdiv((int)kt);
    prm.div_tk = make_fastdiv(prm.tiles_k);
    if (prm.a.groups == 1) conv_rag_kernel<BM, BK, true><<<(unsigned)grid, kRagThreads, 0, st>>>(prm);
    else conv_rag_kernel<BM, BK, false><<<(unsigned)grid, kRagThreads, 0, st>>>(prm);
    return hipGetLastError();
}

}  // namespace

bool conv_rag_supports(const ConvArgs &a)
{
    if (a.add) return false;
    const long long w_bytes = (long long)a.K * a.R * a.S * (a.C / a.groups), image = (long long)a.H * a.W * a.C;
    if ((long long)a.W * a.C < 16 || w_bytes < 16) return false;          // a piece is fetched whole
    // 32-bit offsets: the weights, and an image with the padding's reach on all sides (a batch is cut into runs of images)
    if (w_bytes >= (1LL << 30)) return false;
    if ((a.H + 2LL * a.pad + a.R) * a.W * a.C >= (1LL << 31) || (a.W + 2LL * a.pad + a.S) * a.C >= (1LL << 30)) return false;
    if ((long long)a.P * a.Q >= (1LL << 31) - 256 || image >= (1LL << 31)) return false;
    return (((long long)a.P * a.Q + 63) / 64) * a.groups * ((a.K / a.groups + 31) / 32) < (1LL << 31);
}

double conv_direct_time(const ConvArgs &a)
{
    const double Cg = a.C / a.groups, taps = (double)a.R * a.S, outputs = (double)a.N * a.P * a.Q * a.K;
    return 2990.0 + taps * (100.0 + 70.0 * Cg) + outputs * 0.0035 + outputs * taps * Cg * (taps > 1 && (Cg > 2 || taps >= 16) ? 58e-5 : 44e-5);
}

double conv_rag_time(const ConvArgs &a)
{
    const long long Cg = a.C / a.groups, Kg = a.K / a.groups, taps = (long long)a.R * a.S;
    const double M = (double)a.N * a.P * a.Q;
    const long long pieces = a.groups == 1 ? a.R * ((a.S * Cg + 15) / 16) : taps * ((Cg + 15) / 16), steps = (pieces + 3) / 4;
    const int bm = Kg <= 32 ? 128 : 64;
    const double tiles = (double)((long long)(M + bm - 1) / bm) * a.groups * ((Kg + 31) / 32), tail = tiles > 1280 ? tiles - 1280 : 0;
    double here = 3630.0 + 725.0 * steps + tiles * (1.36 + 1.4 * steps) + 1.1 * tail * steps;
    // the general epilogue, by the outputs a lane has of a group, as fitted while it stored a byte or a sum at a time (870 pixels, 1x1, 8 groups of
    // 18 -> 16, formats per channel: 6.7 us, 4.7; accumulators of 24180 pixels in 12 groups of 3 -> 24 47.3, 34.9; of 45288 pixels in four groups of 31 -> 5
    // 9.9, 42.0).  It stores words now, and the line still lies well: of conv_rag and one output per lane 643 layers (183 of them ungrouped) take 1.007
    // of the better in the mean with sums and 1.014 with shifts past 23; plain ones 1.011.
    if (a.acc_out || a.frac_w || a.shift < 0 || a.shift > 23) {
        const double part = (Kg < 16 ? Kg : 16) / 16.0, shares = part * tiles * (Kg <= 32 ? 1.0 : 0.5);
        here += a.acc_out ? 900.0 * part + 5.8 * shares : 1200.0 + 1000.0 * part + 2.4 * shares;
    }
    return here;
}

// Against one output per lane (conv_direct.hip).  A tile has at least 32 output channels of one group and 16 bytes for every tap of
// one, so with few channels in a group most of its products are padding, while the other kernel's time grows with the products that
// are wanted.  Both times as fitted to 6000 layers (1 to 64 groups of 1 .. 64 -> 1 .. 256 channels, 1x1 to 5x5, 25 to 100000 pixels), in
// ns; the line lies where they meet, with a sixteenth for the fit.  One or two outputs in a group were not fitted and stay with
// the other kernel; so do fewer than four products per output with fewer than twelve outputs in a group, where both mostly load.
// Measured, this kernel against the other: 8 x 28 x 28 pixels, 3x3, 32 groups of 1 -> 3 16.7 us, 9.9; of 2 -> 3 18.0, 12.0; of
// 3 -> 3 18.7, 20.7; of 15 -> 16, 5x5, 32.7, 3470; 14 x 14 pixels, 3x3, 32 groups of 1 -> 8 6.6, 4.9; 28 x 28, 1x1, 8 images, one
// group of 2 -> 11 4.6, 3.6; of 83 -> 131, 16 x 57 x 43, 3x3 22.6 us against 9.2 ms.
bool conv_rag_pays(const ConvArgs &a)
{
    const long long Cg = a.C / a.groups, Kg = a.K / a.groups, taps = (long long)a.R * a.S;
    if ((a.groups > 1 && Kg < 3) || !conv_rag_supports(a)) return false;
    if (taps * Cg < 4 && Kg < 12) return false;
    return conv_direct_time(a) * 15.0 > conv_rag_time(a) * 16.0;
}

// Layers whose kernel rows are at most 32 bytes (conv_smallc.hip takes every one) with more than a first layer's channels: that kernel's tiles
// of 64 channels and its packed weights pay from many tiles on only.  Of 86 such layers 60 are faster here, 1.26 times in the mean (8 x 18 x 14
// of 9 -> 68, 3x3 7.9 us, here 5.1; 26 x 14 x 7 of 26 -> 117, 1x1 / 2 6.5, 4.5); above the line 164 x 33 x 25 of 6 -> 9, 5x5 10.2, 11.5.
bool conv_rag_small(const ConvArgs &a)
{
    if (a.groups != 1 || a.C < 5 || a.frac_w || (a.acc_out && a.K <= 32) || !conv_rag_supports(a)) return false;
    return conv_rag_time(a) < 9500.0;
}

static hipError_t launch_images(const ConvArgs &a, hipStream_t st)
{
    const int rows_ct = rows_tile(a);
    if (rows_ct) return rows_ct == 1 ? launch_rows<1>(a, st) : launch_rows<2>(a, st);
    if (conv_rag_groups_faster(a)) return launch_conv_rag_groups(a, st);
    RagParams prm{};
    prm.a = a;
    prm.M = a.N * a.P * a.Q;
    prm.Cg = a.C / a.groups;
    prm.Kg = a.K / a.groups;
    prm.segs_row = a.groups == 1 ? 1 : a.S;
    prm.seglen = a.groups == 1 ? a.S * a.C : prm.Cg;
    prm.seg_end = (prm.seglen + 15) / 16 * 16;
    prm.nsteps = (int)(((long long)a.R * prm.segs_row * (prm.seg_end / 16) + 3) / 4);
    prm.row_bytes = a.W * a.C;
    prm.w_row = a.R * a.S * prm.Cg;
    prm.w_bytes = a.K * prm.w_row;
    prm.div_pq = make_fastdiv(a.P * a.Q);
    prm.div_q = make_fastdiv(a.Q);
    // 128 x 64 tiles where the groups fill them and there are two for every compute unit; 64 x 64 for fewer pixels, 128 x 32 for
    // groups of at most 32 output channels (half of a wider tile would be padding)
    if (prm.Kg <= 32) return launch_rag<128, 32>(prm, st);
    if ((prm.M + 127LL) / 128 * a.groups * ((prm.Kg + 63) / 64) >= 512) return launch_rag<128, 64>(prm, st);
    return launch_rag<64, 64>(prm, st);
}

hipError_t launch_conv_rag(const ConvArgs &a, hipStream_t st)
{
    const long long image = (long long)a.H * a.W * a.C, pixels = (long long)a.P * a.Q;
    const long long most = rag_images(a.H, a.W, a.C, a.K, a.R, a.stride, a.pad, a.groups, a.P, a.Q);
    for (long long n = 0; n < a.N; n += most) {
        ConvArgs part = a;
        part.N = (int)(a.N - n < most ? a.N - n : most);
        part.x = a.x + n * image;
        if (a.y) part.y = a.y + n * pixels * a.ldy;
        if (a.acc_out) part.acc_out = a.acc_out + n * pixels * a.K;
        const hipError_t e = launch_images(part, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace dfq
