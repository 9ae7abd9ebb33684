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

namespace dfq {

namespace {

constexpr int kRagThreads = 256;

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
            } else {
                store_tile_lane_ragged(acc[c][p], a, m, kc, count);
            }
        }
    }
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
    const double M = (double)a.N * a.P * a.Q, outputs = M * a.K;
    const double direct = 2990.0 + taps * (100.0 + 70.0 * Cg) + outputs * 0.0035 + outputs * taps * Cg * (taps > 1 && (Cg > 2 || taps >= 16) ? 58e-5 : 44e-5);
    const long long pieces = a.groups == 1 ? a.R * ((a.S * Cg + 15) / 16) : taps * ((Cg + 15) / 16), steps = (pieces + 3) / 4;
    const int bm = Kg <= 32 ? 128 : 64;
    const double tiles = (double)((long long)(M + bm - 1) / bm) * a.groups * ((Kg + 31) / 32), tail = tiles > 1280 ? tiles - 1280 : 0;
    double here = 3630.0 + 725.0 * steps + tiles * (1.36 + 1.4 * steps) + 1.1 * tail * steps;
    // the general epilogue, by the outputs a lane has of a group (870 pixels, 1x1, 8 groups of 18 -> 16, formats per channel: 6.7 us, 4.7;
    // accumulators of 24180 pixels in 12 groups of 3 -> 24 47.3, 34.9; of 45288 pixels in four groups of 31 -> 5 9.9, 42.0)
    if (a.acc_out || a.frac_w || a.shift < 0 || a.shift > 23) {
        const double part = (Kg < 16 ? Kg : 16) / 16.0, shares = part * tiles * (Kg <= 32 ? 1.0 : 0.5);
        here += a.acc_out ? 900.0 * part + 5.8 * shares : 1200.0 + 1000.0 * part + 2.4 * shares;
    }
    return direct * 15.0 > here * 16.0;
}

static hipError_t launch_images(const ConvArgs &a, hipStream_t st)
{
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
    // as many images per launch as 31-bit byte offsets into the input and 31-bit pixel and tile numbers reach
    const long long image = (long long)a.H * a.W * a.C, pixels = (long long)a.P * a.Q;
    const long long margin = ((long long)a.pad + a.R) * a.W * a.C;
    const long long tiles = (pixels / 64 + 1) * a.groups * ((a.K / a.groups + 31) / 32);
    long long most = ((1LL << 31) - 1 - margin) / image;
    most = most < ((1LL << 31) - 257) / pixels ? most : ((1LL << 31) - 257) / pixels;
    most = most < ((1LL << 31) - 1) / tiles ? most : ((1LL << 31) - 1) / tiles;
    if (most < 1) most = 1;
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
