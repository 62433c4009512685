// Window convolution for fp16 / bf16 layers of any stride in one launch: no conversion ahead of it, no workspace.
//
// The packed-filter kernels (pwin_kernel.h, bwin_kernel.h) want filters in MFMA operand order; on the other formats that is
// a conversion launch of 3 to 7 us and a workspace, more than a layer of a few thousand pixels takes to compute, and a call
// without a workspace cannot have it at all.  Here both operands are brought to MFMA order on the way through LDS:
//   * pixels are one linear run over (image, row, column), as in pwin_kernel.h, so that tiles are full whatever the image
//     size; the slab addresses input in the stacked position space of that kernel.  Strided layers keep the columns of a
//     row apart by their remainder, column c at (c mod stride)*hp + c / stride, so that neighbouring pixels read
//     neighbouring positions for every tap, whatever the stride;
//   * [N][C][H][W]: a thread loads four neighbouring pixels of eight channels (8 bytes each), puts the channels of a pixel
//     together with byte permutes and writes 16 bytes per pixel into a slab cleared once, borders and all;
//     (a row may start on an odd element: such loads are slower, but one of them replaces four);
//     [N][H][W][C]: 16-byte copies;
//   * [K][C][R][S]: the rows of a tile go to LDS as they are (whole 16-byte runs); a lane reads its 8 channels x R*S taps,
//     consecutive in memory, into registers and picks each tap's operand with byte permutes.  Rows that start on an odd
//     element are fetched from the 4-byte boundary ahead and shifted by a half word on the way to the permutes;
//     [K][R][S][C]: 16-byte pieces go to LDS in operand order, one window row at a time where the slab is large;
//   * WK waves share the channels of a chunk where a layer has few outputs, and add their sums through LDS in wave order;
//   * DB variants hold two buffers of each operand: pieces of the next stage are written between the MFMAs of this one, and
//     their registers loaded again for the stage after.  A wave that issues a whole chunk's loads at once waits 2000 to 3400
//     clocks for the memory pipeline to take them, ahead of its MFMAs.  The other variants are for layers of one chunk and
//     for tiles that share a CU.
// What bounds it (time stamps): a workgroup's start (arguments, addresses, first loads: 3000 to 5000 clocks) and end (sums,
// stores: 1500 to 3000) for small layers; LDS traffic in the loop, 1.5 KB an MFMA for 32 x 64 outputs per wave where an MFMA
// takes 8 clocks of the CU and LDS delivers 128 bytes in each.  Address arithmetic uses 24-bit multiplications throughout: a
// 32-bit one takes four times as long, and a thread's 9 pieces of filters cost 1500 clocks of a 12000-clock kernel with them.
// Measured, us per call with other inputs each time, before -> with this kernel: one image of 13x13x256 -> 384 in fp16 8.9 -> 6.7, 8 of
// 33x35x100 -> 130 15.4 -> 11.6 (both behind a conversion launch before), 32 of 56x56x128 -> 128 at stride 2 in bf16,
// channel-innermost, 16.8 -> 15.0.  Best variant over 2200 drawn 16-bit layers of 3x3 and 5x5 windows, geometric mean of the gain:
// plain formats without a workspace 2.1 (stride 1), 1.9 (stride 2), 2.4 (5x5), with one 1.23, 1.18, 1.19; channel-innermost
// 1.43, 1.17, 1.38.
#pragma once

#include "pwin_kernel.h"

namespace convfwd {

// v / D for 0 <= v < VMAX in one full-rate 24-bit multiplication and a shift (a 32-bit multiplication takes four times as long)
template <int D, int VMAX>
struct SmallDiv {
    static constexpr int SH = 22;
    static constexpr uint32_t MUL = ((1u << SH) + D - 1) / D;
    static constexpr bool exact()
    {
        for (int v = 0; v < VMAX; ++v)
            if ((int)(((uint64_t)v * MUL) >> SH) != v / D) return false;
        return (uint64_t)VMAX * MUL < (1ull << 32) && MUL < (1u << 24);
    }
    static_assert(exact(), "range of the multiplication");
    static __device__ __forceinline__ int div(int v) { return (int)(__umul24((uint32_t)v, MUL) >> SH); }
};

template <int DT_, int R_, bool NHWC_, int MB_, int WM_, int WN_, int WK_, int TMB_, int NBW_, int CG_, int SLOTS_, bool DB_, int FR_ = R_>
struct DwinCfg {
    static_assert(DT_ == CONV_F16 || DT_ == CONV_BF16, "16-bit storage only");
    static constexpr int DT = DT_, R = R_, RS = R_ * R_, MB = MB_, WM = WM_, WN = WN_, WK = WK_, TMB = TMB_, NBW = NBW_;
    static constexpr bool NHWC = NHWC_, DB = DB_;  // DB: the next chunk is written while this one is multiplied
    static constexpr int FR = FR_, NST = R_ / FR_;   // window rows whose filters are in LDS at a time, such stages of a chunk
    static_assert(NST * FR == R_ && (NST == 1 || (NHWC_ && DB_)), "stages of filters");
    static constexpr int CG = CG_, CB = 8 * CG_;      // groups of 8 channels and channels of a chunk
    static constexpr int SLOTS = SLOTS_;              // positions of the slab
    static constexpr int GPM = 64 / MB;               // channel groups an MFMA takes
    static constexpr int STEPS = CG / (GPM * WK);     // MFMA depths of a wave and chunk
    static_assert(STEPS * GPM * WK == CG, "a chunk is whole MFMAs for every wave");
    static constexpr int NT = 64 * WM * WN * WK;
    static constexpr int TM = MB * TMB * WM, TNP = MB * NBW * WN;
    // channel-innermost input: units (16 bytes: 8 channels of a position) of a thread
    static constexpr int UPT = (SLOTS * CG + NT - 1) / NT;
    // planar input: units of 8 channels x 4 pixels of a row
    static constexpr int QS = SLOTS / 4, QPT = (QS * CG + NT - 1) / NT;
    // planes of a channel group; 8 lanes of a channel-innermost copy (all groups of 8 / CG positions) write distinct banks
    static constexpr size_t PLANE = (size_t)SLOTS * 16 + (NHWC ? (CG >= 8 ? 16 : 128 / CG) : 0);
    // filters: rows of CG*RS 16-byte pieces, padded so that 8 rows read distinct banks; or planes of TM pieces per tap and group
    static constexpr int PPR = CG * FR * R;
    static constexpr size_t ROWP = (size_t)PPR * 16 + 16;
    static constexpr size_t APLANE = (size_t)TM * 16 + (CG >= 8 ? 16 : 128 / CG);
    static constexpr size_t A_BYTES = NHWC ? APLANE * FR * R * CG : ROWP * TM;
    static constexpr int FPT = (TM * PPR + NT - 1) / NT;
    static constexpr int EP = (NHWC ? TM : TNP) + 4;  // row pitch of the sums' buffer: [pixel][channel] or [channel][pixel]
    static constexpr size_t E_BYTES = (size_t)WK * (NHWC ? TNP : TM) * EP * 4;
    static constexpr size_t B_BYTES = PLANE * CG;
    static constexpr size_t DUMP = (A_BYTES + B_BYTES) * (DB ? 2 : 1);  // 16 bytes: where pixels outside the slab are written
    static constexpr size_t BODY_BYTES = ((DUMP + 16 > E_BYTES ? DUMP + 16 : E_BYTES) + 15) / 16 * 16;
    static constexpr size_t LDS_BYTES = BODY_BYTES + TM * 4;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
    // workgroups of a CU by LDS, and the waves per SIMD that the registers are fitted to
    static constexpr int PER_CU = LDS_BYTES * 3 <= 160 * 1024 ? 3 : LDS_BYTES * 2 <= 160 * 1024 ? 2 : 1;
    static constexpr int WPS_LDS = PER_CU * NT / 256;
    static constexpr int WPS_MAX = NHWC ? 3 : 2;
    static constexpr int WPS = WPS_LDS < 1 ? 1 : WPS_LDS > WPS_MAX ? WPS_MAX : WPS_LDS;
};

struct DwinGeom {
    int PW, IP, hp;  // row pitch, rows of an image, positions of one column remainder (stride > 1)
    int coff[5];     // position of window column s relative to column 0
    int reach;       // the largest of them
    int PT, MT;      // pixel tiles, channel tiles
    int span;        // most slab positions any pixel tile needs
    int rows;        // most slab rows
    int order;       // 1: the channel tiles of one pixel tile are consecutive
    int W4;          // 4-pixel pieces of a row
    FastDiv dT, dIP;
    uint32_t mPW, mIP, mHP, mST, mW4;  // ceil(2^20 / x): division of small numbers
};

inline DwinGeom dwin_geom(int TM, int TNP, int R, int N, int H, int W, int K, int stride, int pad, int OH, int OW)
{
    DwinGeom g;
    g.IP = H + pad;  // images share their borders; rows do too at stride 1
    g.hp = stride == 1 ? W + pad : (W + 2 * pad + stride - 1) / stride;
    g.PW = stride == 1 ? W + pad : g.hp * stride;
    g.reach = 0;
    for (int s = 0; s < 5; ++s) {
        g.coff[s] = s < R ? (s % stride) * (stride == 1 ? 0 : g.hp) + s / stride : 0;
        if (g.coff[s] > g.reach) g.reach = g.coff[s];
    }
    const long long P = (long long)N * OH * OW;
    g.PT = (int)((P + TNP - 1) / TNP);
    g.MT = (K + TM - 1) / TM;
    // a tile's first and last pixel are at most this many output rows and images apart
    long long rows = (TNP - 1 + OW - 1) / OW;
    if (rows > (long long)N * OH - 1) rows = (long long)N * OH - 1;
    long long imgs = (rows + OH - 1) / OH;
    if (imgs > N - 1) imgs = N - 1;
    const long long cross = (long long)g.IP - (long long)OH * stride;
    const long long span = (rows * stride + (cross > 0 ? imgs * cross : 0)) * g.PW + (OW - 1) + (long long)(R - 1) * g.PW + g.reach + 1;
    g.span = span > 0x7fffffff ? 0x7fffffff : (int)span;
    const long long nrows = rows * stride + (cross > 0 ? imgs * cross : 0) + R;
    g.rows = nrows > 0x7fffffff ? 0x7fffffff : (int)nrows;
    return g;
}

template <class CFG>
__global__ __launch_bounds__(CFG::NT, CFG::WPS) void dwin_kernel(ConvArgs a, DwinGeom d)
{
    typedef uint16_t elem_t;
    constexpr int DT = CFG::DT, R = CFG::R, RS = CFG::RS, MB = CFG::MB, WM = CFG::WM, WN = CFG::WN, WK = CFG::WK, TMB = CFG::TMB, NBW = CFG::NBW;
    constexpr int CG = CFG::CG, CB = CFG::CB, SLOTS = CFG::SLOTS, GPM = CFG::GPM, STEPS = CFG::STEPS, NT = CFG::NT, TM = CFG::TM, TNP = CFG::TNP;
    constexpr int FT = CFG::FR * R, NST = CFG::NST;  // taps of a stage, stages of a chunk
    constexpr int UPT = CFG::UPT, QPT = CFG::QPT, PPR = CFG::PPR, FPT = CFG::FPT, EP = CFG::EP;
    constexpr bool NHWC = CFG::NHWC;
    constexpr uint32_t kGone = 0x80000000u;  // past any tensor of these layers, whatever channel offset is added
    typedef Mma<DT, MB> mma_t;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    float* const bias_s = (float*)(smem_raw + CFG::BODY_BYTES);

    // The arguments are fetched together here: left to their first uses, each line of them is waited for by itself (2 images of
    // 14x14x64 -> 64 4.7 -> 4.3 us; with eight waves, whose first loads wait for fewer of them, 6.9 -> 7.1)
    if constexpr (NT <= 256) {
        asm volatile("" ::"s"(a.in), "s"(a.filt), "s"(a.bias), "s"(a.out), "s"(a.N), "s"(a.C), "s"(a.H), "s"(a.W), "s"(a.K), "s"(a.stride), "s"(a.pad),
                     "s"(a.P), "s"(a.HW), "s"(a.OHW), "s"(a.relu), "s"(a.in_bytes), "s"(a.filt_bytes), "s"(a.out_bytes));
        asm volatile("" ::"s"(a.dOHW.mul), "s"(a.dOHW.shift), "s"(a.dOHW.d), "s"(a.dOW.mul), "s"(a.dOW.shift), "s"(a.dOW.d), "s"(d.PW), "s"(d.IP), "s"(d.hp),
                     "s"(d.coff[R - 1]), "s"(d.reach), "s"(d.order), "s"(d.W4), "s"(d.dT.mul), "s"(d.dIP.mul), "s"(d.mPW), "s"(d.mIP), "s"(d.mW4));
    }
    const int tid = threadIdx.x, lane = tid & 63, li = lane & (MB - 1), g = lane / MB;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wm = (wave / WN) % WM, wk = wave / (WN * WM);

    // ---- which tile: ids b, b+8, ... run on one XCD; each XCD gets a contiguous run of logical tiles ------------------
    uint32_t mt_u, pt_u;
    {
        const int T = (int)gridDim.x, b = blockIdx.x, x = b & 7, per = T >> 3, rem = T & 7;
        const uint32_t logical = (uint32_t)(x * per + (x < rem ? x : rem) + (b >> 3));
        if (d.order)
            d.dT.divmod(logical, pt_u, mt_u);
        else
            d.dT.divmod(logical, mt_u, pt_u);
    }
    const int m0 = (int)mt_u * TM, p0 = (int)pt_u * TNP;
    const int plast = (p0 + TNP < a.P ? p0 + TNP : a.P) - 1;

    // ---- filters: what this thread loads of a stage ------------------------------------------------------------------
    const int chunks = (a.C + CB - 1) / CB;
    const bool odd = !NHWC && (a.C & 1);  // rows of the tile start on odd elements
    uint4 fr[FPT];
    uint32_t foff[FPT], fx = 0, fxoff = kGone;
    typedef SmallDiv<PPR, FPT * NT> div_t;
    const uint32_t rowb = (uint32_t)(a.C * RS) * 2u, fbase = (uint32_t)m0 * rowb;  // bytes of a row (below 2^24), the tile's first
    const int gx = tid & (CG - 1);  // channel group of this thread's channel-innermost pieces
#pragma unroll
    for (int i = 0; i < FPT; ++i) {
        const int v = i * NT + tid;
        if constexpr (NHWC) {
            const int row = (v / CG) & (TM - 1), tap = v / (CG * TM);
            foff[i] = tap < FT ? fbase + __umul24((uint32_t)(row * RS + tap), (uint32_t)a.C * 2u) + (uint32_t)gx * 16u : kGone;
        } else {
            const int row = div_t::div(v), pc = v - row * PPR;
            foff[i] = row < TM ? (fbase + __umul24((uint32_t)row, rowb) + (uint32_t)pc * 16u) & ~3u : kGone;
        }
    }
    if (odd && tid < TM) fxoff = (fbase + __umul24((uint32_t)tid, rowb) + (uint32_t)PPR * 16u) & ~3u;
    const __amdgpu_buffer_rsrc_t rfilt = make_rsrc(a.filt, a.filt_bytes);
    auto load_fi = [&](int i, int chunk, int stage) {
        const uint32_t soff = (uint32_t)chunk * CB * (NHWC ? 1 : RS) * 2u + (NST > 1 ? (uint32_t)(stage * FT * a.C) * 2u : 0u);
        const uint32_t o = NHWC && (chunk * CG + gx) * 8 >= a.C ? kGone : foff[i];
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rfilt, (int)o, (int)soff, 0);
        fr[i] = make_uint4(v.x, v.y, v.z, v.w);
        if (!NHWC && i == 0) fx = __builtin_amdgcn_raw_buffer_load_b32(rfilt, (int)fxoff, (int)soff, 0);
    };
    // (requested ahead of the tiles, for loads arrive in order, and put down behind them)
    const float bias_r = buffer_load_elem<float>(make_rsrc(a.bias, a.bias ? (uint32_t)a.K * 4u : 0u), tid < TM ? (uint32_t)(m0 + tid) * 4u : kOutOfRange);
#pragma unroll
    for (int i = 0; i < FPT; ++i) load_fi(i, 0, 0);

    // ---- input: what this thread loads of a chunk, and where it goes in the slab ------------------------------------------
    auto base_row = [&](int p, uint32_t& ox) {
        uint32_t n, pix, oy;
        a.dOHW.divmod((uint32_t)p, n, pix);
        a.dOW.divmod(pix, oy, ox);
        return (int)n * d.IP + (int)oy * a.stride;
    };
    auto base_pos = [&](int p) {
        uint32_t ox;
        const int Y = base_row(p, ox);
        return Y * d.PW + (int)ox;
    };
    uint32_t ox0, oxl;
    const int Y0 = __builtin_amdgcn_readfirstlane(base_row(p0, ox0)), Yl = __builtin_amdgcn_readfirstlane(base_row(plast, oxl));
    const int lo = __builtin_amdgcn_readfirstlane(Y0 * d.PW + (int)ox0);
    uint32_t n0, yy0;
    d.dIP.divmod((uint32_t)Y0, n0, yy0);
    // rows and columns relative to the slab's first row: small numbers, divided with 24-bit multiplications
    auto small_div = [&](uint32_t v, uint32_t mul) { return __umul24(v, mul) >> 20; };
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    const uint32_t plane = (uint32_t)a.HW * 2u;
    constexpr int UPT_ = NHWC ? UPT : 1, QPT_ = NHWC ? 1 : QPT, XP = NHWC ? UPT : QPT;
    uint32_t goff[XP];
    uint32_t woff[QPT_][4];
    if constexpr (NHWC) {
        const int nposw = __builtin_amdgcn_readfirstlane(Yl * d.PW + (int)oxl) + (R - 1) * d.PW + d.reach + 1 - lo;  // positions needed
#pragma unroll
        for (int i = 0; i < UPT; ++i) {
            const int j = i * (NT / CG) + tid / CG;
            const uint32_t c = ox0 + (uint32_t)j, r = small_div(c, d.mPW);
            uint32_t X = c - __umul24(r, (uint32_t)d.PW);
            const uint32_t yr = yy0 + r, dn = small_div(yr, d.mIP);
            const int n = (int)(n0 + dn), yy = (int)(yr - __umul24(dn, (uint32_t)d.IP));
            if (a.stride > 1) {
                const uint32_t ph = small_div(X, d.mHP);
                X = __umul24(X - __umul24(ph, (uint32_t)d.hp), (uint32_t)a.stride) + ph;
            }
            const bool ok = j < nposw && (int)X >= a.pad && (int)X < a.pad + a.W && yy >= a.pad && n < a.N;
            goff[i] = ok ? (uint32_t)(((n * a.H + yy - a.pad) * a.W + (int)X - a.pad) * a.C + gx * 8) * 2u : kGone;
        }
    } else {
        // four neighbouring pixels of one row and 8 channels; the last four of a row end with the row.  Only pixels are
        // written to the slab, chunk after chunk: it is cleared once, whole, and its borders stay zero
        const int rows = Yl - Y0 + R;
        const int swap = (tid >> 2) & 1;
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const int u = i * NT + tid, gg = u / CFG::QS;
            const uint32_t q = (uint32_t)(u % CFG::QS), r = small_div(q, d.mW4), k = q - __umul24(r, (uint32_t)d.W4);
            const uint32_t yr = yy0 + r, dn = small_div(yr, d.mIP);
            const int n = (int)(n0 + dn), yy = (int)(yr - __umul24(dn, (uint32_t)d.IP));
            const int x = (int)k * 4 < a.W - 4 ? (int)k * 4 : a.W - 4;
            const bool ok = gg < CG && (int)r < rows && yy >= a.pad && n < a.N;
            goff[i] = ok ? (uint32_t)(((n * a.C + gg * 8) * a.H + yy - a.pad) * a.W + x) * 2u : kGone;
            const int row0 = (int)__umul24(r, (uint32_t)d.PW) - (int)ox0;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                int X = x + (v ^ swap) + a.pad;
                if (a.stride > 1) {
                    const int quo = (int)small_div((uint32_t)X, d.mST);
                    X = (X - quo * a.stride) * d.hp + quo;
                }
                const int pos = row0 + X;
                woff[i][v] = ok && pos >= 0 && pos < SLOTS ? (uint32_t)(gg * CFG::PLANE) + (uint32_t)pos * 16u : kGone;
            }
        }
    }
    uint4 xv[UPT_];
    uint32_t xr[QPT_][8][2];
    // every other four lanes write the pixels of a pair in the other order: eight lanes, 64 bytes apart, then write distinct banks
    const uint32_t sel_even = (tid >> 2) & 1 ? 0x07060302u : 0x05040100u, sel_odd = sel_even ^ 0x02020202u;
    auto load_xi = [&](int i, int chunk) {
        if constexpr (NHWC) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rin, (int)((chunk * CG + gx) * 8 < a.C ? goff[i] : kGone), chunk * CB * 2, 0);
            xv[i] = make_uint4(v.x, v.y, v.z, v.w);
        } else {
            const uint32_t o = chunk * CB + (i * NT + tid) / CFG::QS * 8 < a.C ? goff[i] : kGone;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(rin, (int)o, (int)((uint32_t)(chunk * CB + j) * plane), 0);
                xr[i][j][0] = v[0], xr[i][j][1] = v[1];
            }
        }
    };
#pragma unroll
    for (int i = 0; i < XP; ++i) load_xi(i, 0);
    // one piece of filters to the buffer at A, one of input to the slab at B (offsets in LDS)
    auto store_fi = [&](int i, int chunk, uint32_t A) {
        const int v = i * NT + tid;
        uint4 f = fr[i];
        if constexpr (NHWC) {
            const int row = (v / CG) & (TM - 1), tap = v / (CG * TM);
            if ((i + 1) * NT <= TM * PPR || tap < FT) *(uint4*)(smem_raw + A + (size_t)(tap * CG + gx) * CFG::APLANE + row * 16) = f;
        } else {
            const int row = div_t::div(v);
            if ((chunk + 1) * CB > a.C) {
                // what follows the last channel of a row is the next row: its elements must not meet the zeros of the input,
                // for they may be infinite
                const int left = (a.C - chunk * CB) * RS + (odd ? (m0 + row) & 1 : 0), pc = v - row * PPR;  // halves of the row to keep
                const int n = left - pc * 8;
                if (n < 8) {
                    f.x &= n > 1 ? ~0u : n == 1 ? 0xFFFFu : 0u, f.y &= n > 3 ? ~0u : n == 3 ? 0xFFFFu : 0u;
                    f.z &= n > 5 ? ~0u : n == 5 ? 0xFFFFu : 0u, f.w &= n == 7 ? 0xFFFFu : 0u;
                }
                fx = 0;
            }
            // (rows of PPR pieces and one of padding)
            if ((i + 1) * NT <= TM * PPR || v < TM * PPR) *(uint4*)(smem_raw + A + (size_t)(v + row) * 16) = f;
            if (i == 0 && odd && tid < TM) *(uint32_t*)(smem_raw + A + (size_t)tid * CFG::ROWP + PPR * 16) = fx;
        }
    };
    auto store_xi = [&](int i, int chunk, uint32_t B) {
        if constexpr (NHWC) {
            const int j = i * (NT / CG) + tid / CG;
            if ((i + 1) * NT <= SLOTS * CG || j < SLOTS) *(uint4*)(smem_raw + B + (size_t)gx * CFG::PLANE + j * 16) = xv[i];
        } else {
            if ((a.C & 7) && (chunk + 1) * CB > a.C && (i * NT + tid) / CFG::QS == (a.C - chunk * CB) / 8) {
                // the last group holds channels of another image behind the last one
#pragma unroll
                for (int j = 1; j < 8; ++j)
                    if (j >= (a.C & 7)) xr[i][j][0] = xr[i][j][1] = 0;
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = __builtin_amdgcn_perm(xr[i][2 * j + 1][v / 2], xr[i][2 * j][v / 2], v & 1 ? sel_odd : sel_even);
                *(uint4*)(smem_raw + (woff[i][v] == kGone ? (uint32_t)CFG::DUMP : B + woff[i][v])) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    };
    // LDS: filters (one or two buffers), then slabs
    constexpr uint32_t A0 = 0, AN = (uint32_t)CFG::A_BYTES, B0 = AN * (CFG::DB ? 2 : 1), BN = (uint32_t)CFG::B_BYTES;
    if constexpr (!NHWC) {
        for (uint32_t u = tid; u < BN / 16 * (CFG::DB ? 2 : 1); u += NT) *(uint4*)(smem_raw + B0 + u * 16) = make_uint4(0, 0, 0, 0);
        __syncthreads();
    }

    // ---- this wave's block -----------------------------------------------------------------------------------------------
    int bpos[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
        const int p = p0 + (wn * NBW + nb) * MB + li;
        bpos[nb] = (base_pos(p < a.P ? p : plast) - lo) * 16;
    }
    constexpr int AV = MB == 32 ? 16 : 4;
    typename mma_t::acc_t acc[TMB][NBW];
#pragma unroll
    for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int v = 0; v < AV; ++v) acc[mb][nb][v] = 0.0f;

    const int rowoff = d.PW * 16;
    int coff[R];
#pragma unroll
    for (int s = 0; s < R; ++s) coff[s] = d.coff[s] * 16;

    // A chunk is XSL slots: stage after stage, a wave's MFMA depths, the taps of the stage.  A slot's operands are read during
    // the slot before it, across the barrier between two stages too: that stands in a stage's last slot, whose operands every
    // wave then holds.
    constexpr int FSL = FT * STEPS, XSL = FSL * NST;
    uint4 bf[2][NBW], af[2][TMB];
    uint32_t raw[NHWC ? 1 : TMB][NHWC ? 1 : RS * 4 + 1];
    auto read_slot = [&](auto slot_c, int chunk, int set) {
        constexpr int k = decltype(slot_c)::value, stage = k / FSL, st = k % FSL / FT, t = k % FT;
        const uint32_t par = CFG::DB ? (uint32_t)(chunk * NST + stage) & 1u : 0u, xpar = CFG::DB ? (uint32_t)chunk & 1u : 0u;
        const unsigned char* const As = smem_raw + A0 + par * AN;
        const unsigned char* const Bs = smem_raw + B0 + xpar * BN + stage * CFG::FR * rowoff;
        const int q = (wk * STEPS + st) * GPM + g;
        const unsigned char* const Bq = Bs + (size_t)q * CFG::PLANE;
        const int toff = (t / R) * rowoff + coff[t % R];
#pragma unroll
        for (int mb = 0; mb < TMB; ++mb) {
            const int row = (wm * TMB + mb) * MB + li;
            if constexpr (NHWC) {
                af[set][mb] = *(const uint4*)(As + (size_t)(t * CG + q) * CFG::APLANE + row * 16);
            } else if constexpr (t == 0) {
                const unsigned char* const Ar = As + (size_t)row * CFG::ROWP + (size_t)q * RS * 16;
#pragma unroll
                for (int i = 0; i < RS; ++i) {
                    const uint4 v = *(const uint4*)(Ar + i * 16);
                    raw[mb][4 * i] = v.x, raw[mb][4 * i + 1] = v.y, raw[mb][4 * i + 2] = v.z, raw[mb][4 * i + 3] = v.w;
                }
                if (odd) raw[mb][RS * 4] = *(const uint32_t*)(Ar + RS * 16);
            }
        }
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) bf[set][nb] = *(const uint4*)(Bq + bpos[nb] + toff);
    };
    // One chunk; 2 or more, 1 or no others follow (MORE).  DB: piece by piece between the MFMAs, the next stage's filters and
    // the next chunk's input go to the other buffers and their registers are loaded again for the stage and the chunk after,
    // so that every load has a whole stage or chunk to arrive and the issue of loads (which waits where the memory pipeline is
    // full) keeps no wave from its MFMAs.  The second chunk's input is requested beneath the FIRST chunk's products, for the same
    // reason: ahead of them it held the workgroup for 2000 of 23000 clocks (8 images of 33x35x100 -> 130 11.55 -> 11.26 us; over 190 drawn
    // layers the tiles of 64 and 128 channels take 0.97 to 0.98 of what they took)
    auto compute = [&](auto more_c, auto first_c, int chunk) {
        constexpr int MORE = decltype(more_c)::value;
        constexpr bool FIRST = decltype(first_c)::value;
        if constexpr (!CFG::DB) read_slot(std::integral_constant<int, 0>{}, chunk, 0);
        static_for<XSL>([&](auto slot_c) {
            constexpr int k = decltype(slot_c)::value, stage = k / FSL, fs = k % FSL, t = k % FT, cur = k & 1;
            if constexpr (!NHWC) {
                if constexpr (t == 0) {
                    if (odd) {
#pragma unroll
                        for (int mb = 0; mb < TMB; ++mb) {
                            const uint32_t sh = ((m0 + (wm * TMB + mb) * MB + li) & 1) * 2;  // bytes
#pragma unroll
                            for (int i = 0; i < RS * 4; ++i) raw[mb][i] = __builtin_amdgcn_alignbyte(raw[mb][i + 1], raw[mb][i], sh);
                        }
                    }
                }
#pragma unroll
                for (int mb = 0; mb < TMB; ++mb) {
                    uint32_t w[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        constexpr int RSc = RS;
                        const int e0 = 2 * j * RSc + t, e1 = (2 * j + 1) * RSc + t;
                        w[j] = __builtin_amdgcn_perm(raw[mb][e1 >> 1], raw[mb][e0 >> 1],
                                                     (e1 & 1 ? 0x07060000u : 0x05040000u) | (e0 & 1 ? 0x0302u : 0x0100u));
                    }
                    af[cur][mb] = make_uint4(w[0], w[1], w[2], w[3]);
                }
            }
            if constexpr (CFG::DB && fs == FSL - 1) __syncthreads();
            if constexpr (k + 1 < XSL)
                read_slot(std::integral_constant<int, k + 1 < XSL ? k + 1 : 0>{}, chunk, cur ^ 1);
            else if constexpr (CFG::DB && MORE >= 1)
                read_slot(std::integral_constant<int, 0>{}, chunk + 1, cur ^ 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) {
                    if constexpr (NHWC)
                        acc[mb][nb] = mma_t::run(af[cur][mb], bf[cur][nb], acc[mb][nb]);
                    else
                        acc[mb][nb] = mma_t::run(bf[cur][nb], af[cur][mb], acc[mb][nb]);
                }
            if constexpr (CFG::DB) {
                // channel-innermost pieces (a copy each) spread evenly over the slots ahead of the barrier; planar ones, which
                // are turned on the way, in two places
                constexpr int d1 = stage + 1 < NST ? 0 : 1, d2 = stage + 2 < NST ? 0 : NST == 1 ? 2 : 1;  // chunks from here to the next stages
                constexpr int fat = FSL - 2 - FT / 3, xat = XSL - 2, FN = FSL - 1, XN = XSL - 1;
                constexpr int f0 = fs == FN ? 0 : NHWC ? fs * FPT / FN : 0, f1 = fs == FN ? 0 : NHWC ? (fs + 1) * FPT / FN : fs == fat ? FPT : 0;
                // the first chunk's products stand above the requests for the second chunk's input too, in the slots ahead of XL
                constexpr int XL = FIRST ? (XSL + 2) / 3 : 0, KX = k - XL;
                constexpr int x0 = k == XN || KX < 0 ? 0 : NHWC ? KX * XP / (XN - XL) : 0;
                constexpr int x1 = k == XN || KX < 0 ? 0 : NHWC ? (KX + 1) * XP / (XN - XL) : k == xat ? XP : 0;
                if constexpr (KX < 0 && MORE >= 1)
                    static_for<(k + 1) * XP / (XL ? XL : 1) - k * XP / (XL ? XL : 1)>([&](auto ic) { load_xi(k * XP / (XL ? XL : 1) + decltype(ic)::value, chunk + 1); });
                const uint32_t A = A0 + (((uint32_t)(chunk * NST + stage) & 1u) ^ 1u) * AN, B = B0 + (((uint32_t)chunk & 1u) ^ 1u) * BN;
                static_for<f1 - f0>([&](auto ic) {
                    if constexpr (d1 <= MORE) store_fi(f0 + decltype(ic)::value, chunk + d1, A);
                    if constexpr (d2 <= MORE) load_fi(f0 + decltype(ic)::value, chunk + d2, (stage + 2) % NST);
                });
                static_for<x1 - x0>([&](auto ic) {
                    if constexpr (MORE >= 1) store_xi(x0 + decltype(ic)::value, chunk + 1, B);
                    if constexpr (MORE >= 2) load_xi(x0 + decltype(ic)::value, chunk + 2);
                });
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        if constexpr (CFG::DB && (XSL & 1) != 0 && MORE >= 1) {  // the next chunk starts with set 0
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) bf[0][nb] = bf[1][nb];
            if constexpr (NHWC) {
#pragma unroll
                for (int mb = 0; mb < TMB; ++mb) af[0][mb] = af[1][mb];
            }
        }
    };

    auto store_all = [&](int chunk) {
        static_for<FPT>([&](auto ic) { store_fi(decltype(ic)::value, chunk, A0); });
        static_for<XP>([&](auto ic) { store_xi(decltype(ic)::value, chunk, B0); });
    };
    auto load_all = [&](int fchunk, int fstage, int xchunk) {
        static_for<FPT>([&](auto ic) { load_fi(decltype(ic)::value, fchunk, fstage); });
        static_for<XP>([&](auto ic) { load_xi(decltype(ic)::value, xchunk); });
    };
    store_all(0);
    if (tid < TM) bias_s[tid] = bias_r;
    if constexpr (CFG::DB) {
        if (chunks * NST > 1) static_for<FPT>([&](auto ic) { load_fi(decltype(ic)::value, NST > 1 ? 0 : 1, NST > 1 ? 1 : 0); });
        __syncthreads();
        read_slot(std::integral_constant<int, 0>{}, 0, 0);
        constexpr std::true_type first{};
        constexpr std::false_type later{};
        int chunk = 0;
        if (chunks > 2) {
            compute(std::integral_constant<int, 2>{}, first, chunk++);
            for (; chunk + 2 < chunks; ++chunk) compute(std::integral_constant<int, 2>{}, later, chunk);
            compute(std::integral_constant<int, 1>{}, later, chunk++);
        } else if (chunks == 2) {
            compute(std::integral_constant<int, 1>{}, first, chunk++);
        }
        compute(std::integral_constant<int, 0>{}, later, chunk);
    } else {
        if (chunks > 1) load_all(1, 0, 1);
        __syncthreads();
        for (int chunk = 0;;) {
            compute(std::integral_constant<int, 0>{}, std::false_type{}, chunk);
            __syncthreads();
            if (++chunk == chunks) break;
            store_all(chunk);
            if (chunk + 1 < chunks) load_all(chunk + 1, 0, chunk + 1);
            __syncthreads();
        }
    }

    // ---- sums to LDS, added in wave order; bias + activation + rounding; stored along the contiguous axis -----------------
    float* const E = (float*)smem_raw;
    constexpr int EWK = (NHWC ? TNP : TM) * EP;
#pragma unroll
    for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int i = 0; i < AV / 4; ++i) {
                const int m = (wm * TMB + mb) * MB, p = (wn * NBW + nb) * MB, r = 8 * i + 4 * g;
                float* const e = E + wk * EWK + (NHWC ? (p + li) * EP + m + r : (m + li) * EP + p + r);
                *(float4*)e = make_float4(acc[mb][nb][4 * i], acc[mb][nb][4 * i + 1], acc[mb][nb][4 * i + 2], acc[mb][nb][4 * i + 3]);
            }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(a.out, a.out_bytes);
    auto finish = [&](float x, float b) {
        x += b;
        return a.relu ? (x > 0.0f ? x : 0.0f) : x;
    };
    auto sum4 = [&](int at) {
        float4 v = *(const float4*)(E + at);
#pragma unroll
        for (int w = 1; w < WK; ++w) {
            const float4 u = *(const float4*)(E + w * EWK + at);
            v.x += u.x, v.y += u.y, v.z += u.z, v.w += u.w;
        }
        return v;
    };
    // a thread keeps its place along the contiguous axis and steps along the other one
    if (NHWC || (a.OHW & 7) == 0) {
        // eight consecutive channels of a pixel, or pixels of a channel (one image, 16-byte boundary of its plane)
        constexpr int PER = NHWC ? TM / 8 : TNP / 8, STEP = NT / PER, OUTER = NHWC ? TNP : TM;
        static_assert(NT % PER == 0, "threads of a row");
        const int inner = tid % PER * 8, outer0 = tid / PER;
        uint32_t o = kOutOfRange;
        float4 b0, b1;
        if constexpr (NHWC) {
            b0 = *(const float4*)(bias_s + inner), b1 = *(const float4*)(bias_s + inner + 4);
            if (m0 + inner < a.K) o = ((uint32_t)(p0 + outer0) * (uint32_t)a.K + (uint32_t)(m0 + inner)) * 2u;
        } else {
            uint32_t n, pix;
            a.dOHW.divmod((uint32_t)(p0 + inner), n, pix);
            if (p0 + inner < a.P) o = ((n * (uint32_t)a.K + (uint32_t)(m0 + outer0)) * (uint32_t)a.OHW + pix) * 2u;
        }
        const uint32_t step = (uint32_t)STEP * (uint32_t)(NHWC ? a.K : a.OHW) * 2u;
#pragma unroll 4
        for (int outer = outer0; outer < OUTER; outer += STEP) {
            const float4 v0 = sum4(outer * EP + inner), v1 = sum4(outer * EP + inner + 4);
            if constexpr (!NHWC) {
                const float b = bias_s[outer];
                b0 = b1 = make_float4(b, b, b, b);
            }
            const u32x4 w = {Prec<DT>::pack2_from_f32(finish(v0.x, b0.x), finish(v0.y, b0.y)),
                             Prec<DT>::pack2_from_f32(finish(v0.z, b0.z), finish(v0.w, b0.w)),
                             Prec<DT>::pack2_from_f32(finish(v1.x, b1.x), finish(v1.y, b1.y)),
                             Prec<DT>::pack2_from_f32(finish(v1.z, b1.z), finish(v1.w, b1.w))};
            const bool in = o != kOutOfRange && (NHWC ? p0 + outer < a.P : m0 + outer < a.K);
            __builtin_amdgcn_raw_buffer_store_b128(w, rout, (int)(in ? o + (uint32_t)((outer - outer0) / STEP) * step : kOutOfRange), 0, 0);
        }
    } else if constexpr (!NHWC) {
        constexpr int PX = TNP < NT ? TNP : NT, STEP = NT / PX;
#pragma unroll
        for (int px = tid % PX; px < TNP; px += PX) {
            const int outer0 = tid / PX, p = p0 + px;
            uint32_t n, pix;
            a.dOHW.divmod((uint32_t)(p < a.P ? p : 0), n, pix);
            uint32_t o = ((n * (uint32_t)a.K + (uint32_t)(m0 + outer0)) * (uint32_t)a.OHW + pix) * 2u;
            const int left = p < a.P ? a.K - m0 : 0;  // channels of the tile to store
            const float* e = E + outer0 * EP + px;
#pragma unroll 8
            for (int m = outer0; m < TM; m += STEP) {
                float v = e[0];
#pragma unroll
                for (int w = 1; w < WK; ++w) v += e[w * EWK];
                buffer_store_elem<elem_t>(Prec<DT>::from_f32(finish(v, bias_s[m])), rout, m < left ? o : kOutOfRange);
                e += STEP * EP;
                o += (uint32_t)STEP * (uint32_t)a.OHW * 2u;
            }
        }
    }
}

template <class CFG>
hipError_t dwin_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    const hipError_t e = ensure_dynamic_lds((const void*)dwin_kernel<CFG>, CFG::LDS_BYTES);
    if (e != hipSuccess) return e;
    DwinGeom g = dwin_geom(CFG::TM, CFG::TNP, CFG::R, a.N, a.H, a.W, a.K, a.stride, a.pad, a.OH, a.OW);
    // a run of tiles shares an XCD's L2, and what its tiles do not share every XCD fetches for itself: the channel tiles of one
    // pixel tile run side by side where the input is the larger tensor, the pixel tiles of one channel tile where the filters are
    g.order = a.filt_bytes <= a.in_bytes ? 1 : 0;
    g.dT = make_fastdiv((uint32_t)(g.order ? g.MT : g.PT));
    g.dIP = make_fastdiv((uint32_t)g.IP);
    g.W4 = (a.W + 3) / 4;
    auto magic = [](int x) { return (uint32_t)(((1 << 20) + x - 1) / x); };
    g.mPW = magic(g.PW), g.mIP = magic(g.IP), g.mHP = magic(g.hp), g.mST = magic(a.stride), g.mW4 = magic(g.W4);
    hipLaunchKernelGGL(dwin_kernel<CFG>, dim3((unsigned)(g.PT * g.MT)), dim3(CFG::NT), CFG::LDS_BYTES, s, a, g);
    return hipGetLastError();
}

template <class CFG>
bool dwin_valid(const Variant&, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != CFG::DT || d.R != CFG::R || d.S != CFG::R || d.stride > 4) return false;
    const uint32_t fmt = CFG::NHWC ? CONV_FLAG_IN_NHWC | CONV_FLAG_FILT_KRSC | CONV_FLAG_OUT_NHWC : 0u;
    if ((d.flags & ~(uint32_t)CONV_FLAG_RELU) != fmt) return false;
    if (CFG::NHWC && ((d.C % 8) != 0 || (d.K % 8) != 0)) return false;
    if (d.C < 8 || ((d.C & 1) && (d.K & 1))) return false;  // (filters are fetched in whole 4-byte words)
    if (d.pad > CFG::R - 1) return false;                   // shared borders must hold every out-of-image tap
    const DwinGeom g = dwin_geom(CFG::TM, CFG::TNP, CFG::R, d.N, d.H, d.W, d.K, d.stride, d.pad, OH, OW);
    if (g.span > CFG::SLOTS) return false;
    if (!CFG::NHWC && (d.W < 4 || (long long)g.rows * ((d.W + 3) / 4) > CFG::QS)) return false;
    // v / x = v * ceil(2^20 / x) >> 20 for v * x < 2^20: columns and rows of a slab
    const long long small = 1LL << 20;
    if ((long long)(CFG::SLOTS + g.PW) * g.PW >= small || (long long)(g.IP + g.rows) * g.IP >= small) return false;
    // (a tile more than half empty in either direction only wastes time: leave such layers to the smaller tiles)
    if (CFG::TM > 32 && CFG::TM > ((d.K + 31) / 32) * 32) return false;
    if (CFG::TNP > 64 && (long long)CFG::TNP > 2LL * d.N * OH * OW) return false;
    const long long lim = 1LL << 31;
    if ((long long)g.PT * g.MT >= lim || ((long long)d.N * g.IP + d.pad + CFG::R) * g.PW + CFG::SLOTS >= lim) return false;
    if ((long long)d.N * (d.C + CFG::CB) * d.H * d.W * 2 >= lim || (long long)d.N * d.K * OH * OW * 2 >= lim) return false;
    if ((long long)d.C * CFG::RS * 2 >= 1 << 24) return false;
    return ((long long)d.K + CFG::TM) * (d.C + CFG::CB) * CFG::RS * 2 < lim;
}

template <class CFG>
void dwin_register_one(std::vector<Variant>& out, const TileModel& model)
{
    Variant v;
    char buf[160];  // (without the rows of a stage: no two tiles differ in them alone, and a test holds the names apart)
    snprintf(buf, sizeof buf, "%sdwin_%s_%dx%d_M%dN%d_w%dx%dx%d_b%d_c%d_s%d%s", CFG::NHWC ? "nhwc_" : "", dtype_name(CFG::DT), CFG::R, CFG::R,
             CFG::TM, CFG::TNP, CFG::WM, CFG::WN, CFG::WK, CFG::MB, CFG::CB, CFG::SLOTS, CFG::DB ? "_db" : "");
    v.name = buf;
    v.dtype = CFG::DT;
    v.split = 1;
    v.tm = CFG::TM;
    v.tn = CFG::TNP;
    v.tk = CFG::CB * CFG::RS;
    v.threads = CFG::NT;
    v.family = CFG::NHWC ? FAM_NHWC : FAM_WINDOW;
    v.specificity = 4;
    v.traits = TRAIT_DIRECT_WINDOW;
    v.per_cu = CFG::PER_CU;
    v.model = model;
    v.valid = &dwin_valid<CFG>;
    v.launch = &dwin_launch<CFG>;
    out.push_back(v);
}

// planar
template <int DT, int R, int MB, int WM, int WN, int WK, int TMB, int NBW, int CG, int SLOTS, bool DB>
void dwin_planar(std::vector<Variant>& out, const TileModel& model)
{
    dwin_register_one<DwinCfg<DT, R, false, MB, WM, WN, WK, TMB, NBW, CG, SLOTS, DB>>(out, model);
}
// channel-innermost
template <int DT, int R, int MB, int WM, int WN, int WK, int TMB, int NBW, int CG, int SLOTS, bool DB, int FR = R>
void dwin_inner(std::vector<Variant>& out, const TileModel& model)
{
    dwin_register_one<DwinCfg<DT, R, true, MB, WM, WN, WK, TMB, NBW, CG, SLOTS, DB, FR>>(out, model);
}

template <int DT>
void dwin_register_all(std::vector<Variant>& out)
{
    //          DT  R  MB WM WN WK TMB NBW CG SLOTS DB     call  own   chunk  grow
    dwin_planar<DT, 3, 16, 1, 1, 8, 1, 2, 32, 128, false>(out, {1.60, 3.09, 2.628, 0.80});  // M16  N32
    dwin_planar<DT, 3, 16, 1, 1, 4, 1, 2, 16, 128, false>(out, {2.63, 1.68, 1.661, 0.45});  // M16  N32
    dwin_planar<DT, 3, 16, 1, 1, 4, 1, 2, 16, 256, false>(out, {1.86, 3.12, 2.489, 0.80});  // M16  N32
    dwin_planar<DT, 3, 16, 1, 4, 1, 1, 2, 4, 512, false>(out, {2.23, 1.36, 1.316, 0.67});  // M16  N128
    dwin_planar<DT, 3, 32, 1, 1, 4, 1, 1, 8, 128, true>(out, {1.73, 2.48, 1.125, 0.30});  // M32  N32
    dwin_planar<DT, 3, 32, 1, 1, 4, 1, 1, 8, 256, false>(out, {2.29, 1.95, 1.602, 0.38});  // M32  N32
    dwin_planar<DT, 3, 32, 1, 2, 2, 1, 1, 4, 256, false>(out, {2.51, 1.23, 0.998, 0.48});  // M32  N64
    dwin_planar<DT, 3, 32, 1, 2, 2, 1, 1, 4, 256, true>(out, {2.26, 1.55, 0.905, 0.40});  // M32  N64
    dwin_planar<DT, 3, 32, 1, 2, 2, 1, 1, 4, 768, false>(out, {2.30, 2.22, 1.703, 0.36});  // M32  N64
    dwin_planar<DT, 3, 32, 1, 4, 1, 1, 1, 2, 512, true>(out, {2.58, 1.30, 0.789, 0.55});  // M32  N128
    dwin_planar<DT, 3, 32, 2, 2, 1, 1, 2, 2, 512, true>(out, {2.23, 2.33, 1.021, 0.49});  // M64  N128
    dwin_planar<DT, 3, 32, 2, 2, 1, 1, 2, 2, 1024, true>(out, {1.34, 4.13, 1.286, 0.80});  // M64  N128
    dwin_planar<DT, 3, 32, 2, 2, 1, 1, 2, 2, 1024, false>(out, {2.38, 2.37, 1.527, 0.60});  // M64  N128
    dwin_planar<DT, 3, 32, 2, 2, 2, 1, 2, 4, 512, true>(out, {1.52, 3.62, 1.455, 0.80});  // M64  N128
    dwin_planar<DT, 5, 16, 1, 1, 4, 1, 2, 16, 128, false>(out, {1.05, 4.53, 3.479, 0.30});  // M16  N32
    dwin_planar<DT, 5, 32, 1, 2, 2, 1, 1, 4, 256, false>(out, {0.50, 2.96, 2.807, 0.39});  // M32  N64
    dwin_planar<DT, 5, 32, 1, 4, 1, 1, 1, 2, 512, false>(out, {1.99, 2.06, 1.573, 0.68});  // M32  N128
    dwin_planar<DT, 5, 32, 1, 4, 1, 1, 1, 2, 512, true>(out, {1.43, 2.67, 1.447, 0.80});  // M32  N128
    dwin_planar<DT, 5, 32, 1, 4, 1, 1, 2, 2, 768, false>(out, {1.19, 2.91, 4.510, 0.73});  // M32  N256
    dwin_inner<DT, 3, 16, 1, 4, 1, 1, 2, 4, 512, true, 1>(out, {2.78, 0.99, 0.650, 0.74});  // M16  N128
    dwin_inner<DT, 3, 32, 1, 1, 4, 1, 1, 8, 128, true>(out, {1.92, 1.78, 0.575, 0.30});  // M32  N32
    dwin_inner<DT, 3, 32, 1, 1, 4, 1, 1, 8, 256, true, 1>(out, {1.96, 1.87, 0.762, 0.30});  // M32  N32
    dwin_inner<DT, 3, 32, 1, 2, 2, 1, 1, 4, 256, true, 1>(out, {3.29, 0.55, 0.473, 0.85});  // M32  N64
    dwin_inner<DT, 3, 32, 1, 2, 2, 1, 2, 4, 512, true, 1>(out, {2.47, 1.48, 0.809, 0.67});  // M32  N128
    dwin_inner<DT, 3, 32, 2, 1, 2, 1, 2, 4, 512, true, 1>(out, {1.75, 2.46, 0.889, 0.30});  // M64  N64
    dwin_inner<DT, 3, 32, 2, 2, 2, 1, 2, 4, 512, true, 1>(out, {1.28, 2.63, 1.125, 0.80});  // M64  N128
    dwin_inner<DT, 3, 32, 2, 2, 2, 2, 2, 4, 832, true, 1>(out, {0.83, 4.13, 1.730, 0.30});  // M128 N128
    dwin_inner<DT, 5, 16, 1, 1, 4, 1, 2, 16, 128, false>(out, {1.79, 1.63, 3.108, 0.80});  // M16  N32
    dwin_inner<DT, 5, 32, 1, 2, 2, 1, 1, 4, 256, true, 1>(out, {2.83, 0.63, 1.147, 0.90});  // M32  N64
    dwin_inner<DT, 5, 32, 2, 2, 2, 1, 2, 4, 512, true, 1>(out, {1.28, 2.76, 2.720, 0.30});  // M64  N128
}

}  // namespace convfwd
