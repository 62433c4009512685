// Window-reuse convolution for stride-1 layers with many pixels, fp16 / bf16 storage, filters in MFMA operand order.
//
// The packed-filter kernel of pwin_kernel.h splits the channels of a chunk over its waves, so that a layer of a few
// thousand pixels fills the chip; on a layer of a few hundred thousand pixels that is the wrong shape: its waves meet in
// an fp32 exchange through LDS that is larger than the operands (100 KB for 64 x 192 outputs, one workgroup per CU), so
// nothing covers a workgroup's prologue and epilogue, and each is paid again for every 3 us of multiplication.  Here
//   * no wave shares an output with another: a wave owns 32*TMB channels x 32*NBW pixels and walks all channels, 16 at a
//     time (one chunk = R*S taps of 16 channels).  Per tap and wave TMB fragments of filters come from L2 straight into
//     registers (1 KB each, coalesced) and NBW fragments of the input from the LDS slab, for TMB*NBW MFMAs: with
//     TMB = 2, NBW = 4 the vector memory path is asked for half of its 64 B/clk and LDS for half of its 128 B/clk;
//   * a slab position is 32 bytes (its 16 channels of the chunk), so the operand of tap (r,s) is one 16-byte read at a
//     constant offset from the window origin and eight consecutive pixels fall on distinct banks without padding;
//   * LDS is small enough for two workgroups per CU: one multiplies while the other starts or stores;
//   * the result is rounded in registers, turned in a wave-private piece of LDS and stored in 16-byte runs along the
//     output's contiguous axis.  For [N][K][OH][OW] the operands trade places (pixels are the rows of the MFMA block), so
//     that a lane holds four consecutive pixels of one channel; for [N][OH][OW][K] it holds four channels of one pixel.
//
// Measured (us per call, autotuned, before -> with this kernel): 64 images of 56x56x64 -> 192 in bf16 on the plain formats
// 115.6 -> 55.1 (conversion launch 7.5, this kernel 47 = 0.94 PFLOP/s of the 1.4 a large library product reaches), with
// packed filters 84 -> 47; 8 of 33x35x100 -> 130 (fp16) 35.2 -> 15.5; 16 of 112x112x64 -> 128 88 -> 46; 64 of 13x13x256 ->
// 384 32.7 -> 28.0.  Traced on the first layer: conversion launch 11 us (8 back to back), this kernel 43, the matrix units busy
// for 47 % of it (they reach 1.4 PFLOP/s under load, 32 us for this layer); the start and end of a workgroup, in which it does not
// multiply, are covered only as far as the other one on the CU does.  A persistent form of the kernel, whose first slab and
// filters of the next tile were fetched during the previous tile, needed 20 more registers and was slower (49.9).
//
// The input slab comes from a channel-innermost tensor (BWIN_INNER) or, on the plain formats,
//   * BWIN_BLOCKED: from a copy in the workspace that one conversion launch has written in exactly the order the slabs have:
//     [16-channel group][position][16 channels], position = the stacked, border-sharing position space of pwin_kernel.h with its
//     zero borders written out.  A slab is then one contiguous run of that copy, whatever the layer's width, channel count or
//     number of images: no per-position arithmetic, no bounds, and channel counts that are no multiple of 16 are padded with
//     zeros on the way;
//   * BWIN_PLANAR: from the planar input itself, for rows of whole 8-byte pieces: a thread loads four pixels of eight channels and
//     puts the channels of a pixel together with byte permutes, as in dwin_kernel.h; the slabs are cleared once, borders and all.
//     The copy moves the input three times (64 images of 56x56x64 10 us of 56.7); the launch ahead then packs the filters alone.
//     A workgroup's start takes longer (clearing, turning), and every channel tile turns the input again, so that small inputs
//     and layers of one chunk keep the copy (bwin_valid).  us per call with other inputs each time, copied -> as it is: 64 of
//     56x56x64 -> 192 in bf16 56.7 -> 54.2; on the same inputs 1012 of 16x16x32 -> 64 24.0 -> 18.6, 475 of 28x28x32 -> 64 30.6 ->
//     25.8, 33 of 24x24x256 -> 192 27.9 -> 24.7.  Rows that are no multiple of four pixels, or tiles of 32 channels, which turn as
//     much for half of the products, gained nothing.
#pragma once

#include "pwin_kernel.h"

namespace convfwd {

enum BwinInput { BWIN_INNER, BWIN_BLOCKED, BWIN_PLANAR };

template <int DT_, int R_, int S_, int WM_, int WN_, int TMB_, int NBW_, int AD_, int LBT_, BwinInput IN_, bool ONHWC_>
struct BwinCfg {
    static_assert(DT_ == CONV_F16 || DT_ == CONV_BF16, "16-bit storage only");
    static constexpr int DT = DT_, R = R_, S = S_, WM = WM_, WN = WN_, TMB = TMB_, NBW = NBW_, AD = AD_, LBT = LBT_;
    static constexpr bool BLK = IN_ == BWIN_BLOCKED, PLANAR = IN_ == BWIN_PLANAR, ONHWC = ONHWC_;
    static constexpr int RS = R * S;
    static_assert(RS % AD == 0, "the filter-fragment ring must divide the taps of a chunk");
    static constexpr int NT = 64 * WM * WN;
    static constexpr int TM = 32 * TMB * WM;      // output channels per workgroup
    static constexpr int TNP = 32 * NBW * WN;     // pixels per workgroup
    static constexpr int SLOTS = LBT * NT / 2;    // slab positions of one buffer: every thread stages LBT 16-byte vectors
    // a slab is two planes, channels 0..7 and 8..15 of each position; their distance leaves 64 bytes mod 128, so that
    // the staging writes (eight lanes = four positions of both planes) fall on distinct banks
    static constexpr size_t PLANE = ((size_t)SLOTS * 16 + 127) / 128 * 128 + 64;
    // planar input: half of the threads load a plane, QPT pieces of 4 pixels x 8 channels each; pieces without pixels are
    // written behind the planes
    static constexpr int QPT = (SLOTS / 4 + NT / 2 - 1) / (NT / 2);
    static constexpr size_t BUF_BYTES = 2 * PLANE + (PLANAR ? 64 : 0);
    // the wave's turned piece of the tile, rows padded by 16 bytes: [channel][pixel], one 32-channel block of EB*32 pixels
    // at a time (planar output), or [pixel][channel], 32 pixels of its channels at a time
    static constexpr int EB = NBW % 2 == 0 && !ONHWC ? 2 : 1;
    static constexpr int EROWS = 32, EPITCH = (ONHWC ? 32 * TMB : 32 * EB) + 8;
    static constexpr size_t EPI_BYTES = (size_t)WM * WN * EROWS * EPITCH * 2;
    static constexpr size_t SLAB_BYTES = BUF_BYTES > EPI_BYTES ? BUF_BYTES : EPI_BYTES;
    static constexpr size_t LDS_BYTES = 2 * SLAB_BYTES;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

struct BwinGeom {
    int PWs, PHs;   // row pitch and image pitch (in rows) of the stacked position space
    int PT, MT;     // pixel tiles, channel tiles
    long long NP;   // positions of the whole stack, borders included
    int span;       // most slab positions any pixel tile needs
    int rows;       // most slab rows
};

inline BwinGeom bwin_geom(int TM, int TNP, int R, int S, int N, int H, int W, int K, int pad, int OH, int OW)
{
    BwinGeom g;
    g.PWs = W + pad;
    g.PHs = H + pad;
    const long long P = (long long)N * OH * OW;
    g.PT = (int)((P + TNP - 1) / TNP);
    g.MT = (K + TM - 1) / TM;
    g.NP = ((long long)N * g.PHs + pad) * g.PWs + pad;
    long long rows = (TNP - 1 + OW - 1) / OW;  // a tile's first and last pixel are at most this many output rows apart
    if (rows > (long long)N * OH - 1) rows = (long long)N * OH - 1;
    long long imgs = (rows + OH - 1) / OH;
    if (imgs > N - 1) imgs = N - 1;
    const long long span = (rows + imgs * (g.PHs - OH)) * g.PWs + (OW - 1) + (long long)(R - 1) * g.PWs + S;
    g.span = span > 0x7fffffff ? 0x7fffffff : (int)span;
    const long long nrows = rows + imgs * (g.PHs - OH) + R;
    g.rows = nrows > 0x7fffffff ? 0x7fffffff : (int)nrows;
    return g;
}

// a.dX divides by PT (or by MT when channel tiles run fastest: a.order), a.dY by W + pad, a.dZ by H + pad; a.ws is the
// blocked input copy for BLK, a.in the channel-innermost or planar tensor otherwise; a.dW4 divides by W / 4 for PLANAR; a.blk_stride = bytes of one channel group of
// the copy.
template <class CFG>
__global__ __launch_bounds__(CFG::NT, 2) void bwin_kernel(ConvArgs a)
{
    typedef uint16_t elem_t;
    constexpr int DT = CFG::DT, R = CFG::R, S = CFG::S, RS = CFG::RS, WN = CFG::WN, TMB = CFG::TMB, NBW = CFG::NBW;
    constexpr int AD = CFG::AD, LBT = CFG::LBT, NT = CFG::NT, TM = CFG::TM, TNP = CFG::TNP;
    constexpr bool BLK = CFG::BLK, PLANAR = CFG::PLANAR, ONHWC = CFG::ONHWC;
    constexpr int QPT = CFG::QPT;
    typedef Mma<DT, 32> mma_t;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wm = wave / WN;
    const int li = lane & 31, g = lane >> 5;

    // ---- which tile: ids b, b+8, b+16, ... run on one XCD; give each XCD a contiguous run of logical tiles ---------
    const int PWs = (int)a.dY.d, PHs = (int)a.dZ.d, C16 = (a.C + 15) >> 4;
    int logical;
    {
        const int T = (int)gridDim.x;
        const int b = blockIdx.x, x = b & 7, q = b >> 3;
        const int per = T >> 3, rem = T & 7;
        logical = x * per + (x < rem ? x : rem) + q;
    }
    uint32_t mt_u, pt_u;
    if (a.order)
        a.dX.divmod((uint32_t)logical, pt_u, mt_u);
    else
        a.dX.divmod((uint32_t)logical, mt_u, pt_u);
    const int p0 = (int)pt_u * TNP;
    const int plast = (p0 + TNP < a.P ? p0 + TNP : a.P) - 1;
    const int mw0 = (int)mt_u * TM + wm * 32 * TMB;  // first channel of this wave
    const int pw0 = p0 + wn * 32 * NBW;              // first pixel of this wave

    auto base_pos = [&](int p) {
        uint32_t n, pix, oy, ox;
        a.dOHW.divmod((uint32_t)p, n, pix);
        a.dOW.divmod(pix, oy, ox);
        return ((int)n * PHs + (int)oy) * PWs + (int)ox;
    };
    // (a planar slab starts with a row)
    int lo;
    if constexpr (PLANAR)
        lo = __builtin_amdgcn_readfirstlane((int)a.dY.div((uint32_t)base_pos(p0))) * PWs;
    else
        lo = __builtin_amdgcn_readfirstlane(base_pos(p0));
    const int nposw = __builtin_amdgcn_readfirstlane(base_pos(plast)) + (R - 1) * PWs + S - lo;  // slab positions needed

    // ---- filter fragments: ring of AD taps, TMB fragments of 1 KB each ----------------------------------------------
    const __amdgpu_buffer_rsrc_t rfilt = make_rsrc(a.filt, a.filt_bytes);
    const uint32_t a_lane = (uint32_t)lane * 16u;
    const uint32_t a_mb_stride = (uint32_t)C16 * RS * 1024u;
    uint32_t a_soff = (uint32_t)(mw0 >> 5) * a_mb_stride;
    uint4 ar[AD][TMB];
    auto load_a = [&](auto slot_c, uint32_t soff) {
        constexpr int slot = decltype(slot_c)::value;
#pragma unroll
        for (int mb = 0; mb < TMB; ++mb) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rfilt, (int)a_lane, (int)(soff + (uint32_t)mb * a_mb_stride), 0);
            ar[slot][mb] = make_uint4(v.x, v.y, v.z, v.w);
        }
    };

    // ---- staging of the slab ------------------------------------------------------------------------------------------
    uint4 b_reg[PLANAR ? 1 : LBT];
    uint32_t t_goff[BLK || PLANAR ? 1 : LBT];
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    // planar: pieces of four neighbouring pixels of a row and eight channels
    constexpr uint32_t kGone = 0x80000000u;  // past any input of these layers, whatever channel offset is added
    constexpr int QP = PLANAR ? QPT : 1;
    uint32_t xr[QP][8][2], q_goff[QP], q_lds[QP][2];  // q_lds: pixels 0 and 2, 1 and 3
    const int gg = PLANAR ? wave / (NT / 128) : 0;    // plane of this wave's pieces
    // every other four lanes write the pixels of a pair in the other order: eight lanes, 64 bytes apart, then write distinct banks
    const uint32_t swap = (tid >> 2) & 1, sel_even = swap ? 0x07060302u : 0x05040100u, sel_odd = sel_even ^ 0x02020202u;
    if constexpr (PLANAR) {
        const int Y0 = (int)a.dY.div((uint32_t)lo);
        const int nrows = __builtin_amdgcn_readfirstlane((int)a.dY.div((uint32_t)base_pos(plast))) - Y0 + R;
        uint32_t n0, yy0;
        a.dZ.divmod((uint32_t)Y0, n0, yy0);
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            uint32_t r, k, dn, yy;
            a.dW4.divmod((uint32_t)(i * (NT / 2) + (tid & (NT / 2 - 1))), r, k);
            a.dZ.divmod(yy0 + r, dn, yy);
            const int n = (int)(n0 + dn), x = (int)k * 4;
            const bool ok = (int)r < nrows && (int)yy >= a.pad && n < a.N;
            q_goff[i] = ok ? (uint32_t)(((n * a.C + gg * 8) * a.H + (int)yy - a.pad) * a.W + x) * 2u : kGone;
            const uint32_t at = ok ? (uint32_t)gg * (uint32_t)CFG::PLANE + (uint32_t)((int)r * PWs + x + a.pad) * 16u : (uint32_t)(2 * CFG::PLANE);
            q_lds[i][0] = at + swap * 16u, q_lds[i][1] = at + 16u - swap * 16u;
        }
    }
    const uint32_t in_plane = (uint32_t)a.HW * 2u;
    auto load_piece = [&](int i, int chunk) {
        const int c0 = chunk * 16 + gg * 8;
        const uint32_t o = c0 < a.C ? q_goff[i] : kGone;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rin, (int)o, (int)((uint32_t)(chunk * 16 + j) * in_plane), 0);
            xr[i][j][0] = v[0], xr[i][j][1] = v[1];
        }
    };
    auto store_piece = [&](int i, int chunk, int buf) {
        const int have = a.C - chunk * 16 - gg * 8;
        if (have < 8) {  // what follows the last channel is another image's
#pragma unroll
            for (int j = 1; j < 8; ++j)
                if (j >= have) xr[i][j][0] = xr[i][j][1] = 0;
        }
        unsigned char* const Bs = smem_raw + (size_t)buf * CFG::SLAB_BYTES;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = __builtin_amdgcn_perm(xr[i][2 * j + 1][v / 2], xr[i][2 * j][v / 2], v & 1 ? sel_odd : sel_even);
            *(uint4*)(Bs + q_lds[i][v & 1] + (v / 2) * 32) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    };
    if constexpr (!BLK && !PLANAR) {
#pragma unroll
        for (int i = 0; i < LBT; ++i) {
            const int t = i * NT + tid;
            const int j = t >> 1, v8 = t & 1;
            uint32_t Y, X, n, yy;
            a.dY.divmod((uint32_t)(lo + j), Y, X);
            a.dZ.divmod(Y, n, yy);
            const bool ok = j < nposw && (int)X >= a.pad && (int)X < a.pad + a.W && (int)yy >= a.pad && (int)n < a.N;
            t_goff[i] = ok ? (uint32_t)((((int)n * a.H + (int)yy - a.pad) * a.W + (int)X - a.pad) * a.C + v8 * 8) * 2u : kOutOfRange;
        }
    }
    auto load_slab = [&](int chunk) {
        if constexpr (PLANAR) {
#pragma unroll
            for (int i = 0; i < QPT; ++i) load_piece(i, chunk);
        } else if constexpr (BLK) {
            // one contiguous run of the copy; the descriptor ends where the tile's positions do, so the loads past them
            // (and those past the last chunk) fetch nothing
            const char* base = (const char*)a.ws + (size_t)chunk * a.blk_stride + (size_t)lo * 32;
            const __amdgpu_buffer_rsrc_t rb = make_rsrc(base, chunk < C16 ? (uint32_t)nposw * 32u : 0u);
#pragma unroll
            for (int i = 0; i < LBT; ++i) {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rb, tid * 16, i * NT * 16, 0);
                b_reg[i] = make_uint4(v.x, v.y, v.z, v.w);
            }
        } else {
            const uint32_t c_bytes = (uint32_t)chunk * 32u;
#pragma unroll
            for (int i = 0; i < LBT; ++i) b_reg[i] = buffer_load_vec(rin, t_goff[i] == kOutOfRange ? kOutOfRange : t_goff[i] + c_bytes);
        }
    };
    auto store_slab = [&](int buf) {
        if constexpr (PLANAR) {  // (the first chunk)
#pragma unroll
            for (int i = 0; i < QPT; ++i) store_piece(i, 0, buf);
            return;
        }
        unsigned char* Bs = smem_raw + (size_t)buf * CFG::SLAB_BYTES + (tid & 1) * CFG::PLANE + (tid >> 1) * 16;
#pragma unroll
        for (int i = 0; i < (PLANAR ? 0 : LBT); ++i) *(uint4*)(Bs + i * (NT / 2) * 16) = b_reg[i];
    };

    load_slab(0);
    static_for<AD>([&](auto ic) { load_a(ic, a_soff + (uint32_t)decltype(ic)::value * 1024u); });

    // slab byte offset of the window origin of each of this lane's pixels, at this lane's 8 channels
    int bpos[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
        const int p = pw0 + nb * 32 + li;
        bpos[nb] = (base_pos(p < a.P ? p : plast) - lo) * 16 + g * (int)CFG::PLANE;
    }
    const int rowoff = PWs * 16;

    typename mma_t::acc_t acc[TMB][NBW];
#pragma unroll
    for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.0f;

    if constexpr (PLANAR) {  // only pixels are written to the slabs: their borders stay zero
        for (uint32_t u = tid; u < 2 * CFG::SLAB_BYTES / 16; u += NT) *(uint4*)(smem_raw + u * 16) = make_uint4(0, 0, 0, 0);
        __syncthreads();
    }
    store_slab(0);
    load_slab(1);
    __syncthreads();

    uint4 bf[2][NBW];
    auto read_tap = [&](const unsigned char* Bs, int r, int s, int set) {
        const int toff = r * rowoff + s * 16;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) bf[set][nb] = *(const uint4*)(Bs + bpos[nb] + toff);
    };
    read_tap(smem_raw, 0, 0, 0);

    constexpr int TSTORE = RS / 2;  // tap after which the next chunk's slab goes to LDS
    int buf = 0;
    // One chunk, as in pwin_kernel.h: STORE when another chunk follows, LOAD when one follows that.
    auto do_chunk = [&](auto store_c, auto load_c, int chunk) {
        constexpr bool STORE = decltype(store_c)::value, LOAD = decltype(load_c)::value;
        const unsigned char* Bs = smem_raw + (size_t)buf * CFG::SLAB_BYTES;
        const unsigned char* Bn = smem_raw + (size_t)(buf ^ 1) * CFG::SLAB_BYTES;
        static_for<RS>([&](auto tc) {
            constexpr int t = decltype(tc)::value, cur = t & 1, slot = t % AD;
            if constexpr (t + 1 < RS) {
                read_tap(Bs, (t + 1) / S, (t + 1) % S, cur ^ 1);
            } else if constexpr (STORE) {
                __syncthreads();  // publishes the slab stored at tap TSTORE; every wave holds its last operands of this one
                read_tap(Bn, 0, 0, cur ^ 1);
            } else {
                __syncthreads();  // the slabs are dead: the epilogue's rows overlay them
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) {
                    if constexpr (ONHWC)
                        acc[mb][nb] = mma_t::run(ar[slot][mb], bf[cur][nb], acc[mb][nb]);
                    else
                        acc[mb][nb] = mma_t::run(bf[cur][nb], ar[slot][mb], acc[mb][nb]);
                }
            constexpr int ta = t + AD;  // taps of consecutive chunks follow each other in the packed tensor
            if constexpr (ta < RS || STORE) load_a(std::integral_constant<int, slot>{}, a_soff + (uint32_t)ta * 1024u);
            if constexpr (PLANAR) {  // a piece at a time, spread around the middle of the chunk
                constexpr int i = (t - (TSTORE - QPT + 1)) / 2;
                if constexpr (t >= TSTORE - QPT + 1 && (t - (TSTORE - QPT + 1)) % 2 == 0 && i < QPT) {
                    if constexpr (STORE) store_piece(i, chunk + 1, buf ^ 1);
                    if constexpr (LOAD) load_piece(i, chunk + 2);
                }
            } else if constexpr (t == TSTORE) {
                if constexpr (STORE) store_slab(buf ^ 1);
                if constexpr (LOAD) load_slab(chunk + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr ((RS & 1) != 0) {
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) bf[0][nb] = bf[1][nb];
        }
        buf ^= 1;
        a_soff += RS * 1024u;
    };
    {
        int chunk = 0;
        for (; chunk + 2 < C16; ++chunk) do_chunk(std::true_type{}, std::true_type{}, chunk);
        if (chunk + 1 < C16) do_chunk(std::true_type{}, std::false_type{}, chunk++);
        do_chunk(std::false_type{}, std::false_type{}, chunk);
    }

    // ---- bias + activation + rounding, turned in this wave's own LDS rows, stored along the contiguous axis ----------
    constexpr int EPITCH = CFG::EPITCH;
    elem_t* const T = (elem_t*)smem_raw + (size_t)wave * CFG::EROWS * EPITCH;
    const __amdgpu_buffer_rsrc_t rbias = make_rsrc(a.bias, a.bias ? (uint32_t)a.K * 4u : 0u);
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(a.out, a.out_bytes);
    // lanes read what other lanes of the wave wrote (and the next round overwrites it): LDS serves a wave's accesses in
    // order, the compiler must keep theirs
    auto wave_order = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // the activation is a uniform branch around the whole conversion: one instruction per value inside it
    auto epilogue = [&](auto relu_c) {
        auto act = [&](float x) { return decltype(relu_c)::value ? (x > 0.0f ? x : 0.0f) : x; };
        if constexpr (ONHWC) {
            constexpr int LPR = TMB * 4, RPI = 64 / LPR;  // lanes per pixel (8 channels each), pixels per step
            const int px0 = lane / LPR, k = mw0 + (lane % LPR) * 8;
            f32x4 bs[TMB][4];
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    bs[mb][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rbias, (mw0 + mb * 32 + 8 * i + 4 * g) * 4, 0, 0));
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {  // a round: 32 pixels of all the wave's channels
                wave_order();
#pragma unroll
                for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const f32x4 b = bs[mb][i];
                        const uint32_t w0 = Prec<DT>::pack2_from_f32(act(acc[mb][nb][4 * i] + b[0]), act(acc[mb][nb][4 * i + 1] + b[1]));
                        const uint32_t w1 = Prec<DT>::pack2_from_f32(act(acc[mb][nb][4 * i + 2] + b[2]), act(acc[mb][nb][4 * i + 3] + b[3]));
                        *(uint2*)&T[li * EPITCH + mb * 32 + 8 * i + 4 * g] = make_uint2(w0, w1);
                    }
                wave_order();
#pragma unroll
                for (int it = 0; it < (32 + RPI - 1) / RPI; ++it) {
                    const int px = it * RPI + px0, p = pw0 + nb * 32 + px;
                    const uint4 x = *(const uint4*)&T[(px < 32 ? px : 0) * EPITCH + (lane % LPR) * 8];
                    // (a store past K or P is pointed out of range; K % 8 == 0 with this format)
                    const uint32_t o = px0 < RPI && px < 32 && p < a.P && k < a.K ? ((uint32_t)p * (uint32_t)a.K + (uint32_t)k) * 2u : kOutOfRange;
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{x.x, x.y, x.z, x.w}, rout, (int)o, 0, 0);
                }
            }
        } else {
            constexpr int EB = CFG::EB;  // 32-pixel blocks per round: a round is one 32-channel block of EB*32 pixels
            float bs[TMB];
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb) bs[mb] = buffer_load_elem<float>(rbias, (uint32_t)(mw0 + mb * 32 + li) * 4u);
            const bool vec = (a.OHW & 7) == 0;
            constexpr int LPR = EB * 4, RPI = 64 / LPR;  // lanes per channel (8 pixels each), channels per step
            const int c0 = lane / LPR;
#pragma unroll
            for (int nb0 = 0; nb0 < NBW; nb0 += EB) {
                // vec: eight consecutive pixels lie in one image and start on a 16-byte boundary of its plane; else
                // one pixel per lane and 2-byte stores, runs of up to 128 bytes of a plane
                const int pxl = vec ? (lane % LPR) * 8 : lane % (32 * EB), p = pw0 + nb0 * 32 + pxl;
                uint32_t n, pix;
                a.dOHW.divmod((uint32_t)(p < a.P ? p : 0), n, pix);
                const uint32_t o0 = ((n * (uint32_t)a.K + (uint32_t)mw0) * (uint32_t)a.OHW + pix) * 2u;
#pragma unroll
                for (int mb = 0; mb < TMB; ++mb) {
                    wave_order();
#pragma unroll
                    for (int j = 0; j < EB; ++j)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int nb = nb0 + j;
                            const uint32_t w0 = Prec<DT>::pack2_from_f32(act(acc[mb][nb][4 * i] + bs[mb]), act(acc[mb][nb][4 * i + 1] + bs[mb]));
                            const uint32_t w1 = Prec<DT>::pack2_from_f32(act(acc[mb][nb][4 * i + 2] + bs[mb]), act(acc[mb][nb][4 * i + 3] + bs[mb]));
                            *(uint2*)&T[li * EPITCH + j * 32 + 8 * i + 4 * g] = make_uint2(w0, w1);
                        }
                    wave_order();
                    if (vec) {
#pragma unroll
                        for (int it = 0; it < 32 / RPI; ++it) {
                            const int c = it * RPI + c0;
                            const uint4 x = *(const uint4*)&T[c * EPITCH + pxl];
                            const bool ok = p < a.P && mw0 + mb * 32 + c < a.K;
                            __builtin_amdgcn_raw_buffer_store_b128(u32x4{x.x, x.y, x.z, x.w}, rout,
                                                                   (int)(ok ? o0 + (uint32_t)((mb * 32 + c) * a.OHW) * 2u : kOutOfRange), 0, 0);
                        }
                    } else {
                        constexpr int CPI = 64 / (32 * EB);  // channels per step
                        const int cc = lane / (32 * EB);
#pragma unroll 4
                        for (int it = 0; it < 32 / CPI; ++it) {
                            const int c = it * CPI + cc;
                            const bool ok = p < a.P && mw0 + mb * 32 + c < a.K;
                            buffer_store_elem<elem_t>(T[c * EPITCH + pxl], rout, ok ? o0 + (uint32_t)((mb * 32 + c) * a.OHW) * 2u : kOutOfRange);
                        }
                    }
                }
            }
        }
    };
    if (a.relu)
        epilogue(std::true_type{});
    else
        epilogue(std::false_type{});
}

template <class CFG>
hipError_t bwin_launch_main(ConvArgs& a, hipStream_t s)
{
    const hipError_t e = ensure_dynamic_lds((const void*)bwin_kernel<CFG>, CFG::LDS_BYTES);
    if (e != hipSuccess) return e;
    const BwinGeom g = bwin_geom(CFG::TM, CFG::TNP, CFG::R, CFG::S, a.N, a.H, a.W, a.K, a.pad, a.OH, a.OW);
    a.filt_bytes = (uint32_t)packed_filter_bytes(a.K, ((a.C + 15) / 16) * 16, a.RS);
    // filters that fit an XCD's L2 beside the input: the channel tiles of one pixel tile run side by side, so the slab is
    // fetched from memory once; larger filters: pixel tiles of one channel tile, which stream the same fragments
    a.order = a.filt_bytes <= (2u << 20) ? 1 : 0;
    a.dX = make_fastdiv((uint32_t)(a.order ? g.MT : g.PT));
    a.dY = make_fastdiv((uint32_t)g.PWs);
    a.dZ = make_fastdiv((uint32_t)g.PHs);
    if (CFG::PLANAR) a.dW4 = make_fastdiv((uint32_t)(a.W / 4));
    a.blk_stride = (uint64_t)g.NP * 32;
    hipLaunchKernelGGL(bwin_kernel<CFG>, dim3((unsigned)(g.PT * g.MT)), dim3(CFG::NT), CFG::LDS_BYTES, s, a);
    return hipGetLastError();
}

template <class CFG>
hipError_t bwin_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    return bwin_launch_main<CFG>(a, s);
}

inline size_t bwin_copy_bytes(int N, int C, int H, int W, int pad)
{
    const size_t np = ((size_t)N * (H + pad) + pad) * (W + pad) + pad;
    return ((np * 32 * ((C + 15) / 16)) + 255) & ~(size_t)255;
}

template <class CFG>
size_t bwin_prep_workspace(const Variant&, const conv_desc& d, int, int)
{
    return bwin_copy_bytes(d.N, d.C, d.H, d.W, d.pad) + packed_filter_bytes(d.K, ((d.C + 15) / 16) * 16, CFG::RS);
}

template <class CFG>
hipError_t bwin_prep_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    unsigned char* const ws = (unsigned char*)a.ws;
    void* const ws_filt = ws + bwin_copy_bytes(a.N, a.C, a.H, a.W, a.pad);
    const hipError_t e = launch_prep_blk16(a.in, ws, a.N, a.C, a.H, a.W, a.pad, a.filt, ws_filt, a.K, a.RS, s);
    if (e != hipSuccess) return e;
    ConvArgs b = a;
    b.filt = ws_filt;
    return bwin_launch_main<CFG>(b, s);
}

// planar input: the filters alone are converted
template <class CFG>
size_t bwin_planar_workspace(const Variant&, const conv_desc& d, int, int)
{
    return packed_filter_bytes(d.K, ((d.C + 15) / 16) * 16, CFG::RS);
}

template <class CFG>
hipError_t bwin_planar_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    const hipError_t e = launch_pack_filters16_any(a.filt, a.ws, a.K, a.C, a.RS, s);
    if (e != hipSuccess) return e;
    ConvArgs b = a;
    b.filt = a.ws;
    return bwin_launch_main<CFG>(b, s);
}

template <class CFG>
bool bwin_valid(const Variant&, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != CFG::DT || d.R != CFG::R || d.S != CFG::S || d.stride != 1) return false;
    if (d.flags & CONV_FLAG_MAXPOOL_3X3S2) return false;
    const uint32_t fmt = d.flags & (CONV_FLAG_IN_NHWC | CONV_FLAG_FILT_KRSC | CONV_FLAG_FILT_PACKED | CONV_FLAG_FILT_WINOGRAD | CONV_FLAG_OUT_NHWC);
    if (CFG::BLK || CFG::PLANAR) {
        if (fmt != 0 || d.C < 8) return false;
    } else {
        if (fmt != (CONV_FLAG_IN_NHWC | CONV_FLAG_FILT_PACKED | (CFG::ONHWC ? CONV_FLAG_OUT_NHWC : 0u))) return false;
        if ((d.C % 16) != 0 || (CFG::ONHWC && (d.K % 8) != 0)) return false;
    }
    if (d.pad > CFG::R - 1 || d.pad > CFG::S - 1) return false;  // shared borders must hold every out-of-image tap
    const BwinGeom g = bwin_geom(CFG::TM, CFG::TNP, CFG::R, CFG::S, d.N, d.H, d.W, d.K, d.pad, OH, OW);
    if (CFG::PLANAR) {
        // below 4 MiB the copy is the cheaper way (it is read from L2, and a workgroup's start is most of such a call), and with a
        // single chunk of channels nothing hides the turning.  us per call, copied -> as it is: 119 images of 25x20x48 -> 64, 5.7 MB,
        // 13.1 -> 11.7; 41 of 20x20x96 -> 64, 3 MB, 10.5 -> 12.4; 66 of 56x56x16 -> 256, 7 MB, 33.2 -> 36.3.  Every kernel called, with the
        // line taken away: of 1122 drawn layers below 2 MiB this form was the fastest for none, from 2 to 4 MiB for 26 of 512, by 2 %, from 4 to
        // 8 for 69 of 226, from 8 to 32 for 249 of 497; as a valid variant it would only be measured in vain by every tuned call down there.
        // (The limits below rely on more than one chunk, too: the second is always asked for, with offsets that one image of C <= 16 would
        // carry past 32 bits)
        if (d.C <= 16 || (long long)d.N * d.C * d.H * d.W * 2 < 4 << 20) return false;
        // whole rows, the right border of the last one behind them; a piece of four aligned pixels for every thread's turn
        if ((d.W & 3) || (long long)g.rows * g.PWs + d.pad > CFG::SLOTS || (long long)g.rows * (d.W / 4) > CFG::QPT * (CFG::NT / 2)) return false;
    }
    if (g.span > CFG::SLOTS) return false;
    // (a tile more than half empty in either direction only wastes time: leave such layers to the smaller tiles)
    if (CFG::TM > ((d.K + 31) / 32) * 32 || (long long)CFG::TNP > 2LL * d.N * OH * OW) return false;
    const long long lim = 1LL << 31;
    if ((long long)g.PT * g.MT >= lim || g.NP >= lim / 32 + (CFG::BLK ? lim : 0)) return false;
    if (!CFG::BLK && (long long)d.N * (d.C + (CFG::PLANAR ? 16 : 0)) * d.H * d.W * 2 >= lim) return false;
    if ((long long)packed_filter_bytes(d.K, ((d.C + 15) / 16) * 16, CFG::RS) >= lim) return false;
    return true;
}

template <class CFG>
void bwin_register_one(std::vector<Variant>& out)
{
    Variant v;
    char buf[160];
    snprintf(buf, sizeof buf, "%s_%s_%dx%d_M%dN%d_w%dx%d_a%d_s%d%s", CFG::BLK || CFG::PLANAR ? "bwin" : "pwin_big", dtype_name(CFG::DT), CFG::R, CFG::S,
             CFG::TM, CFG::TNP, CFG::WM, CFG::WN, CFG::AD, CFG::SLOTS, CFG::BLK ? "" : CFG::PLANAR ? "_p" : CFG::ONHWC ? "_nhwc" : "_nchw");
    v.name = buf;
    v.dtype = CFG::DT;
    v.split = 1;
    v.tm = CFG::TM;
    v.tn = CFG::TNP;
    v.tk = 16 * CFG::RS;
    v.threads = CFG::NT;
    v.family = CFG::BLK || CFG::PLANAR ? FAM_WINDOW : FAM_NHWC;
    v.specificity = 4;
    v.traits = (CFG::BLK ? TRAIT_CONVERTS_FIRST : CFG::PLANAR ? TRAIT_CONVERTS_FILTERS : TRAIT_PACKED_FILTERS) | TRAIT_BIG_WINDOW;
    v.per_cu = CFG::LDS_BYTES * 2 <= 160 * 1024 ? 2 : 1;
    v.valid = &bwin_valid<CFG>;
    if constexpr (CFG::BLK) {
        v.launch = &bwin_prep_launch<CFG>;
        v.ws_extra = &bwin_prep_workspace<CFG>;
    } else if constexpr (CFG::PLANAR) {
        v.launch = &bwin_planar_launch<CFG>;
        v.ws_extra = &bwin_planar_workspace<CFG>;
    } else {
        v.launch = &bwin_launch<CFG>;
    }
    out.push_back(v);
}

// one tile shape for the three uses: plain formats behind the conversion launch, channel-innermost input to either output
// (PLANAR: and plain formats with the input as it is)
template <int DT, int R, int S, int WM, int WN, int TMB, int NBW, int AD, int LBT, bool PLANAR = false>
void bwin_register(std::vector<Variant>& out)
{
    if constexpr (PLANAR) bwin_register_one<BwinCfg<DT, R, S, WM, WN, TMB, NBW, AD, LBT, BWIN_PLANAR, false>>(out);
    bwin_register_one<BwinCfg<DT, R, S, WM, WN, TMB, NBW, AD, LBT, BWIN_BLOCKED, false>>(out);
    bwin_register_one<BwinCfg<DT, R, S, WM, WN, TMB, NBW, AD, LBT, BWIN_INNER, true>>(out);
    bwin_register_one<BwinCfg<DT, R, S, WM, WN, TMB, NBW, AD, LBT, BWIN_INNER, false>>(out);
}

}  // namespace convfwd
