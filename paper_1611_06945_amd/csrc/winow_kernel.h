// Winograd F(2x2, 3x3) on split products, 64 channels x 64 tiles a workgroup, a row of planes per wave (fp32 3x3 stride-1
// layers of many tiles).
//
// Arithmetic, filter transform and the fate of sums that are not finite are those of winos_kernel.h.  That kernel waits for its
// filters: a wave there has two planes of 32 tiles, a step of 96 x 32 brings 147 KB of filters, and what a plane needs of the
// input goes through LDS twice.  Here
//   * wave i of four has the planes (i, 0..3) of all 64 tiles: a fragment of filters is used for twelve products, not six, and
//     the 256 sums of a lane fill the accumulator registers (one wave per SIMD, 512 registers).
//   * Row i of B^T d needs two rows of a tile, so a lane reads those of its own tile and eight channels from the staged input and
//     has V in MFMA operand order without another pass through LDS.
//   * Input rows go straight to LDS (16 bytes a lane), two steps ahead, two buffers, one barrier a step.  A row's last vector may reach
//     into what follows it and no border is staged: columns outside the image are read from the end of a channel's slab, which
//     holds zeros.
//   * Between two MFMAs stand six vector instructions (a part of the next plane's operands, a row transform) or a load, in the
//     order of the source: a lone wave has to find its own cover.
//   * In the end a wave sums its row's columns, and the rows' sums meet in LDS in the wave that stores their channels.
//   * Workgroups take tile after tile, one per CU; a last round with tiles for no more than half of the workgroups halves them (winow_deal.h).  us a
//     call of fewer than 128 tiles, halved on XCDs that happened to have two workgroups for each -> on all: 17 of 13x13x256 -> 384 (84 tiles) 50.5 ->
//     37.0, 27 of 28x28x128 -> 64 (83) 28.4 -> 20.7, 8 of 56x56x64 -> 64 (98) 20.7 -> 16.0, 19 of 28x28x128 -> 128 (118) 30.7 -> 23.3.
// What bounds it: instruction issue.  A step is 96 MFMAs (3100 clocks) among 900 instructions, 4200 clocks on rows of 28 pixels, 5000 on rows of 56;
// vector loads cost 25 to 30 clocks of issue each.  Per tile the epilogue takes 7700, the next tile's addresses 2500, a workgroup's start 7300 to
// 8300 once.  On the layer below the clock falls to 1.94 GHz (2.23 with filters of zeros): the power limit is near.
// Measured (us per call, other inputs each time, filter transform included, winos_kernel's best -> here, same box in turn): 64 images of 56x56x64 ->
// 192 182 -> 160, 16 of 28x28x128 -> 256 40.6 -> 34.4, 33 of 28x28x128 -> 192 48.9 -> 47.4; 20 of 13x13x256 -> 384, 96 tiles, 35.1 -> 36.6
// (not taken).  Of 754 drawn layers 177 have 100 and more tiles; it is the fastest for 100 of them, there at 0.89 of the best time before (winos_kernel and
// the kernels ahead of it), and for 14 of 42 with 64 to 99, at 0.94.
// Tried: eight waves, a block of tiles each (225 us: the filters' loads twice over, 64 bytes a clock and CU); planes to LDS as
// they stand, without the columns' sums (11300 clocks an epilogue against 9600: LDS takes 64 bytes a clock); eight groups of filters ahead
// instead of four, and v_dot2_f32_bf16 for what a part leaves (no faster, a fifth slower).
#pragma once

#include "winos_kernel.h"
#include "winow_deal.h"

namespace convfwd {

template <int PITCH_>
struct WinowCfg {
    static constexpr int PITCH = PITCH_;  // floats per channel of the staged rows
    static constexpr int NT = 256, TM = 64, TT = 64;
    static constexpr int RING = 4;              // groups of filters in registers
    static constexpr int PV = PITCH / 4;        // 16-byte vectors per channel
    static constexpr int LV = PITCH / 64;       // vectors a thread fetches per step
    static constexpr int PERIOD = PV % 256 == 0 || 256 % PV == 0 ? (PV > 256 ? PV / 256 : 1) : 3;  // vectors of a thread until its place in a channel repeats
    static constexpr int CSTEP = PERIOD * 256 / PV;  // channels from there to its next vector at that place
    static constexpr int BUF = 16 * PITCH;      // floats of a step's rows
    static constexpr int EX = 4 * 4 * 2 * 64 * 4;  // floats of an exchange buffer: [from wave][to wave][pair of channels][lane][2 channels, 2 columns]
    static constexpr int FLOATS = 2 * BUF + 2 * EX;
    static_assert(PERIOD * 256 % PV == 0 && LV % PERIOD == 0 && FLOATS * 4 <= 160 * 1024, "");
};

struct WinowGeom {
    int TH, TW, tiles;
    int IR;        // staged rows of an image: 2 * TH + 2
    int rows_max;  // most rows a workgroup stages
    int W4;        // 16-byte vectors of a row
    int RW4;       // ... and of a staged row
    int KT, TN;    // channel tiles, groups of tiles
    FastDiv dTW, dIR, dTH, dRW4, dGroup;  // by TW, IR, TH, RW4 and 3 * TN
};

inline WinowGeom winow_geom(int pitch, int N, int K, int W, int OH, int OW)
{
    WinowGeom g;
    g.TH = (OH + 1) / 2;
    g.TW = (OW + 1) / 2;
    g.tiles = N * g.TH * g.TW;
    g.IR = 2 * g.TH + 2;
    const int up = (64 + g.TW - 2) / g.TW;  // tile rows between a workgroup's first and last tile
    int cross = (up + g.TH - 1) / g.TH;
    if (cross > N - 1) cross = N - 1;
    g.rows_max = 2 * up + 4 + 2 * cross;
    g.W4 = (W + 3) / 4;
    // Rows are padded where that spreads the tiles of a half wave, two floats apart, over more of the 64 banks
    g.RW4 = g.W4;
    int best = 33;
    for (int rw = g.W4; rw <= g.W4 + 4 && g.rows_max * rw < pitch / 4; ++rw) {
        uint8_t at[32] = {};
        int most = 0;
        for (int t = 0; t < 32; ++t) {
            const int n = ++at[(t / g.TW * rw * 4 + t % g.TW) & 31];
            if (n > most) most = n;
        }
        if (most < best) best = most, g.RW4 = rw;
    }
    g.KT = (K + 63) / 64;
    g.TN = (g.tiles + 63) / 64;
    return g;
}

struct WinowArgs {
    ConvArgs a;  // a.ws holds U
    WinowGeom d;
};

__device__ __forceinline__ const WinowArgs& winow_args_again()
{
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const WinowArgs*)p;
}

// EVEN: output rows of an even number of pixels, a tile's two outputs of a row are 8-byte aligned and both inside
template <class CFG, bool EVEN>
__global__ __launch_bounds__(CFG::NT, 1) void winow_kernel(WinowArgs w)
{
    const ConvArgs& a = w.a;
    const WinowGeom& d = w.d;
    constexpr int NT = CFG::NT, TM = CFG::TM, TT = CFG::TT, PITCH = CFG::PITCH, LV = CFG::LV, RING = CFG::RING;
    constexpr uint32_t kFar = 0x80000000u;  // tensors stay below 2 GiB: this offset plus any scalar offset is out of range
    asm volatile("" ::"s"(a.in), "s"(a.ws), "s"(a.N), "s"(a.C), "s"(a.H), "s"(a.W), "s"(a.K), "s"(a.pad), "s"(a.HW), "s"(a.OH), "s"(a.OW), "s"(a.OHW), "s"(a.in_bytes), "s"(d.TW), "s"(d.tiles), "s"(d.IR), "s"(d.W4), "s"(d.RW4));
    asm volatile("" ::"s"(d.KT), "s"(d.TN), "s"(d.dTW.mul), "s"(d.dTW.shift), "s"(d.dTW.d), "s"(d.dIR.mul), "s"(d.dIR.shift), "s"(d.dIR.d), "s"(d.dTH.mul), "s"(d.dTH.shift), "s"(d.dTH.d), "s"(d.dRW4.mul), "s"(d.dRW4.shift), "s"(d.dRW4.d), "s"(d.dGroup.mul), "s"(d.dGroup.shift), "s"(d.dGroup.d));
    typedef Mma<CONV_BF16, 32> mma_t;
    typedef __attribute__((address_space(3))) float lds_float;
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    extern __shared__ __attribute__((aligned(16))) float smem[];
    constexpr int BUF = CFG::BUF;
    float* const Ex = smem + 2 * BUF;  // exchange buffers of the epilogue

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C16 = (a.C + 15) >> 4, MBK = (a.K + 31) >> 5;
    const int mine = blockIdx.x >> 3;
    const WinowShare share = winow_share(d.KT * d.TN, (int)gridDim.x, blockIdx.x & 7);
    const int first = share.first, count = share.count, wgs = share.wgs, full = share.full, units = share.units;
    const bool halved = share.halved;
    if (mine >= units) return;
    struct Place {
        int t0, m0, t1;  // first tile, first channel, behind the last tile
    };
    auto place_of = [&](const WinowGeom& d, int q) {
        const bool half = halved && q >= full;
        const int at = first + (half ? full + ((q - full) >> 1) : q), second = half ? (q - full) & 1 : 0;
        uint32_t gr, rem;
        d.dGroup.divmod((uint32_t)at, gr, rem);
        const int left = d.KT - 3 * (int)gr, gs = left < 3 ? left : 3;
        const uint32_t tg = gs == 3 ? rem / 3u : rem >> (gs - 1);
        const int t0 = (int)tg * TT + second * (TT / 2), t1 = t0 + (half ? TT / 2 : TT);
        return Place{t0, (3 * (int)gr + (int)(rem - tg * gs)) * TM, t1 < d.tiles ? t1 : d.tiles};
    };

    // ---- transformed filters: group = (plane j of this wave's row, 32-channel block), three parts each -------------------
    const __amdgpu_buffer_rsrc_t ru = make_rsrc(a.ws, (uint32_t)C16 * 16u * (uint32_t)MBK * 3072u);
    const uint32_t a_lane = (uint32_t)lane * 16u;
    const uint32_t u_plane = (uint32_t)MBK * 3072u, u_step = u_plane * 16u;
    auto filters_of = [&](const Place& p) { return (uint32_t)(wave * 4) * u_plane + (uint32_t)(p.m0 >> 5) * 3072u; };
    uint4 ar[RING][3];
    auto load_a = [&](auto slot_c, auto grp_c, int q, uint32_t base) {
        constexpr int slot = decltype(slot_c)::value, grp = decltype(grp_c)::value;
        const uint32_t soff = base + (uint32_t)(grp >> 1) * u_plane + (uint32_t)(grp & 1) * 3072u;
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(ru, (int)(a_lane + q * 1024u), (int)soff, 0);
        ar[slot][q] = make_uint4(v.x, v.y, v.z, v.w);
    };

    // ---- input rows, straight to LDS: task = (channel of the step, staged row, 16-byte vector of the row) ------------------
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    auto stacked_row = [&](const WinowGeom& d, uint32_t tile_row) {
        uint32_t n, ty;
        d.dTH.divmod(tile_row, n, ty);
        return (int)n * d.IR + 2 * (int)ty;
    };
    auto first_row = [&](const WinowGeom& d, int t0) { return __builtin_amdgcn_readfirstlane(stacked_row(d, d.dTW.div((uint32_t)t0))); };
    constexpr int PV = CFG::PV, PERIOD = CFG::PERIOD;
    uint32_t r_goff[PERIOD];
    int row_q = mine, row_step = 0;
    auto aim_rows = [&](const WinowArgs& w) {
        const ConvArgs& a = w.a;
        const WinowGeom& d = w.d;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // (or what follows from it would be kept in registers through the steps)
        int s0 = 0, nrows = 0;         // (no rows behind the last tile)
        if (row_q < units) {
            const Place p = place_of(d, row_q);
            s0 = first_row(d, p.t0);
            if (p.t1 > p.t0) nrows = first_row(d, p.t1 - 1) + 4 - s0;
        }
#pragma unroll
        for (int i = 0; i < PERIOD; ++i) {
            const uint32_t v = (uint32_t)(i * NT + tid), c = v / PV, e = v % PV;
            uint32_t ri, xv, n, yy;
            d.dRW4.divmod(e, ri, xv);
            d.dIR.divmod((uint32_t)s0 + ri, n, yy);
            const int y = (int)yy - a.pad;
            const bool ok = (int)ri < nrows && (int)xv < d.W4 && (unsigned)y < (unsigned)a.H && (int)n < a.N;
            const uint32_t off = (uint32_t)((((int)n * a.C + (int)c) * a.H + y) * a.W + 4 * (int)xv) * 4u;
            r_goff[i] = ok ? off : kFar;
        }
    };
    const uint32_t chan_bytes = (uint32_t)a.HW * 4u;
    typedef __attribute__((address_space(3))) void lds_void;
    // The whole offset goes into the vector register, for the bounds check: a row's last vector reaches into what follows it.  (So
    // do channels past the last one into the next image; their filters are zero.)
    auto load_row = [&](int i, int buf) {
        const uint32_t at = (uint32_t)(row_step * 16 + i / PERIOD * CFG::CSTEP) * chan_bytes;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rin, (lds_void*)((lds_float*)smem + buf * BUF + wave * 256 + i * NT * 4), 16, (int)(r_goff[i % PERIOD] + at), 0, 0, 0);
    };
    auto rows_on = [&]() {
        if (++row_step == C16) {
            row_step = 0;
            row_q += wgs;
            aim_rows(winow_args_again());
        }
    };

    // ---- input transform: lane (li, g) makes column li of the blocks from channels 8g .. 8g+7, row `wave` of B^T d B ----------
    const int ra = wave == 0 ? 0 : wave == 2 ? 2 : 1, rb = wave == 2 ? 1 : wave == 3 ? 3 : 2;
    const float sb = wave == 1 ? kSplitScale : -kSplitScale;
    // LDS address, in buffer 0, of [row a, row b][block of tiles], and of zeros: the last vector of each channel holds no row
    uint32_t v_src[2][2], edges = 0;  // `edges`: bit 4 * block + column where a tile's column lies outside the image
    const uint32_t v_zero = (uint32_t)(uintptr_t)(lds_float*)smem + (uint32_t)(g * 8 * PITCH + PITCH - 4) * 4u;
    uint32_t o_src[2];  // byte offset of a tile's first output in channel 0, for the epilogue; bits 8 .. of `edges`: which of the four exist
    auto aim_transform = [&](const WinowArgs& w, const Place& p) {
        const int t0 = p.t0;
        const WinowGeom& d = w.d;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int li = tid & 31, g = tid >> 5 & 1;
        const int RW = d.RW4 * 4;
        edges = 0;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const bool in = t0 + nb * 32 + li < p.t1;
            const int t = in ? t0 + nb * 32 + li : t0;  // tiles past the end repeat the first one; never stored
            uint32_t gr, tx, n, ty;
            d.dTW.divmod((uint32_t)t, gr, tx);
            d.dTH.divmod(gr, n, ty);
            const int x = 2 * (int)tx - w.a.pad, srow = (int)n * d.IR + 2 * (int)ty;
            const uint32_t at = (uint32_t)(uintptr_t)(lds_float*)smem + (uint32_t)(g * 8 * PITCH + (srow - first_row(d, t0)) * RW + x) * 4u;
            v_src[0][nb] = at + (uint32_t)(ra * RW) * 4u;
            v_src[1][nb] = at + (uint32_t)(rb * RW) * 4u;
            edges |= (x < 0 ? 1u : 0u) << 4 * nb | (x + 2 >= w.a.W ? 4u : 0u) << 4 * nb | (x + 3 >= w.a.W ? 8u : 0u) << 4 * nb;
            o_src[nb] = (uint32_t)((int)n * w.a.K * w.a.OHW + 2 * (int)ty * w.a.OW + 2 * (int)tx) * 4u;
            const bool right = 2 * (int)tx + 1 < w.a.OW, below = 2 * (int)ty + 1 < w.a.OH;
            edges |= !in ? 0u : ((right ? 0xfu : 0x5u) & (below ? 0xfu : 0x3u)) << (8 * nb + 8);
        }
    };
    float t[4][2][8];  // [column][block of tiles][channel]
    struct Raw {
        float v[2][2];  // [row a, row b][channel of a pair]
    };
    // pair = (block of tiles, two channels)
    struct Source {
        uint32_t at[2][2];
    };
    auto source = [&](int j, uint32_t buf_off) {
        Source s;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int x = 0; x < 2; ++x)
                s.at[x][nb] = (j == 1 ? v_src[x][nb] : edges >> (4 * nb + j) & 1 ? v_zero : v_src[x][nb]) + buf_off;
        return s;
    };
    auto read_pair = [&](int j, int p, const Source& s) {
        Raw r;
#pragma unroll
        for (int x = 1; x >= 0; --x)  // (row a is needed first: one wait for both)
#pragma unroll
            for (int c = 0; c < 2; ++c) r.v[x][c] = *(const lds_float*)(uintptr_t)(s.at[x][p >> 2] + (uint32_t)(((p & 3) * 2 + c) * PITCH + j) * 4u);
        return r;
    };
    auto row_transform = [&](int j, int p, const Raw& r, int c) {
        t[j][p >> 2][(p & 3) * 2 + c] = __builtin_fmaf(r.v[1][c], sb, r.v[0][c] * kSplitScale);
    };
    // the parts of plane j, a pair of channels and one part at a time
    struct Parts {
        uint32_t w[2][3][4];  // [block of tiles][part][pair]
        __device__ __forceinline__ uint4 operand(int nb, int q) const { return make_uint4(w[nb][q][0], w[nb][q][1], w[nb][q][2], w[nb][q][3]); }
    };
    auto plane_value = [&](int j, int nb, int c) {
        return j == 0 ? t[0][nb][c] - t[2][nb][c] : j == 1 ? t[1][nb][c] + t[2][nb][c] : j == 2 ? t[2][nb][c] - t[1][nb][c] : t[1][nb][c] - t[3][nb][c];
    };
    float x0, x1;  // what is left of the pair at hand
    auto take_part = [&](int j, int p, int q, Parts& to) {
        if (q == 0) x0 = plane_value(j, p >> 2, (p & 3) * 2), x1 = plane_value(j, p >> 2, (p & 3) * 2 + 1);
        const uint32_t word = Prec<CONV_BF16>::pack2_from_f32(x0, x1);
        to.w[p >> 2][q][p & 3] = word;
        if (q < 2) {
            x0 -= __builtin_bit_cast(float, word << 16);
            x1 -= __builtin_bit_cast(float, word & 0xffff0000u);
        }
    };

    typename mma_t::acc_t acc[4][2][2];  // [plane][32-channel block][block of tiles]
    typedef std::integral_constant<int, 0> c0_t;
    // ---- epilogue: columns in the wave, rows through LDS, 16 channels x 32 tiles at a time -----------------------------------
    auto finish = [&](auto nbsc, const Place& at, const uint32_t* o_at, uint32_t outs) {
        constexpr int NBS = decltype(nbsc)::value;
        const WinowArgs& w = winow_args_again();
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, li = lane & 31, g = lane >> 5;
        const int kr = wave * 8 + g * 4;  // of 32 channels this thread stores four
        const __amdgpu_buffer_rsrc_t rbias = make_rsrc(w.a.bias, w.a.bias ? (uint32_t)w.a.K * 4u : 0u);
        f32x4 bias[2];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) bias[mb] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rbias, (at.m0 + mb * 32 + kr) * 4, 0, 0));
        // A round is a 32-channel block of a block of tiles: the columns' sums of this wave's plane row go to the wave that adds up
        // the rows of their channels, registers 4q .. 4q+3 to wave q and there to the same lane
        auto put = [&](auto rc) {
            constexpr int r = decltype(rc)::value, mb = r / NBS, nb = r % NBS;
            f32x4* const dst = (f32x4*)(Ex + (r & 1) * CFG::EX) + wave * 8 * 64 + lane;
#pragma unroll
            for (int v0 = 0; v0 < 16; v0 += 4) {
                float m[4][4];  // (read here: left alone, the compiler copies all 256 sums first and spills)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int j = 0; j < 4; ++j) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(m[v][j]) : "a"(acc[j][mb][nb][v0 + v]));
                float s0[4], s1[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) s0[v] = m[v][0] + m[v][1], s1[v] = m[v][1] - m[v][2];
#pragma unroll
                for (int v = 0; v < 4; ++v) s0[v] += m[v][2], s1[v] -= m[v][3];
                dst[(v0 / 2) * 64] = f32x4{s0[0], s1[0], s0[1], s1[1]};
                dst[(v0 / 2 + 1) * 64] = f32x4{s0[2], s1[2], s0[3], s1[3]};
            }
        };
        auto barrier = [&]() {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        asm volatile("s_nop 15\n\ts_nop 15");  // (the last products before the sums are read)
        put(c0_t{});
        // (what the rounds need, held in registers: the compiler would load it from the arguments again in each)
        uint64_t out = (uint64_t)w.a.out;
        uint32_t out_bytes = w.a.out_bytes, plane = (uint32_t)w.a.OHW * 4u, row = (uint32_t)w.a.OW * 4u;
        asm volatile("" : "+s"(out), "+s"(out_bytes), "+s"(plane));
        const __amdgpu_buffer_rsrc_t rout = make_rsrc((const void*)out, out_bytes);
        float floor = w.a.relu ? 0.0f : __builtin_nanf("");  // (the maximum with a NaN is the other operand; a NaN, of the bias, stays)
        int room = w.a.K - at.m0 - kr;  // channels from the first of the four to the last one
        asm volatile("" : "+v"(floor), "+v"(room));
        uint32_t base[2][4];  // of a tile's four outputs in the first of the channels
#pragma unroll
        for (int nb = 0; nb < NBS; ++nb)
#pragma unroll
            for (int q = 0; q < 4; q += EVEN ? 2 : 1) {
                const uint32_t o = o_at[nb] + (uint32_t)(at.m0 + kr) * plane + (q >> 1 ? row : 0u) + (q & 1) * 4u;
                base[nb][q] = outs >> (8 * nb + 8 + q) & 1 ? o : kFar;
                asm volatile("" : "+v"(base[nb][q]));
            }
        uint32_t bad = 0;  // bit 4 * round + channel: sums that are not finite
        barrier();
        static_for<2 * NBS>([&](auto rc) {
            constexpr int r = decltype(rc)::value, mb = r / NBS, nb = r % NBS;
            const f32x4* src = (const f32x4*)(Ex + (r & 1) * CFG::EX) + wave * 2 * 64 + lane;
            f32x4 m[4][2];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int p = 0; p < 2; ++p) m[i][p] = src[(i * 8 + p) * 64];
            if constexpr (r < 2 * NBS - 1) put(std::integral_constant<int, r + 1>{});
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float y[4];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const int e = (c & 1) * 2 + x;
                    y[x] = (m[0][c >> 1][e] + m[1][c >> 1][e]) + m[2][c >> 1][e];
                    y[2 + x] = (m[1][c >> 1][e] - m[2][c >> 1][e]) - m[3][c >> 1][e];
                }
                // no NaN and no infinity in any of the four (else they are stored again, below)
                const float all = (y[0] + y[1]) + (y[2] + y[3]);
                bad |= __builtin_fabsf(all) < __builtin_inff() ? 0u : 1u << (4 * r + c);
                const bool ok = mb * 32 + c < room;
#pragma unroll
                for (int q = 0; q < 4; ++q) y[q] = __builtin_fmaxf(__builtin_fmaf(y[q], kSplitUnscale, bias[mb][c]), floor);
                const int at = (int)((uint32_t)(mb * 32 + c) * plane);
#pragma unroll
                for (int dy = 0; dy < 2; ++dy) {
                    if constexpr (EVEN) {
                        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{__builtin_bit_cast(uint32_t, y[2 * dy]), __builtin_bit_cast(uint32_t, y[2 * dy + 1])},
                                                              rout, (int)(ok ? base[nb][2 * dy] : kFar), at, 0);
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, y[2 * dy]), rout, (int)(ok ? base[nb][2 * dy] : kFar), at, 0);
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, y[2 * dy + 1]), rout, (int)(ok ? base[nb][2 * dy + 1] : kFar), at, 0);
                    }
                }
            }
            if constexpr (r < 2 * NBS - 1) barrier();
        });
        if (__any(bad != 0)) {
            const ConvArgs& a = w.a;
            const WinowGeom& d = w.d;
#pragma unroll 1
            for (int e = 0; e < 8 * NBS; ++e) {
                const int r = e >> 2, ko = r / NBS * 32 + (e & 3), k = at.m0 + kr + ko, t = at.t0 + r % NBS * 32 + li;
                const bool mine_ = (bad >> e & 1) && k < a.K && t < at.t1;
                const uint64_t again = __ballot(mine_);
                if (!again) continue;
                uint32_t gr, tx, n, ty;
                d.dTW.divmod(mine_ ? (uint32_t)t : 0u, gr, tx);
                d.dTH.divmod(gr, n, ty);
                const int oy = 2 * (int)ty, ox = 2 * (int)tx;
                float y[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                winos_sum_again(a, lane, again, k, (int)n, oy - a.pad, ox - a.pad, y);
                const float b = a.bias && mine_ ? a.bias[k] : 0.0f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    y[q] += b;
                    if (a.relu) y[q] = y[q] > 0.0f ? y[q] : 0.0f;
                    const int y_ = oy + (q >> 1), x_ = ox + (q & 1);
                    buffer_store_elem<float>(y[q], rout, mine_ && y_ < a.OH && x_ < a.OW ? (uint32_t)(((int)n * a.K + k) * a.OHW + y_ * a.OW + x_) * 4u : kFar);
                }
            }
        }
    };

    // ---- pipeline: entering step i, `b0` holds the parts of its plane 0, t its columns 1 .. 3 (the last two pairs of column 3
    // still in `raw`), buffer (i + 1) % 2 the rows of step i+1.  The steps of a workgroup's tiles follow each other without a gap.
    Place here = place_of(d, mine);
    uint32_t now = filters_of(here);
    aim_rows(w);
#pragma unroll
    for (int i = 0; i < LV; ++i) load_row(i, 0);
    rows_on();
    __builtin_amdgcn_sched_barrier(0);  // (the wait below counts on this order)
    static_for<3 * RING - 3>([&](auto ic) {
        typedef std::integral_constant<int, decltype(ic)::value / 3> grp_t;
        load_a(grp_t{}, grp_t{}, 2 - decltype(ic)::value % 3, now);
    });
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < LV; ++i) load_row(i, 1);
    rows_on();
    aim_transform(w, here);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * RING - 3 + LV) : "memory");  // (the first rows)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    Parts b0, b1;
    Raw raw[2];
    static_for<4>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const Source src = source(j, 0u);
        Raw r[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) r[p] = read_pair(j, p, src);
#pragma unroll
        for (int p = 0; p < 8; ++p) row_transform(j, p, r[p], 0), row_transform(j, p, r[p], 1);
        raw[0] = r[6], raw[1] = r[7];
    });
    static_for<24>([&](auto ic) { take_part(0, decltype(ic)::value / 3, decltype(ic)::value % 3, b0); });
    int par = 0;  // buffer the rows of step i+2 go to
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // Plane j of a step for NBS blocks of tiles: one MFMA at a time, with what fits beneath it: a part of the next plane's operands, the
    // reads of a pair of column `col` of the next step's rows and, a few products later, the row transform of that pair (of `before`, of
    // the plane before, for the first two; none for before < 0)
    auto plane = [&](auto nbsc, auto firstc, auto jc, auto colc, auto beforec, const Parts& b, Parts& to, uint32_t buf_off, uint32_t next) {
        constexpr int NBS = decltype(nbsc)::value, j = decltype(jc)::value, col = decltype(colc)::value, before = decltype(beforec)::value, pairs = 4 * NBS;
        const Source src = source(col, buf_off);
        static_for<12 * NBS>([&](auto mc) {
            constexpr int m = decltype(mc)::value, mb = m / (6 * NBS), q = m % (6 * NBS) / NBS, nb = m % NBS, grp = j * 2 + mb, ahead = grp + RING - 1, p = m / 3;
            constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
            if constexpr (m % (2 * NBS) == 0)
                load_a(std::integral_constant<int, ahead % RING>{}, std::integral_constant<int, ahead % 8>{}, 2 - m % (6 * NBS) / (2 * NBS), ahead < 8 ? now : next);
            if constexpr (decltype(firstc)::value && q == 0)
                acc[j][mb][nb] = mma_t::run(ar[grp % RING][pa[q]], b.operand(nb, pb[q]), typename mma_t::acc_t{});
            else
                acc[j][mb][nb] = mma_t::run(ar[grp % RING][pa[q]], b.operand(nb, pb[q]), acc[j][mb][nb]);
            if constexpr (m % 3 > 0 && (p > 1 || before >= 0)) row_transform(p > 1 ? col : before, (p + pairs - 2) % pairs, raw[p & 1], m % 3 - 1);
            take_part((j + 1) % 4, p, m % 3, to);
            if constexpr (m % 3 == 2) raw[p & 1] = read_pair(col, p, src);
            if constexpr (j < 3 && m % (2 * NBS) == NBS) {  // (an instruction at a time: the waves' requests are served 64 bytes a clock)
                constexpr int at = j * 6 + m / (2 * NBS);
                if constexpr ((at + 1) * LV / 18 > at * LV / 18) load_row(at * LV / 18, par);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    typedef std::integral_constant<int, 1> c1_t;
    typedef std::integral_constant<int, 2> c2_t;
    typedef std::integral_constant<int, 3> c3_t;
    auto step = [&](auto nbsc, auto firstc, uint32_t next) {
        constexpr int NBS = decltype(nbsc)::value;
        const uint32_t buf_off = par ? 0u : (uint32_t)BUF * 4u;
        // (a half tile follows a whole one, or nothing: its columns are complete)
        typedef std::integral_constant<int, NBS == 1 && decltype(firstc)::value ? -1 : 3> before_t;
        __builtin_amdgcn_sched_barrier(0);
        plane(nbsc, firstc, c0_t{}, c0_t{}, before_t{}, b0, b1, buf_off, next);
        plane(nbsc, firstc, c1_t{}, c2_t{}, c0_t{}, b1, b0, buf_off, next);
        plane(nbsc, firstc, c2_t{}, c1_t{}, c2_t{}, b0, b1, buf_off, next);
        plane(nbsc, firstc, c3_t{}, c3_t{}, c1_t{}, b1, b0, buf_off, next);
        // (these belong beneath the products, not behind the branches that follow)
#pragma unroll
        for (int nb = 0; nb < NBS; ++nb)
#pragma unroll
            for (int q = 0; q < 3; ++q) asm volatile("" ::"v"(__builtin_bit_cast(u32x4, b0.operand(nb, q))));
#pragma unroll
        for (int nb = 0; nb < NBS; ++nb)
#pragma unroll
            for (int c = 0; c < 8; ++c) asm volatile("" ::"v"(t[1][nb][c]), "v"(t[2][nb][c]), "v"(t[3][nb][c]));
        asm volatile("s_waitcnt vmcnt(6)" ::: "memory");  // (six loads of filters are behind the rows)
        rows_on();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        par ^= 1;
        now = next;
    };
    int q = mine;
    Place there = here;
    auto ahead = [&](int i) {
        if (i < C16) return now + u_step;
        // the last step of a tile prepares the first one of the next
        q += wgs;
        if (q < units) {
            const WinowArgs& w = winow_args_again();
            there = place_of(w.d, q);
            aim_transform(w, there);
        }
        return filters_of(there);
    };
    auto tile = [&](auto nbsc) {
        const uint32_t o_at[2] = {o_src[0], o_src[1]}, outs = edges;
        step(nbsc, std::true_type{}, ahead(1));
#pragma unroll 1
        for (int i = 2; i <= C16; ++i) step(nbsc, std::false_type{}, ahead(i));
        finish(nbsc, here, o_at, outs);
        here = there;
    };
    const int whole = halved ? full : count;
    while (q < whole) tile(c2_t{});
    if (q < units) tile(c1_t{});
}

template <class CFG>
hipError_t winow_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    WinowArgs w = {a, winow_geom(CFG::PITCH, a.N, a.K, a.W, a.OH, a.OW)};
    WinowGeom& g = w.d;
    const size_t lds = sizeof(float) * CFG::FLOATS;
    const bool even = a.OW % 2 == 0;
    const hipError_t e = ensure_dynamic_lds(even ? (const void*)winow_kernel<CFG, true> : (const void*)winow_kernel<CFG, false>, lds);
    if (e != hipSuccess) return e;
    g.dTW = make_fastdiv((uint32_t)g.TW);
    g.dIR = make_fastdiv((uint32_t)g.IR);
    g.dTH = make_fastdiv((uint32_t)g.TH);
    g.dRW4 = make_fastdiv((uint32_t)g.RW4);
    g.dGroup = make_fastdiv((uint32_t)(3 * g.TN));
    hipLaunchKernelGGL(winos_filter_kernel, dim3((unsigned)((a.K + 31) / 32), (unsigned)((a.C + 15) / 16)), dim3(512), 0, s,
                       (const float*)a.filt, (uint4*)a.ws, a.K, a.C);
    const hipError_t e2 = hipGetLastError();
    if (e2 != hipSuccess) return e2;
    const dim3 grid((unsigned)winow_grid(g.TN * g.KT));
    if (even) hipLaunchKernelGGL((winow_kernel<CFG, true>), grid, dim3(CFG::NT), lds, s, w);
    else hipLaunchKernelGGL((winow_kernel<CFG, false>), grid, dim3(CFG::NT), lds, s, w);
    return hipGetLastError();
}

template <class CFG>
bool winow_valid(const Variant&, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != CONV_F32 || d.R != 3 || d.S != 3 || d.stride != 1 || d.pad > 1) return false;
    if (d.flags & ~(uint32_t)CONV_FLAG_RELU) return false;  // plain formats and filters, no fused pool
    if (d.C < 8 || d.K <= 32 || d.W < 4) return false;
    // 32-bit byte offsets beside an out-of-range marker
    const long long lim = 1LL << 31;
    if (((long long)d.N * d.C + 64) * d.H * d.W * 4 >= lim || (long long)d.N * d.K * OH * OW * 4 >= lim) return false;
    if ((long long)winos_filter_bytes(d.K, d.C) * 2 >= lim || (d.C + 15) / 16 > 65535) return false;
    if ((long long)d.N * ((OH + 1) / 2 + 2) * ((OW + 1) / 2 + 1) >= (1LL << 28)) return false;
    const WinowGeom g = winow_geom(CFG::PITCH, d.N, d.K, d.W, OH, OW);
    if (g.rows_max * g.W4 >= CFG::PV) return false;
    if ((long long)g.KT * g.TN >= lim) return false;
    return true;
}

template <class CFG>
void winow_register(std::vector<Variant>& out, const TileModel& model)
{
    Variant v;
    char buf[96];
    snprintf(buf, sizeof buf, "winos_f32_M%dT%d_p%d", CFG::TM, CFG::TT, CFG::PITCH);
    v.name = buf;
    v.dtype = CONV_F32;
    v.split = 1;
    v.tm = CFG::TM;
    v.tn = CFG::TT * 4;
    v.tk = 16 * 9;
    v.threads = CFG::NT;
    v.family = FAM_WINOGRAD;
    v.specificity = 5;
    v.traits = TRAIT_SPLIT_PRODUCTS;
    v.per_cu = 1;
    v.model = model;
    v.valid = &winow_valid<CFG>;
    v.launch = &winow_launch<CFG>;
    v.ws_extra = &winos_ws_bytes<CFG>;
    out.push_back(v);
}

}  // namespace convfwd
