// Direct window kernel for fp32 3x3 and 5x5 layers of any stride, its products on the 16-bit matrix units.
//
// The fp32 matrix rate is 1/16 of the bf16 one: 5x5 and strided layers ran at 3 to 85 TFLOP/s on the implicit GEMMs and pwin32_kernel.
// Arithmetic as in winos_kernel.h: every fp32 operand is three bf16 numbers, six partial products a product, operands scaled by 2^24
// ahead of the splits; sums that are not finite are taken again from the definition.
//   * Leading products and the five small ones have accumulators of their own: a sum is then rounded once for sixteen channels and tap.
//     Error against 64 bits (2-norm, relative, half-normal inputs; six products in one accumulator -> here, the pick before): 20x20x352 ->
//     64 5x5 14.5e-7 -> 5.8e-7, 8.0e-7; 16x16x88 -> 49 7.2e-7 -> 2.7e-7, 4.3e-7; 19x23x130 -> 64 3x3 stride 2 5.1e-7 -> 1.9e-7, 2.1e-7.
//     Where a wave takes all channels, a chunk's leading sums are added to those before it: 3 images of 16x16x220 -> 160 5x5 4.5e-7 ->
//     1.3e-7, 2 of 40x40x176 -> 16 3.7e-7 -> 1.2e-7 (the implicit GEMM split eight ways 4.7e-7, 3.6e-7), 29 of 44x44x304 -> 112 3x3 stride 2 3.3e-7 -> 1.1e-7
//     (that one 3.5e-7), 20 of 13x13x256 -> 96 3x3 2.8e-7 -> 1.0e-7 (the fp32 window kernel split four ways 2.2e-7), for up to 1 % of the time where
//     it is the fastest (17 of 33x33x416 -> 64 5x5 186.5 -> 188.2 us, 5 of 28x31x224 -> 256 107.1 -> 108.4, 48 of 63x66x128 -> 27 3x3 103.8 -> 104.7).  Waves that
//     split the channels: 1.0e-7 to 5.2e-7.  Over 303 drawn layers whose untuned pick moved here the error is 0.34 of the former pick's (geometric
//     mean; 0.72 at most), over 382 that a tuned call moves 0.41 of the fastest other kernel's (0.72 at most).
//   * A small kernel ahead splits the filters into MFMA operand order; fragments come from L2 straight into registers.
//   * Input is read four bytes a lane (any row length, border and stride), split and stored as [part][eight channels][position], rows
//     of the window stacked over images; a lane's window is one address, a tap an offset.  Only positions that the tile has are staged.
//   * Tiles of 128 pixels with four waves side by side for layers that fill the chip; for smaller ones the waves split the channels,
//     with a slab each and, where a wave has its own, no barrier in the loop.
// What bounds it: at 5x5 the matrix units (50 images of 14x14x424 -> 96: 120 GFLOP of bf16 products in 115 us); at 3x3 the
// staging of a chunk, 2200 clocks of loads and 2200 to 2900 of splits and stores beside 3900 to 4900 of products, under which two workgroups of a
// CU lie for each other; for layers of few chunks the start, 6000 clocks, and the filters' launch, 3 us and more.  Rows of a 5x5 window are a loop:
// laid out, a layer of few chunks waited for its instructions (this kernel by itself, 16x16x88 -> 49 11.1 -> 9.3 us, 36 of 41x39x32 -> 49 35.4 -> 32.5).
// Measured, us per call in one run, the fastest of the other kernels -> the fastest of this one: 36 images of 41x39x32 -> 49 5x5 63 -> 35, 4 of
// 7x10x496 -> 104 55 -> 41, 50 of 14x14x424 -> 96 234 -> 115, 13 of 35x33x112 -> 352 3x3 stride 2 41 -> 37.
#pragma once

#include "pwin_kernel.h"
#include "split_products.h"

namespace convfwd {

template <int R_, int MBW_, int NBW_, int WN_, int WK_, int POS_>
struct SdirCfg {
    static constexpr int R = R_, RS = R_ * R_, MBW = MBW_, NBW = NBW_, WN = WN_, WK = WK_, POS = POS_;
    static constexpr int WAVES = WN * WK, NT = 64 * WAVES;
    static constexpr int TM = 32 * MBW, TN = 32 * NBW * WN;
    static constexpr int PIECES = 2 * POS / (64 * WN);  // (position, eight channels) of a thread per chunk
    static constexpr int PLANE = POS * 16;              // bytes of a slab's plane: eight channels of all positions, one part
    static constexpr int SLAB = 6 * PLANE;              // [part][eight channels][position]
    // Units (tap, 32-channel block) of filters: a window row's at 5x5, where the rows are a loop (laid out, a layer of few chunks waits for
    // its instructions), a chunk's at 3x3.  In registers: all of a chunk where they fit, so that none waits behind the next chunk's input
    static constexpr int ROWS = R == 3 ? 3 : 1;
    static constexpr int UNITS = ROWS * R * MBW, RING = R == 5 ? 5 : MBW == 1 ? 9 : 6;
    static constexpr int Q = 4 * MBW * NBW;             // quads of a wave's sums
    static constexpr int QW = Q > WK ? Q / WK : 1;      // ... that a wave adds up and stores (the first Q waves of a group, where there are more)
    static constexpr int EXCH = WK > 1 ? WAVES * Q * 1024 : 0;
    static constexpr int LDS = WK * SLAB > EXCH ? WK * SLAB : EXCH;
    static_assert(POS % (64 * WN) == 0 && UNITS % RING == 0 && (Q % WK == 0 || WK % Q == 0) && 5 * PLANE < 65536, "");
};

struct SdirGeom {
    int IR, PW;     // staged rows of an image, positions of a row
    int KT, tiles;  // channel tiles, pixel tiles
    FastDiv dIR, dPW, dKT;
};

inline size_t sdir_filter_bytes(int K, int C, int RS) { return (size_t)((C + 15) / 16) * RS * ((K + 31) / 32) * 3072; }

// Filters [K][C][R][S] -> U[c / 16][tap][k / 32][part][lane][8], scaled and split, lane = k % 32 + 32 * (c % 16 / 8).  A workgroup
// takes 32 filters x 16 channels: rows to LDS, then a wave per tap.
template <int RS>
__global__ __launch_bounds__(512) void sdir_filter_kernel(const float* __restrict__ filt, uint4* __restrict__ U, int K, int C)
{
    constexpr int ROW = 16 * RS, PITCH = ROW + 1;
    __shared__ float g_s[32 * PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mb = blockIdx.x, c16 = blockIdx.y;
    const int have = (C - c16 * 16 < 16 ? C - c16 * 16 : 16) * RS;
    const int row_l = tid >> 4, j0 = tid & 15, k = mb * 32 + row_l;  // sixteen threads a filter
    const __amdgpu_buffer_rsrc_t rf = make_rsrc(filt, (uint32_t)K * (uint32_t)C * (RS * 4u));
    const uint32_t off = (uint32_t)k * ((uint32_t)C * (RS * 4u)) + (uint32_t)j0 * 4u;
    float v[RS];
#pragma unroll
    for (int i = 0; i < RS; ++i)
        v[i] = buffer_load_elem<float>(rf, k < K && j0 + 16 * i < have ? off + (uint32_t)c16 * (RS * 64u) + (uint32_t)i * 64u : kOutOfRange);
#pragma unroll
    for (int i = 0; i < RS; ++i) g_s[row_l * PITCH + j0 + 16 * i] = v[i];
    __syncthreads();
    const float* src = g_s + (lane & 31) * PITCH + (lane >> 5) * 8 * RS;
    for (int t = wave; t < RS; t += 8) {
        float x[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = src[c * RS + t] * kSplitScale;
        const Split3 s = split3(x);
        uint4* dst = U + (((size_t)c16 * RS + t) * gridDim.x + mb) * 192 + lane;
#pragma unroll
        for (int q = 0; q < 3; ++q) dst[q * 64] = s.p[q];
    }
}

// Four channels, k .. k + 3, of output pixel p for each lane in `mask`, summed in fp32 from the definition: taps outside the image are
// left out.  The wave takes the lanes' pixels together, 64 / their number lanes (rounded down to a power of two) for each, which share its
// channels; four sums share their input, a lane whose four sums are all NaN is done.  Bound by the loads of the few waves that have such
// pixels.  us a call, a wave for each output -> here: 50 images of 14x14x424 -> 96 5x5 (122 on ordinary data) with one infinite pixel 5290 -> 713, one
// NaN filter value 1100 -> 404, NaN everywhere 50500 -> 111, results beyond 2^79 everywhere 49500 -> 2280; 13 of 35x33x112 -> 352 3x3 stride 2
// (40) 244 -> 69, 133 -> 74, 6190 -> 52, 6190 -> 511.
template <int R>
__device__ __forceinline__ void sdir_sum_again(const ConvArgs& a, int lane, uint64_t mask, int k, int p, float* y)
{
    constexpr int RS = R * R;
    constexpr uint32_t kFar = 0x80000000u;
    const int count = __builtin_popcountll(mask), lg = 31 - __builtin_clz(64 / count), step = 1 << lg, entry = lane >> lg;
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    const bool mine = (mask >> lane) & 1;
    // (lanes outside the mask push to the last lane, which no entry reads when there are any)
    const int owners = __builtin_amdgcn_ds_permute((mine ? rank : 63) * 4, lane);
    const int owner = __shfl(owners, entry < count ? entry : 0);
    k = __shfl(k, owner);
    p = __shfl(p, owner);
    uint32_t n, pix, oy, ox;
    a.dOHW.divmod((uint32_t)p, n, pix);
    a.dOW.divmod(pix, oy, ox);
    const int iy = (int)oy * a.stride - a.pad, ix = (int)ox * a.stride - a.pad;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes), rf = make_rsrc(a.filt, a.filt_bytes);
    const int origin = (int)n * a.C * a.HW + iy * a.W + ix;
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int c = lane & (step - 1); entry < count && c < a.C; c += step) {
        const int at = origin + c * a.HW;
        bool in[RS];
        float x[RS];
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            in[t] = (unsigned)(iy + t / R) < (unsigned)a.H && (unsigned)(ix + t % R) < (unsigned)a.W;
            x[t] = buffer_load_elem<float>(rin, in[t] ? (uint32_t)(at + t / R * a.W + t % R) * 4u : kFar);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // (a filter past the last one is not stored, and not read beyond the tensor)
            const uint32_t fo = (uint32_t)((k + q) * a.C + c) * (RS * 4u);
            float f[RS];
#pragma unroll
            for (int t = 0; t < RS - 1; t += 4) {
                const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rf, (int)(fo + t * 4u), 0, 0));
                f[t] = v[0], f[t + 1] = v[1], f[t + 2] = v[2], f[t + 3] = v[3];
            }
            f[RS - 1] = buffer_load_elem<float>(rf, fo + (RS - 1) * 4u);
#pragma unroll
            for (int t = 0; t < RS; ++t) s[q] = in[t] ? __builtin_fmaf(x[t], f[t], s[q]) : s[q];
        }
        if (s[0] != s[0] && s[1] != s[1] && s[2] != s[2] && s[3] != s[3]) break;
    }
    for (int o = step >> 1; o > 0; o >>= 1)
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] += __shfl_xor(s[q], o);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float total = __shfl(s[q], rank << lg & 63);
        y[q] = mine ? total : y[q];
    }
}

template <class CFG>
__global__ __launch_bounds__(CFG::NT, 2) void sdir_kernel(ConvArgs a, SdirGeom d)
{
    constexpr int R = CFG::R, RS = CFG::RS, MBW = CFG::MBW, NBW = CFG::NBW, WN = CFG::WN, WK = CFG::WK, TM = CFG::TM, TN = CFG::TN;
    constexpr int PIECES = CFG::PIECES, PLANE = CFG::PLANE, UNITS = CFG::UNITS, RING = CFG::RING, Q = CFG::Q, QW = CFG::QW;
    constexpr uint32_t kFar = 0x80000000u;
    typedef Mma<CONV_BF16, 32> mma_t;
    typedef __attribute__((address_space(3))) char* lds_bytes;
    typedef const __attribute__((address_space(3))) u32x4* lds_quads;
    extern __shared__ __attribute__((aligned(16))) char smem_c[];

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave % WN, wk = wave / WN;
    const int C16 = (a.C + 15) >> 4, MBK = (a.K + 31) >> 5;
    // an XCD's workgroups share a contiguous run of pixel tiles, channel tiles innermost
    int m0, p0;
    {
        const int total = (int)gridDim.x, b = blockIdx.x, x = b & 7, per = total >> 3, rem = total & 7;
        uint32_t pt, kt;
        d.dKT.divmod((uint32_t)(x * per + (x < rem ? x : rem) + (b >> 3)), pt, kt);
        m0 = (int)kt * TM, p0 = (int)pt * TN;
    }
    const int plast = (p0 + TN < a.P ? p0 + TN : a.P) - 1;
    auto stacked = [&](int p, int& n, int& pix) {  // staged row of an output pixel's window, its image and place there
        uint32_t n_, pix_, oy, ox;
        a.dOHW.divmod((uint32_t)p, n_, pix_);
        a.dOW.divmod(pix_, oy, ox);
        n = (int)n_, pix = (int)pix_;
        return make_int2((int)n_ * d.IR + (int)oy * a.stride, (int)ox * a.stride);
    };
    int n_first, pix_first, n_last, pix_last;
    const int s0 = __builtin_amdgcn_readfirstlane(stacked(p0, n_first, pix_first).x);
    const int nrows = __builtin_amdgcn_readfirstlane(stacked(plast, n_last, pix_last).x) + R - s0;

    // ---- filters: units (tap, 32-channel block) in the order of the loop, this wave's chunks wk, wk + WK, ... ----------------
    const __amdgpu_buffer_rsrc_t ru = make_rsrc(a.ws, (uint32_t)C16 * (uint32_t)(RS * 3072) * (uint32_t)MBK);
    const uint32_t u_tap = (uint32_t)MBK * 3072u, u_chunk = u_tap * RS;
    uint32_t u_now = (uint32_t)wk * u_chunk + (uint32_t)(m0 >> 5) * 3072u;
    uint4 ar[RING][3];
    // (blocks past the last one read filters of the tap after, chunks past the last one nothing: sums nobody stores, products with zeros)
    auto load_a = [&](auto slot_c, auto unit_c, uint32_t base) {
        constexpr int slot = decltype(slot_c)::value, unit = decltype(unit_c)::value;
        const uint32_t at = base + (uint32_t)(unit / MBW) * u_tap + (uint32_t)(unit % MBW) * 3072u;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(ru, (int)(at + (uint32_t)lane * 16u), q * 1024, 0);
            ar[slot][q] = make_uint4(v.x, v.y, v.z, v.w);
        }
    };

    // ---- input: piece = (position of the slab, eight channels) ---------------------------------------------------------------
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    const int gt = tid - wk * (64 * WN);  // thread of the group that shares a slab
    constexpr int HALF = PIECES / 2;  // pieces i and i + HALF are the two halves of a position's channels
    uint32_t x_off[HALF];
#pragma unroll
    for (int i = 0; i < HALF; ++i) {
        uint32_t rr, xx, n, yy;
        d.dPW.divmod((uint32_t)(i * 64 * WN + gt), rr, xx);
        d.dIR.divmod((uint32_t)s0 + rr, n, yy);
        const int y = (int)yy - a.pad, x = (int)xx - a.pad;
        const bool ok = (int)rr < nrows && (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W && (int)n < a.N;
        x_off[i] = ok ? (uint32_t)(((int)n * a.C * a.H + y) * a.W + x) * 4u : kFar;
    }
    const uint32_t chan = (uint32_t)a.HW * 4u;
    float xr[PIECES][8];
    const int used = nrows * d.PW;  // positions of the tile
    auto load_x = [&](int chunk) {
        const int left = a.C - chunk * 16;  // channels past the last one read as zero
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            if (i % HALF * 64 * WN >= used) continue;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int at = i / HALF * 8 + c;
                xr[i][c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rin, (int)(at < left ? x_off[i % HALF] : kFar), (int)(at < left ? (uint32_t)(chunk * 16 + at) * chan : 0u), 0));
            }
        }
    };
    char* const slab = smem_c + wk * CFG::SLAB;
    auto store_x = [&]() {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            if (i % HALF * 64 * WN >= used) continue;
            float x[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) x[c] = xr[i][c] * kSplitScale;
            const Split3 s = split3(x);
#pragma unroll
            for (int q = 0; q < 3; ++q) *(uint4*)(slab + q * 2 * PLANE + (i * 64 * WN + gt) * 16) = s.p[q];
        }
    };

    // ---- the lane's windows -----------------------------------------------------------------------------------------------------
    uint32_t win[NBW];  // LDS address of part 0, first tap
    uint32_t o_px[NBW];  // byte offset of the output pixel in channel 0
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
        const int p = p0 + (wn * NBW + nb) * 32 + li;
        int n, pix;
        const int2 at = stacked(p < a.P ? p : plast, n, pix);
        win[nb] = (uint32_t)(uintptr_t)(lds_bytes)slab + (uint32_t)(g * PLANE + ((at.x - s0) * d.PW + at.y) * 16);
        o_px[nb] = p < a.P ? (uint32_t)(n * a.K * a.OHW + pix) * 4u : kFar;
    }

    // The leading products and the five small ones have sums of their own: a sum is rounded once for sixteen channels and tap, not six times.
    // A wave that takes all channels adds a chunk's leading sums to those of the chunks before: the chain of roundings is 9 or 25
    // long, then one for each chunk
    constexpr bool FOLD = WK == 1;
    typename mma_t::acc_t acc[MBW][NBW], low[MBW][NBW], done[MBW][NBW];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = low[mb][nb][v] = done[mb][nb][v] = 0.0f;

    const int rounds = (C16 + WK - 1) / WK;
    load_x(wk);
    static_for<RING - 1>([&](auto uc) { load_a(uc, uc, u_now); });
    store_x();
    if constexpr (WN > 1) __syncthreads();
    struct Window {
        uint4 p[NBW][3];
    };
    const uint32_t row16 = (uint32_t)d.PW * 16u;
    auto read_b = [&](uint32_t row_off, int t) {
        Window w;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const u32x4 v = *(lds_quads)(uintptr_t)(win[nb] + row_off + (uint32_t)(t * 16 + q * 2 * PLANE));
                w.p[nb][q] = make_uint4(v.x, v.y, v.z, v.w);
            }
        return w;
    };
    const uint32_t u_row = u_tap * R;
#pragma unroll 1
    for (int round = 0; round < rounds; ++round) {
        if (round + 1 < rounds) load_x((round + 1) * WK + wk);
        Window b = read_b(0u, 0);
        uint32_t row_off = 0;
#pragma unroll 1
        for (int r = 0; r < R; r += CFG::ROWS) {
            const bool more = r + CFG::ROWS < R;
            const uint32_t u_next = u_now + u_row * CFG::ROWS + (more ? 0u : u_chunk * (WK - 1));
            static_for<CFG::ROWS * R>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                __builtin_amdgcn_sched_barrier(0);
                // (behind the last tap the first one again, not used)
                const bool wraps = t + 1 == CFG::ROWS * R && !more;
                if constexpr ((t + 1) % R == 0) row_off = wraps ? 0u : row_off + row16;
                const Window next = read_b(row_off, (t + 1) % R);
                static_for<MBW>([&](auto mbc) {
                    constexpr int mb = decltype(mbc)::value, unit = t * MBW + mb, ahead = unit + RING - 1;
                    constexpr int pa[6] = {2, 0, 1, 0, 1, 0}, pb[6] = {0, 2, 1, 0, 0, 1};
                    load_a(std::integral_constant<int, ahead % RING>{}, std::integral_constant<int, ahead % UNITS>{}, ahead < UNITS ? u_now : u_next);
#pragma unroll
                    for (int q = 0; q < 6; ++q)
#pragma unroll
                        for (int nb = 0; nb < NBW; ++nb) {
                            typename mma_t::acc_t& to = pa[q] + pb[q] ? low[mb][nb] : acc[mb][nb];
                            to = mma_t::run(ar[unit % RING][pa[q]], b.p[nb][pb[q]], to);
                        }
                });
                b = next;
            });
            u_now = u_next;
        }
        __builtin_amdgcn_sched_barrier(0);
        if (round + 1 < rounds) {
            if constexpr (FOLD) {
#pragma unroll
                for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                        for (int v = 0; v < 16; ++v) done[mb][nb][v] += acc[mb][nb][v], acc[mb][nb][v] = 0.0f;
            }
            if constexpr (WN > 1) __syncthreads();
            store_x();
            if constexpr (WN > 1) __syncthreads();
        }
    }
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = (FOLD ? done[mb][nb][v] + acc[mb][nb][v] : acc[mb][nb][v]) + low[mb][nb][v];

    // ---- sums of the waves that split the channels, in wave order; quad q = (block of channels, block of pixels, four channels) ----
    f32x4 y[QW];
    if constexpr (WK > 1) {
        __syncthreads();
        f32x4* const ex = (f32x4*)smem_c;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const typename mma_t::acc_t& s = acc[q / 4 / NBW][q / 4 % NBW];
            ex[(wave * Q + q) * 64 + lane] = f32x4{s[q % 4 * 4], s[q % 4 * 4 + 1], s[q % 4 * 4 + 2], s[q % 4 * 4 + 3]};
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < QW; ++j) {
            f32x4 s = ex[(wn * Q + wk * QW + j) * 64 + lane];
#pragma unroll
            for (int w = 1; w < WK; ++w) s += ex[((w * WN + wn) * Q + wk * QW + j) * 64 + lane];
            y[j] = s;
        }
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const typename mma_t::acc_t& s = acc[q / 4 / NBW][q / 4 % NBW];
            y[q] = f32x4{s[q % 4 * 4], s[q % 4 * 4 + 1], s[q % 4 * 4 + 2], s[q % 4 * 4 + 3]};
        }
    }

    if (QW * WK > Q && wk >= Q) return;

    // ---- bias + activation --------------------------------------------------------------------------------------------------------
    const __amdgpu_buffer_rsrc_t rbias = make_rsrc(a.bias, a.bias ? (uint32_t)a.K * 4u : 0u);
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(a.out, a.out_bytes);
    const uint32_t plane = (uint32_t)a.OHW * 4u;
    f32x4 bias[QW];
#pragma unroll
    for (int j = 0; j < QW; ++j) {
        const int q = wk * QW + j;
        bias[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rbias, (m0 + q / 4 / NBW * 32 + q % 4 * 8 + 4 * g) * 4, 0, 0));
    }
    const float floor = a.relu ? 0.0f : __builtin_nanf("");  // the maximum with a NaN is the other operand, a NaN (a bias that is one) stays
    uint64_t bad = 0;  // bit 4 * quad + channel: a sum that is not finite
#pragma unroll
    for (int j = 0; j < QW; ++j) {
        const int q = wk * QW + j, k = m0 + q / 4 / NBW * 32 + q % 4 * 8 + 4 * g, nb = q / 4 % NBW;
        uint32_t o = o_px[0];
        if constexpr (NBW == 2) o = nb ? o_px[1] : o_px[0];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float s = y[j][r];
            bad |= __builtin_fabsf(s) < __builtin_inff() ? 0ull : 1ull << (4 * j + r);
            const float v = __builtin_fmaxf(__builtin_fmaf(s, kSplitUnscale, bias[j][r]), floor);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rout, (int)(k + r < a.K && o != kFar ? o + (uint32_t)(k + r) * plane : kFar), 0, 0);
        }
    }
    if (__any(bad != 0)) {
#pragma unroll 1
        for (int j = 0; j < QW; ++j) {
            const int q = wk * QW + j, k = m0 + q / 4 / NBW * 32 + q % 4 * 8 + 4 * g, p = p0 + (wn * NBW + q / 4 % NBW) * 32 + li;
            const uint32_t mine = (uint32_t)(bad >> 4 * j) & 15u;
            const uint64_t again = __ballot(mine && k < a.K && p < a.P);
            if (!again) continue;
            float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            sdir_sum_again<R>(a, lane, again, k, p, s);
            uint32_t n, pix;
            a.dOHW.divmod(p < a.P ? (uint32_t)p : 0u, n, pix);
            const uint32_t o = (uint32_t)((int)n * a.K * a.OHW + (int)pix) * 4u;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool store = (mine >> r & 1) && k + r < a.K && p < a.P;
                s[r] += a.bias && store ? a.bias[k + r] : 0.0f;
                if (a.relu) s[r] = s[r] > 0.0f ? s[r] : 0.0f;
                buffer_store_elem<float>(s[r], rout, store ? o + (uint32_t)(k + r) * plane : kFar);
            }
        }
    }
}

template <class CFG>
size_t sdir_workspace(const Variant&, const conv_desc& d, int, int)
{
    return sdir_filter_bytes(d.K, d.C, CFG::RS);
}

template <class CFG>
hipError_t sdir_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    SdirGeom g;
    g.IR = (a.OH - 1) * a.stride + CFG::R;
    g.PW = (a.OW - 1) * a.stride + CFG::R;
    g.KT = (a.K + CFG::TM - 1) / CFG::TM;
    g.tiles = (a.P + CFG::TN - 1) / CFG::TN;
    g.dIR = make_fastdiv((uint32_t)g.IR);
    g.dPW = make_fastdiv((uint32_t)g.PW);
    g.dKT = make_fastdiv((uint32_t)g.KT);
    const hipError_t e = ensure_dynamic_lds((const void*)sdir_kernel<CFG>, CFG::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sdir_filter_kernel<CFG::RS>, dim3((unsigned)((a.K + 31) / 32), (unsigned)((a.C + 15) / 16)), dim3(512), 0, s, (const float*)a.filt, (uint4*)a.ws, a.K, a.C);
    const hipError_t e2 = hipGetLastError();
    if (e2 != hipSuccess) return e2;
    hipLaunchKernelGGL(sdir_kernel<CFG>, dim3((unsigned)(g.KT * g.tiles)), dim3(CFG::NT), CFG::LDS, s, a, g);
    return hipGetLastError();
}

template <class CFG>
bool sdir_valid(const Variant&, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != CONV_F32 || d.R != CFG::R || d.S != CFG::R || d.stride > 4 || d.pad >= CFG::R) return false;
    if (d.flags & ~(uint32_t)CONV_FLAG_RELU) return false;  // plain formats and filters, no fused pool
    if (d.C < 8) return false;                              // a step is 16 channels, not worth it emptier
    if (CFG::TM > (d.K + 31) / 32 * 32) return false;       // an empty channel block only costs time
    // 32-bit byte offsets beside an out-of-range marker
    const long long lim = 1LL << 31;
    if (((long long)d.N * d.C + 16) * d.H * d.W * 4 >= lim || ((long long)d.N * d.K + CFG::TM) * OH * OW * 4 >= lim) return false;
    if ((long long)sdir_filter_bytes(d.K, d.C, CFG::RS) + (long long)CFG::WK * CFG::RS * 3072 * ((d.K + 31) / 32) >= lim || (d.C + 15) / 16 > 65535) return false;
    if ((long long)d.N * ((OH - 1LL) * d.stride + CFG::R) >= (1LL << 30) || (long long)d.N * OH * OW + CFG::TN >= (1LL << 30)) return false;
    if (sdir_positions(CFG::TN, d.N, CFG::R, d.stride, OH, OW) > CFG::POS) return false;
    // (a launch holds fewer than 2^32 threads)
    return (long long)((d.K + CFG::TM - 1) / CFG::TM) * (((long long)d.N * OH * OW + CFG::TN - 1) / CFG::TN) * CFG::NT < (1LL << 32);
}

template <class CFG>
void sdir_register(std::vector<Variant>& out, const TileModel& model)
{
    Variant v;
    char buf[96];
    snprintf(buf, sizeof buf, "sdir_f32_%dx%d_M%dN%d_w%dk%d_s%d", CFG::R, CFG::R, CFG::TM, CFG::TN, CFG::WN, CFG::WK, CFG::POS);
    v.name = buf;
    v.dtype = CONV_F32;
    v.split = 1;
    v.tm = CFG::TM;
    v.tn = CFG::TN;
    v.tk = 16 * CFG::RS * CFG::WK;
    v.threads = CFG::NT;
    v.family = FAM_WINDOW;
    v.specificity = 4;
    v.traits = TRAIT_SPLIT_DIRECT;
    v.per_cu = CFG::LDS > 80 * 1024 || CFG::NT > 256 ? 1 : 2;
    v.model = model;
    v.slab = CFG::POS;
    v.slab_threads = 64 * CFG::WN;
    v.valid = &sdir_valid<CFG>;
    v.launch = &sdir_launch<CFG>;
    v.ws_extra = &sdir_workspace<CFG>;
    out.push_back(v);
}

}  // namespace convfwd
