// First layers (3 channels, 11x11 stride 4 or 7x7 stride 2) in fp32 with their products on the 16-bit matrix units.
//
// The gather kernels reach 0.67 of the fp32 matrix rate on these layers.  Here every fp32 operand is split into three bf16
// numbers and a product is the sum of six partial products, as in winos_kernel.h (what is left out is below 2^-24 of the
// product, and sixteen reduction elements enter the accumulator with one rounding); operands are scaled by 2^24 ahead of the
// splits, so that every part of every fp32 number is a normal bf16 number or zero.  What remains is at the upper end (operands
// above 2^103, sums above 2^79) and shows as a result that is not finite: those are summed again in fp32 from the definition.
//   * The reduction is that of swin16_kernel.h: lines (filter row, channel) of SQ groups of 4 taps; a lane's 8 elements of an
//     MFMA are two groups, 16 consecutive bytes each of a staged input row at stride 4.
//   * A workgroup is 256 consecutive pixels of one image and 32*TMB channels, a wave 64 pixels: the input rows are staged once,
//     scaled, in fp32 (three bf16 copies would not fit LDS), and split by the wave that multiplies with them: 88 vector
//     instructions a step beneath 12*TMB MFMAs.
//   * Filters are split by a small kernel ahead into the workspace, in MFMA operand order ([step][32-channel block][part][lane]
//     [8], 1 KB each), and come from L2 straight into registers; the four waves of a workgroup share them in L1.
// What bounds it: 20 images of 227x227 -> 96 are one round of 240 workgroups of 49000 clocks, 34800 of them the loop (936 MFMAs
// at 37 clocks, 32 at best), 8000 staging and 5500 stores that nothing covers with one workgroup per CU; 2.2 of 32.1 us are the filters'
// launch (29.9 with the filters split beforehand).  Measured, us per call, best of the other kernels -> this one: 20 of 227x227 -> 96, 11x11 40 -> 32; 20 of 223x223 -> 64, 7x7
// stride 2, 61 -> 38, 49 of 228x228 146 -> 81.  Where it begins (96 filters of 11x11, images of 227x227; best of the others -> this one): 2 images,
// 24 tiles of 256 pixels, 14.8 -> 17.8, 3 17.8 -> 17.8, 5 19.3 -> 18.3, 6 23.9 -> 18.6, 10 30.0 -> 26.3, 12 38.7 -> 27.2; 64 filters
// of 7x7, images of 224x224: 1 image, 49 tiles, 9.6 -> 11.7, 2 12.4 -> 12.2, 4 19.0 -> 15.1.  The selection takes it from there.
// Error against 64 bits (2-norm, relative), gather kernels 3.4e-7, this one 3.0e-7 (11x11) and 1.9e-7 (7x7).
#pragma once

#include "pwin_kernel.h"
#include "split_products.h"

namespace convfwd {

template <int S_, int ST_, int TMB_>
struct SwinsCfg {
    static constexpr int C = 3, R = S_, S = S_, ST = ST_, TMB = TMB_;
    static constexpr int NT = 256, NBW = 2;
    static constexpr int TM = 32 * TMB, TN = 64 * 4;
    static constexpr int SQ = (S + 3) / 4, NROW = C * R;
    static constexpr int KSTEPS = ((NROW + 1) / 2 * SQ + 1) / 2;
    // steps after which the taps repeat, a fixed number of lines further down, and such periods whose lines all exist
    static constexpr int PER = SQ % 2 == 0 ? SQ / 2 : SQ, LPP = 2 * (2 * PER / SQ);
    static constexpr int FULL = NROW / LPP;
    static_assert(PER * 2 % SQ == 0 && KSTEPS - FULL * PER >= 0, "periods");
};

struct SwinsGeom {
    int tpi;    // tiles of an image
    int rows;   // most input rows of a tile
    int pitch;  // floats of a staged row
    int W4;     // 4-column pieces of a row
    FastDiv dT;
};

inline SwinsGeom swins_geom(int TN, int R, int ST, int W, int pad, int OH, int OW)
{
    SwinsGeom g;
    g.tpi = (OH * OW + TN - 1) / TN;
    int span = (TN - 1 + OW - 1) / OW + 1;
    if (span > OH) span = OH;
    g.rows = (span - 1) * ST + R;
    g.pitch = (W + 2 * pad + 3) / 4 * 4 + 4;
    g.W4 = (W + 3) / 4;
    return g;
}

// filters [K][3][R][S] -> U[step][block][part][lane][8], scaled and split: a wave per block of filters (x) and step (y).
// One chain of latencies: the eight loads of a lane are requested together (as conditional loads in twenty workgroups of 256 threads
// they were waited for one by one; call of 20 images of 227x227 -> 96 34.2 -> 32.1 us, 29.9 without this launch.  Traced launches hide it:
// none takes less than 4.8 us under the profiler).
template <class CFG>
__global__ __launch_bounds__(64) void swins_filter_kernel(const float* __restrict__ filt, uint4* __restrict__ U, int K)
{
    const int lane = threadIdx.x, b = blockIdx.x, j = blockIdx.y, blocks = gridDim.x;
    const int k = b * 32 + (lane & 31), h = lane >> 5;
    constexpr uint32_t row = CFG::C * CFG::R * CFG::S * 4;
    const __amdgpu_buffer_rsrc_t rf = make_rsrc(filt, (uint32_t)K * row);
    float x[8];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int i2 = 2 * j + g, t = i2 / CFG::SQ, sq = i2 - t * CFG::SQ, line = 2 * t + h, r = line / CFG::C, c = line - r * CFG::C;
        const uint32_t off = (uint32_t)k * row + (uint32_t)((c * CFG::R + r) * CFG::S + 4 * sq) * 4u;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            x[4 * g + e] = buffer_load_elem<float>(rf, k < K && line < CFG::NROW && 4 * sq + e < CFG::S ? off + e * 4u : kOutOfRange);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] *= kSplitScale;
    const Split3 s = split3(x);
    uint4* dst = U + ((size_t)(j * blocks + b) * 3) * 64 + lane;
#pragma unroll
    for (int q = 0; q < 3; ++q) dst[q * 64] = s.p[q];
}

// a.ws holds U
template <class CFG>
__global__ __launch_bounds__(CFG::NT, 1) void swins_kernel(ConvArgs a, SwinsGeom d)
{
    constexpr int C = CFG::C, R = CFG::R, S = CFG::S, ST = CFG::ST, TMB = CFG::TMB, NBW = CFG::NBW, NT = CFG::NT, TM = CFG::TM, TN = CFG::TN;
    constexpr int SQ = CFG::SQ, KSTEPS = CFG::KSTEPS, PER = CFG::PER, FULL = CFG::FULL;
    typedef Mma<CONV_BF16, 32> mma_t;
    extern __shared__ __attribute__((aligned(16))) float rows_s[];  // [input row][channel][pitch]

    // the arguments are fetched together here: left to their first uses, each line of them is waited for by itself
    asm volatile("" ::"s"(a.in), "s"(a.ws), "s"(a.bias), "s"(a.out), "s"(a.H), "s"(a.W), "s"(a.K), "s"(a.pad), "s"(a.HW), "s"(a.OHW), "s"(a.relu),
                 "s"(a.in_bytes), "s"(a.out_bytes), "s"(a.dOW.mul), "s"(a.dOW.shift), "s"(a.dOW.d), "s"(d.pitch), "s"(d.W4), "s"(d.dT.mul), "s"(d.dT.d));
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // ids b, b+8, ... run on one XCD: give each XCD a contiguous run of tiles, whose input rows overlap
    uint32_t img, tile;
    {
        const int T = (int)gridDim.x, b = blockIdx.x, x = b & 7, per = T >> 3, rem = T & 7;
        d.dT.divmod((uint32_t)(x * per + (x < rem ? x : rem) + (b >> 3)), img, tile);
    }
    const int m0 = (int)blockIdx.y * TM, p0 = (int)tile * TN, blocks = (a.K + 31) >> 5;

    // ---- filters: parts of one step and its TMB blocks, a step ahead -----------------------------------------------------
    const __amdgpu_buffer_rsrc_t ru = make_rsrc(a.ws, (uint32_t)KSTEPS * (uint32_t)blocks * 3072u);
    const uint32_t u_step = (uint32_t)blocks * 3072u, u_base = (uint32_t)(m0 >> 5) * 3072u;
    uint4 af[2][TMB][3];
    auto load_a = [&](int set, uint32_t step) {  // (blocks past the last one read filters of the step after, or nothing: sums nobody stores)
#pragma unroll
        for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(ru, lane * 16, (int)(u_base + step * u_step + (uint32_t)(mb * 3 + q) * 1024u), 0);
                af[set][mb][q] = make_uint4(v.x, v.y, v.z, v.w);
            }
    };

    // ---- input rows: whole rows of the image, 16 bytes a lane, the last piece of a row ending with it ----------------------
    const int plast = (p0 + TN < a.OHW ? p0 + TN : a.OHW) - 1;
    const int oy0 = (int)a.dOW.div((uint32_t)p0), nrows = ((int)a.dOW.div((uint32_t)plast) - oy0) * ST + R;
    const int iy0 = oy0 * ST - a.pad;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    // A wave takes every fourth row, a lane four columns of it: row addresses are scalars.  A short loop with a batch of rows
    // on the way: laid out in full (24 rows) it was 7200 clocks of instruction fetches.
    const int lines = nrows * C;
    constexpr int BATCH = 6;
    const uint32_t img_off = (uint32_t)img * (uint32_t)(C * a.HW);
    load_a(0, 0);
#pragma unroll 1
    for (int k0 = 0; k0 < d.W4; k0 += 64) {
        const int x = (k0 + lane) * 4 < a.W - 4 ? (k0 + lane) * 4 : a.W - 4;  // (lanes past the row's end repeat its last piece)
        const bool whole = ((x + a.pad) & 3) == 0;
        f32x4 v[2][BATCH];
        auto load_rows = [&](int set, int l0) {
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int l = l0 + 4 * i, rr = l / C, c = l - rr * C, iy = iy0 + rr;
                const uint32_t soff = l < lines && (unsigned)iy < (unsigned)a.H ? (img_off + (uint32_t)(c * a.HW + iy * a.W)) * 4u : 0x80000000u;
                v[set][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rin, x * 4, (int)soff, 0));
            }
        };
        auto store_rows = [&](int set, int l0) {
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int l = l0 + 4 * i;
                float* const dst = rows_s + (l < lines ? l : lines + 3) * d.pitch + x + a.pad;  // (rows past the tile's: the spare line)
                const f32x4 w = v[set][i] * kSplitScale;
                if (whole) {
                    *(f32x4*)dst = w;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) dst[j] = w[j];
                }
            }
        };
        load_rows(0, wave);
        load_rows(1, wave + 4 * BATCH);
#pragma unroll 1
        for (int l0 = wave; l0 < lines; l0 += 8 * BATCH) {
            store_rows(0, l0);
            load_rows(0, l0 + 8 * BATCH);
            store_rows(1, l0 + 4 * BATCH);
            load_rows(1, l0 + 12 * BATCH);
        }
    }
    if (a.pad) {  // columns beside the image
        const int side = d.pitch - a.W;
        for (int u = tid; u < lines * side; u += NT) {
            const int rc = u / side, xs = u - rc * side;
            rows_s[rc * d.pitch + (xs < a.pad ? xs : xs + a.W)] = 0.0f;
        }
    }

    typename mma_t::acc_t acc[TMB][NBW];
#pragma unroll
    for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.0f;

    // the lane's windows: line h of its pixels (h = 1 reads the second line of a pair)
    const float* win[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
        const int p = p0 + wave * 64 + nb * 32 + li;
        uint32_t oy, ox;
        a.dOW.divmod((uint32_t)(p < a.OHW ? p : plast), oy, ox);
        win[nb] = rows_s + (((int)oy - oy0) * ST * C + h) * d.pitch + (int)ox * ST;
    }
    __syncthreads();

    // operands of a step: raw[nb][8] of the step after, parts bf of this one
    float raw[NBW][8];
    Split3 bf[2][NBW];
    auto read_x = [&](auto j_c) {  // j: step within its period
        constexpr int j = decltype(j_c)::value;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int i2 = 2 * j + g, t = i2 / SQ, sq = i2 % SQ;
                const float* src = win[nb] + 2 * t * d.pitch + 4 * sq;
                float v[4];
                if constexpr (ST % 4 == 0) {
                    const f32x4 w = *(const f32x4*)src;
                    v[0] = w[0], v[1] = w[1], v[2] = w[2], v[3] = w[3];
                } else {
                    const float2 w0 = *(const float2*)src, w1 = *(const float2*)(src + 2);
                    v[0] = w0.x, v[1] = w0.y, v[2] = w1.x, v[3] = w1.y;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[nb][4 * g + e] = v[e];
            }
    };
    // what no tap of the window reads must not meet the zeros of the filters, for it may be infinite
    auto split_x = [&](auto j_c, auto last_c, int set) {
        constexpr int j = decltype(j_c)::value;
        constexpr bool LAST = decltype(last_c)::value;  // steps behind the full periods
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            float x[8];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int i2 = 2 * j + g, t = i2 / SQ, sq = i2 % SQ;
                const int line = LAST ? FULL * CFG::LPP + 2 * t : 0;  // line of the lower half, the upper half's follows
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool tap = 4 * sq + e < S && line < CFG::NROW;
                    x[4 * g + e] = !tap ? 0.0f : LAST && line + 1 >= CFG::NROW ? (h ? 0.0f : raw[nb][4 * g + e]) : raw[nb][4 * g + e];
                }
            }
            bf[set][nb] = split3(x);
        }
    };
    auto products = [&](int set) {
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};  // the smallest first
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) acc[mb][nb] = mma_t::run(af[set][mb][pa[q]], bf[set][nb].p[pb[q]], acc[mb][nb]);
    };
    // One step: its products, with the next step's filters on the way, the next step's input split and the one after read.
    // Asked for instruction by instruction, for the compiler puts the vector work ahead of the MFMAs it could hide under.
    auto mix = [&]() {
#pragma unroll
        for (int i = 0; i < 6 * TMB * NBW; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            if (i < 3 * TMB) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // filter load
            if (i < 4 * NBW) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
            __builtin_amdgcn_sched_group_barrier(0x002, 112 / (6 * TMB * NBW) + 1, 0);  // vector work
        }
    };
    constexpr std::false_type in_full{};
    constexpr std::true_type in_last{};
    // step s of a period (the next one's first step follows the last): F: this period is full; N: the next step is in a full one
    uint32_t step = 0;
    auto advance = [&](int periods) {
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) win[nb] += periods * CFG::LPP * d.pitch;
    };
    constexpr int TAIL = KSTEPS - FULL * PER;
    static_assert(TAIL >= 1 && FULL >= 2, "shape of the loop");
    // prologue: step 0 split, step 1 read
    read_x(std::integral_constant<int, 0>{});
    split_x(std::integral_constant<int, 0>{}, in_full, 0);
    int period = 0;
    // sets alternate from step to step; an odd period is unrolled twice
    constexpr int UNR = PER % 2 ? 2 : 1;
    auto full_period = [&](auto par_c, auto next_c) {  // next_c: is the period after this one full?
        constexpr int par = decltype(par_c)::value;
        static_for<PER>([&](auto sc) {
            constexpr int s = decltype(sc)::value, set = (par + s) & 1;
            __builtin_amdgcn_sched_barrier(0);
            load_a(set ^ 1, step + 1);
            if constexpr (s + 1 < PER) {
                read_x(std::integral_constant<int, s + 1>{});
                products(set);
                split_x(std::integral_constant<int, s + 1>{}, in_full, set ^ 1);
            } else {
                advance(1);
                read_x(std::integral_constant<int, 0>{});
                products(set);
                split_x(std::integral_constant<int, 0>{}, next_c, set ^ 1);
            }
            mix();
            ++step;
        });
    };
    static_assert(FULL % UNR == 0, "whole rounds of the loop");
    for (; period + UNR < FULL; period += UNR) {
        full_period(std::integral_constant<int, 0>{}, in_full);
        if constexpr (UNR == 2) full_period(std::integral_constant<int, PER & 1>{}, in_full);
    }
    if constexpr (UNR == 2) {
        full_period(std::integral_constant<int, 0>{}, in_full);
        full_period(std::integral_constant<int, PER & 1>{}, in_last);
    } else {
        full_period(std::integral_constant<int, 0>{}, in_last);
    }
    static_for<TAIL>([&](auto sc) {
        constexpr int s = decltype(sc)::value, set = (FULL * PER + s) & 1;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (s + 1 < TAIL) {
            load_a(set ^ 1, step + 1);
            read_x(std::integral_constant<int, s + 1>{});
        }
        products(set);
        if constexpr (s + 1 < TAIL) split_x(std::integral_constant<int, s + 1>{}, in_last, set ^ 1);
        ++step;
    });
    __builtin_amdgcn_sched_barrier(0);

    // ---- bias + activation; a lane holds channels 8i + 4h .. +3 of a block at one pixel: runs of 128 bytes per channel -------
    const __amdgpu_buffer_rsrc_t rbias = make_rsrc(a.bias, a.bias ? (uint32_t)a.K * 4u : 0u);
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(a.out, a.out_bytes);
    const uint32_t plane = (uint32_t)a.OHW * 4u;
    float finite = 0.0f;  // NaN where a sum is not finite
    uint32_t o[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
        const int p = p0 + wave * 64 + nb * 32 + li;
        o[nb] = p < a.OHW ? (uint32_t)p * 4u + (uint32_t)(4 * h) * plane : 0x80000000u;  // (tensors stay below 2 GiB)
    }
    // (all ahead of the stores: a load behind them would be waited for until they are done)
    f32x4 bs[TMB][4];
#pragma unroll
    for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            bs[mb][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rbias, (m0 + mb * 32 + 8 * i + 4 * h) * 4, 0, 0));
    const uint32_t o_tile = (img * (uint32_t)a.K + (uint32_t)m0) * plane;
    auto store = [&](auto relu_c, auto whole_c) {  // whole: all the tile's channels exist
#pragma unroll
        for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = mb * 32 + 8 * i;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) {
                        const float v = acc[mb][nb][4 * i + r];
                        finite = __builtin_fmaf(v, 0.0f, finite);
                        float y = __builtin_fmaf(v, kSplitUnscale, bs[mb][i][r]);
                        if constexpr (decltype(relu_c)::value) y = y > 0.0f ? y : 0.0f;
                        const uint32_t at = decltype(whole_c)::value || m0 + row + 4 * h + r < a.K ? o[nb] : 0x80000000u;
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, y), rout, (int)at, (int)(o_tile + (uint32_t)(row + r) * plane), 0);
                    }
            }
    };
    const bool whole = m0 + TM <= a.K;
    if (a.relu && whole)
        store(std::true_type{}, std::true_type{});
    else if (a.relu)
        store(std::true_type{}, std::false_type{});
    else if (whole)
        store(std::false_type{}, std::true_type{});
    else
        store(std::false_type{}, std::false_type{});
    if (__any(finite != 0.0f)) {
        // which of this lane's sums are not finite, then each again from the definition
        uint32_t bad[TMB * NBW];
#pragma unroll
        for (int q = 0; q < TMB * NBW; ++q) {
            bad[q] = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) bad[q] |= __builtin_isfinite(acc[q / NBW][q % NBW][v]) ? 0u : 1u << v;
        }
#pragma unroll
        for (int q = 0; q < TMB * NBW; ++q) {
            const int p = p0 + wave * 64 + (q % NBW) * 32 + li;
            if (p >= a.OHW) continue;
            uint32_t oy, ox;
            a.dOW.divmod((uint32_t)p, oy, ox);
            for (uint32_t left = bad[q]; left; left &= left - 1) {
                const int v = __builtin_ctz(left), k = m0 + (q / NBW) * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                if (k >= a.K) continue;
                float y = 0.0f;
                for (int c = 0; c < C; ++c)
                    for (int r = 0; r < R; ++r) {
                        const int iy = (int)oy * ST - a.pad + r;
                        if ((unsigned)iy >= (unsigned)a.H) continue;
                        const float* x = (const float*)a.in + ((size_t)(img * C + c) * a.H + iy) * a.W;
                        const float* f = (const float*)a.filt + ((size_t)(k * C + c) * R + r) * S;
                        for (int s = 0; s < S; ++s) {
                            const int ix = (int)ox * ST - a.pad + s;
                            if ((unsigned)ix < (unsigned)a.W) y = __builtin_fmaf(x[ix], f[s], y);
                        }
                    }
                y += a.bias ? a.bias[k] : 0.0f;
                ((float*)a.out)[((size_t)img * a.K + k) * a.OHW + p] = a.relu ? (y > 0.0f ? y : 0.0f) : y;
            }
        }
    }
}

template <class CFG>
size_t swins_workspace(const Variant&, const conv_desc& d, int, int)
{
    return (size_t)CFG::KSTEPS * (size_t)((d.K + 31) / 32) * 3072;
}

// (the last steps read up to three lines past the window's last one, to no use; rows past the tile's go to a fourth)
inline size_t swins_lds(const SwinsGeom& g) { return ((size_t)g.rows * 3 + 4) * g.pitch * 4; }

template <class CFG>
hipError_t swins_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    SwinsGeom g = swins_geom(CFG::TN, CFG::R, CFG::ST, a.W, a.pad, a.OH, a.OW);
    const hipError_t e = ensure_dynamic_lds((const void*)swins_kernel<CFG>, swins_lds(g));
    if (e != hipSuccess) return e;
    const int blocks = (a.K + 31) / 32;
    hipLaunchKernelGGL(swins_filter_kernel<CFG>, dim3((unsigned)blocks, (unsigned)CFG::KSTEPS), dim3(64), 0, s, (const float*)a.filt, (uint4*)a.ws, a.K);
    g.dT = make_fastdiv((uint32_t)g.tpi);
    hipLaunchKernelGGL(swins_kernel<CFG>, dim3((unsigned)(a.N * g.tpi), (unsigned)((a.K + CFG::TM - 1) / CFG::TM)), dim3(CFG::NT), swins_lds(g), s, a, g);
    return hipGetLastError();
}

template <class CFG>
bool swins_valid(const Variant&, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != CONV_F32 || d.C != CFG::C || d.R != CFG::R || d.S != CFG::S || d.stride != CFG::ST || d.pad >= CFG::R || d.W < 4) return false;
    if (d.flags & ~(uint32_t)CONV_FLAG_RELU) return false;               // plain formats, no fused pool
    if (CFG::TM > ((d.K + 31) / 32) * 32 && CFG::TMB > 1) return false;  // an empty channel block only costs time
    const SwinsGeom g = swins_geom(CFG::TN, CFG::R, CFG::ST, d.W, d.pad, OH, OW);
    if (swins_lds(g) > 160 * 1024) return false;
    const long long lim = 1LL << 31;
    // (a channel that does not exist is stored at 2 GiB plus the offset of its row, which must not pass 4 GiB)
    if ((long long)d.N * d.C * d.H * d.W * 4 >= lim || ((long long)d.N * d.K + CFG::TM) * OH * OW * 4 >= lim) return false;
    // split filters and their offsets, a tile's spare blocks behind the last one among them
    if ((long long)CFG::KSTEPS * ((d.K + 31) / 32 + CFG::TMB) * 3072 >= lim) return false;
    return (long long)d.N * g.tpi < lim && (d.K + CFG::TM - 1) / CFG::TM < 65536;
}

template <class CFG>
void swins_register(std::vector<Variant>& out)
{
    Variant v;
    char buf[160];
    snprintf(buf, sizeof buf, "swins_f32_%dx%ds%d_c3_M%dN%d", CFG::R, CFG::S, CFG::ST, CFG::TM, CFG::TN);
    v.name = buf;
    v.dtype = CONV_F32;
    v.split = 1;
    v.tm = CFG::TM;
    v.tn = CFG::TN;
    v.tk = CFG::KSTEPS * 16;
    v.threads = CFG::NT;
    v.family = FAM_WINDOW;
    v.specificity = 6;
    v.traits = TRAIT_SPLIT_FIRST;
    v.valid = &swins_valid<CFG>;
    v.launch = &swins_launch<CFG>;
    v.ws_extra = &swins_workspace<CFG>;
    out.push_back(v);
}

}  // namespace convfwd
