// Winograd F(2x2, 3x3) for fp32 3x3 stride-1 layers with its products on the 16-bit matrix units.
//
// The transforms are those of wino_kernel.h; the 16 products M[xi][k][t] = sum_c U[xi][k][c] * V[xi][c][t] are what bounds
// that kernel: the fp32 matrix rate of this device is 1/16 of the bf16 one and an fp32 MFMA never overlaps with vector-ALU
// work.  Here every fp32 operand x is split into three bf16 numbers, x = x0 + x1 + x2 (each the round-to-nearest bf16 of
// what is left; 3 x 8 significant bits and two signs hold all 24), and a product is the sum of the six partial products
// down to 2^-16 of the leading one,
//     u v ~ u0 v0 + u0 v1 + u1 v0 + u1 v1 + u0 v2 + u2 v0,
// accumulated in fp32 by v_mfma_f32_32x32x16_bf16.  The three left out are below 2^-24 |u v|, and sixteen channels enter
// the accumulator with one rounding, so that the error is no larger than that of the fp32 kernels (2-norm of the difference
// to a 64-bit convolution over its 2-norm, half-normal inputs: 13x13x256 -> 384 3.4e-7 against 4.0e-7 for wino_kernel, 4.4e-7
// for wconv_kernel and 8.6e-7 for the implicit GEMMs; 56x56x64 -> 192 1.7e-7, 2.1e-7, -, 4.3e-7).
//   * U is split by the filter transform, in MFMA operand order: a wave's fragment is 1 KB, loaded straight into registers.
//   * V stays fp32 in LDS ([plane][channel quad][tile][4]): a plane belongs to one wave, so splitting it in that wave costs
//     nothing twice and moves 4 bytes per value through LDS instead of 6.
//   * A step is 16 channels in two stages, one per plane of a wave, with a barrier behind each.  Under the products of its
//     first plane a wave splits the second and transforms its task of step i+1; under those of the second it splits the
//     first plane of step i+1 and writes the input rows of step i+2 to LDS.  One buffer of each kind suffices.  The mix is
//     asked for instruction by instruction: left alone, the compiler puts the vector work first and the loads last.
//   * Input rows are fetched 16 bytes per lane, the last vector of a row ending with the row: with 4-byte loads the issue
//     of the loads alone took 300 .. 1700 clocks of a wave's 4000 per step.  Neighbouring tile rows share their rows.
//   * With 64 or 96 channels (LOOP) the grid is one workgroup per CU, which takes tile after tile; the steps of successive tiles
//     follow each other, so that only the first one pays for its start (64 images of 56x56x64 -> 192 are 12.25 tiles per CU: with
//     a workgroup for each, starts and drained stores took a third of the call).  The inverse transform has its own piece of LDS for
//     that; channels come to it 32 at a time.  A layer of fewer tiles than CUs loses nothing by it.
// What bounds it: bytes from L2 first.  A step of 96 channels x 32 tiles fetches 147 KB of filters and 20 to 36 of rows and takes
// 5600 clocks, 32 bytes a clock and CU; its MFMAs are 2304.  On 64 images of 56x56x64 -> 192 the counters show 2.18 GB from L2 in 185 us and
// MFMAs busy for 54.  Left out one at a time: the inverse transform 42 us (19 of them its stores), loads of filters 25, of rows 44
// (the products are then of zeros), splits 24, input transform 12, the code that sums tiles again 9, by its registers; the thirteenth
// round of tiles is a quarter full.  With 96 channels and five row vectors 4 registers are spilled, reloaded once a tile, outside
// the steps.  Filters requested earlier (each part as soon as its
// last product is issued) gain nothing.  Tiles of 64 would halve the filters' bytes but need twice the accumulators (238 us where
// 96 x 32 took 218, both without LOOP); two workgroups of 32 x 32 per CU double the vector work per product (350).  Taking a
// split's parts out with v_dot2_f32_bf16 (7 instructions a pair instead of 11) was 0 to 5 % slower.
// Measured (us per call, other inputs each time, filter transform included, a workgroup per tile -> LOOP, same box in turn): 64 images of
// 56x56x64 -> 192 217 -> 185 (M96), 251 -> 193 (M64), 16 of 28x28x128 -> 256 43.2 -> 40.0, 8 of 40x40x96 -> 100 21.2 -> 21.1; 20 of
// 13x13x256 -> 384, 186 tiles, 34.9 both ways (7 of them the filter transform).
// Range: the parts of x reach 24 bits below x, which for |x| < 2^-102 is below bf16's normal numbers.  Both operands are
// therefore scaled by 2^24 ahead of the splits: every part of every fp32 number, subnormal ones included, is then a normal
// bf16 number or zero, whatever the other operand is.  Sums carry 2^48 and are scaled back behind the inverse transform.
// What this can lose is at the upper end, and shows: an operand above 2^103, a sum above 2^79 or an infinity gives an
// infinity or a NaN in every output that it reaches.  An output tile that is not finite is summed again in fp32 from the
// definition (winos_sum_again).
#pragma once

#include "pwin_kernel.h"
#include "split_products.h"
#include "wino_kernel.h"

namespace convfwd {

template <int MB_, int LBV_, int RING_>
struct WinosCfg {
    static constexpr int MB = MB_, LBV = LBV_, RING = RING_;
    static_assert((2 * MB) % RING == 0 && RING >= 2, "the filter ring must divide the groups of a step");
    static constexpr int NT = 512;        // 8 waves of two planes
    static constexpr int WPS = MB == 1 && LBV <= 2 ? 4 : 2;  // waves per SIMD the registers are fitted to
    static constexpr bool LOOP = MB > 1;  // a workgroup takes one tile after another, each started beneath the one before
    static constexpr int TM = 32 * MB;    // output channels per workgroup
    static constexpr int TT = 32;         // tiles (2x2 output blocks) per workgroup: one transform task (tile, channel) per thread
    static constexpr int V_FLOATS = 16 * 4 * TT * 4;
    static constexpr int MP = TT + 4;     // row pitch of the plane buffer of the epilogue
    static constexpr int E_FLOATS = 16 * 32 * MP;  // a 32-channel block at a time
    static constexpr int SLOTS = NT * LBV;  // 16-byte vectors of input rows staged per step
    static constexpr int SPARE = 64 * 4;    // a vector per lane behind the rows, for tasks without a row
    // the inputs are scaled where that takes fewer instructions: staged rows 4 * LBV, transform 8 per thread and step (at
    // equal counts the rows are better, beneath the stage with less vector work)
    static constexpr bool SCALE_ROWS = LBV <= 2;
};

struct WinosGeom {
    int TH, TW, tiles;
    int IR;        // staged rows of an image: 2 * TH + 2
    int rows_max;  // most rows a workgroup stages
    int W4;        // 16-byte vectors of a row; the last one ends with the row
    int PWL;       // floats per staged row
    int pitch;     // floats per channel of the staged rows, 16 mod 64: the lanes of a transform read distinct banks
    int KT, TN;    // channel tiles, groups of tiles
    FastDiv dTW, dIR, dTH, dW4, dRow, dGroup;  // by TW, IR, TH, W4, rows_max * W4 and 3 * TN
};

template <class CFG>
inline WinosGeom winos_geom(int N, int K, int W, int OH, int OW)
{
    WinosGeom g;
    g.TH = (OH + 1) / 2;
    g.TW = (OW + 1) / 2;
    g.tiles = N * g.TH * g.TW;
    g.IR = 2 * g.TH + 2;
    const int up = (CFG::TT + g.TW - 2) / g.TW;  // tile rows between a workgroup's first and last tile
    int cross = (up + g.TH - 1) / g.TH;
    if (cross > N - 1) cross = N - 1;
    g.rows_max = 2 * up + 4 + 2 * cross;
    g.W4 = (W + 3) / 4;
    g.PWL = 2 * g.TW + 2;
    g.pitch = g.rows_max * g.PWL;
    g.pitch += ((16 - g.pitch % 64) + 64) % 64;
    g.KT = (K + CFG::TM - 1) / CFG::TM;
    g.TN = (g.tiles + CFG::TT - 1) / CFG::TT;
    return g;
}

template <class CFG>
size_t winos_lds_bytes(const WinosGeom& g)
{
    const size_t pipe = sizeof(float) * (CFG::V_FLOATS + 16 * (size_t)g.pitch + CFG::SPARE);
    const size_t epi = sizeof(float) * CFG::E_FLOATS;
    return CFG::LOOP ? pipe + epi : pipe > epi ? pipe : epi;
}

inline size_t winos_filter_bytes(int K, int C) { return (size_t)((C + 15) / 16) * 16 * ((K + 31) / 32) * 3072; }

// Filter transform, scaled: U[c / 16][xi][k / 32][part][lane][8], lane = k % 32 + 32 * (c % 16 / 8), 8 channels c % 8.  A
// workgroup takes 32 filters x 16 channels: their values go to LDS, then wave w computes planes 2w and
// 2w+1 of its lanes' eight channels and stores each part as one contiguous kilobyte.
__global__ __launch_bounds__(512) void winos_filter_kernel(const float* __restrict__ filt, uint4* __restrict__ U, int K, int C)
{
    constexpr int ROW = 16 * 9 + 1;  // odd pitch
    __shared__ float g_s[32 * ROW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mb = blockIdx.x, c16 = blockIdx.y;
    const int have = (C - c16 * 16 < 16 ? C - c16 * 16 : 16) * 9;
    // sixteen threads a filter, 64 bytes an instruction and filter: contiguous runs took a division and two 64-bit products a load,
    // 0.8 us of the call (20 images of 13x13x256 -> 384 36.3 -> 35.5, 8 of 33x35x100 -> 130 24.2 -> 23.9)
    const int row_l = tid >> 4, j0 = tid & 15, k = mb * 32 + row_l;
    const __amdgpu_buffer_rsrc_t rf = make_rsrc(filt, (uint32_t)K * (uint32_t)C * 36u);
    const uint32_t off = (uint32_t)k * ((uint32_t)C * 36u) + (uint32_t)j0 * 4u;
    float v[9];
#pragma unroll
    for (int i = 0; i < 9; ++i)
        v[i] = buffer_load_elem<float>(rf, k < K && j0 + 16 * i < have ? off + (uint32_t)c16 * 576u + (uint32_t)i * 64u : kOutOfRange);
#pragma unroll
    for (int i = 0; i < 9; ++i) g_s[row_l * ROW + j0 + 16 * i] = v[i];
    __syncthreads();
    const int kl = lane & 31, g8 = lane >> 5, row = wave >> 1;
    float u[2][8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float* g = g_s + kl * ROW + (g8 * 8 + c) * 9;
        float t[3];  // row `row` of G g, scaled (here and not at the loads, which would each be waited for: 1.3 us more)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const float g0 = g[j], g1 = g[3 + j], g2 = g[6 + j];
            t[j] = row == 0 || row == 3 ? kSplitScale * (row == 0 ? g0 : g2) : 0.5f * kSplitScale * ((g0 + g2) + (row == 1 ? g1 : -g1));
        }
        const float s = t[0] + t[2];
        u[0][c] = (wave & 1) ? 0.5f * (s - t[1]) : t[0];
        u[1][c] = (wave & 1) ? t[2] : 0.5f * (s + t[1]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const Split3 s = split3(u[j]);
        uint4* dst = U + (((size_t)c16 * 16 + wave * 2 + j) * gridDim.x + mb) * 192 + lane;
#pragma unroll
        for (int q = 0; q < 3; ++q) dst[q * 64] = s.p[q];
    }
}

struct WinosArgs {
    ConvArgs a;  // a.ws holds U
    WinosGeom d;
};

// The kernel's arguments, to be read again where they are asked for: what a tile needs once would otherwise be kept in scalar
// registers through the loop, more of them than there are (150 moves a step between them and lanes of vector registers)
__device__ __forceinline__ const WinosArgs& winos_args_again()
{
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const WinosArgs*)p;
}

// Entries (filter k, image n, window origin iy, ix of a tile's first output) of the lanes in `mask`, summed in fp32 from the
// definition: taps outside the image are left out.  The wave takes them together, 64 / entries lanes (rounded down to a
// power of two) for each, which share its channels; a tile's four outputs share their loads; a lane whose sums are all
// NaN is done.  Bound by the scattered loads.  Call of 20 images of 13x13x256 -> 384 (39 us on ordinary data) with one
// infinite pixel 141 us, one NaN filter value 120, NaN everywhere 41, results beyond 2^79 everywhere 787; with one lane
// per entry and output 7900, 1370, 5900 and 5900.
__device__ __forceinline__ void winos_sum_again(const ConvArgs& a, int lane, uint64_t mask, int k, int n, int iy, int ix, float* y)
{
    constexpr uint32_t kFar = 0x80000000u;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    const int count = __builtin_popcountll(mask), lg = 31 - __builtin_clz(64 / count);
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    const bool mine = (mask >> lane) & 1;
    const int entry = lane >> lg, step = 1 << lg;
    // (lanes outside the mask push to the last lane, which no entry reads when there are any)
    const int owners = __builtin_amdgcn_ds_permute((mine ? rank : 63) * 4, lane);
    const int owner = __shfl(owners, entry < count ? entry : 0);
    k = __shfl(k, owner);
    n = __shfl(n, owner);
    iy = __shfl(iy, owner);
    ix = __shfl(ix, owner);
    const int x0 = ix < 0 ? 0 : ix > a.W - 4 ? a.W - 4 : ix, d = ix - x0;  // d in -1 .. 2
    bool in_x[4];
    uint32_t row[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        in_x[r] = (unsigned)(ix + r) < (unsigned)a.W;
        const bool in_y = (unsigned)(iy + r) < (unsigned)a.H && entry < count;
        row[r] = in_y ? (uint32_t)((n * a.C * a.H + iy + r) * a.W + x0) * 4u : kFar;
    }
    const __amdgpu_buffer_rsrc_t rf = make_rsrc(a.filt, a.filt_bytes);
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int c = lane & (step - 1); entry < count && c < a.C; c += step) {
        const uint32_t fo = (uint32_t)(k * a.C + c) * 36u;
        const f32x4 f0 = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rf, (int)fo, 0, 0));
        const f32x4 f1 = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rf, (int)fo, 16, 0));
        const float f8 = buffer_load_elem<float>(rf, fo + 32u);
        const float f[9] = {f0[0], f0[1], f0[2], f0[3], f1[0], f1[1], f1[2], f1[3], f8};
        f32x4 v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            v[r] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rin, (int)(row[r] == kFar ? kFar : row[r] + (uint32_t)(c * a.HW) * 4u), 0, 0));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x[4] = {d < 0 ? 0.0f : d == 0 ? v[r][0] : d == 1 ? v[r][1] : v[r][2],
                                d < 0 ? v[r][0] : d == 0 ? v[r][1] : d == 1 ? v[r][2] : v[r][3],
                                d < 0 ? v[r][1] : d == 0 ? v[r][2] : d == 1 ? v[r][3] : 0.0f,
                                d < 0 ? v[r][2] : d == 0 ? v[r][3] : 0.0f};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int w = r - (q >> 1);  // row of the window
                if (w < 0 || w > 2) continue;
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const int cx = (q & 1) + t;
                    s[q] = row[r] != kFar && in_x[cx] ? __builtin_fmaf(x[cx], f[w * 3 + t], s[q]) : s[q];
                }
            }
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
__global__ __launch_bounds__(CFG::NT, CFG::WPS) void winos_kernel(WinosArgs w)
{
    const ConvArgs& a = w.a;
    const WinosGeom& d = w.d;
    constexpr int MB = CFG::MB, LBV = CFG::LBV, NT = CFG::NT, TM = CFG::TM, TT = CFG::TT, MP = CFG::MP;
    asm volatile("" ::"s"(a.in), "s"(a.ws), "s"(a.N), "s"(a.C), "s"(a.H), "s"(a.W), "s"(a.K), "s"(a.pad), "s"(a.HW), "s"(a.in_bytes), "s"(d.tiles), "s"(d.IR), "s"(d.rows_max), "s"(d.PWL), "s"(d.pitch));
    asm volatile("" ::"s"(d.KT), "s"(d.TN), "s"(d.dTW.mul), "s"(d.dTW.shift), "s"(d.dTW.d), "s"(d.dIR.mul), "s"(d.dIR.shift), "s"(d.dIR.d), "s"(d.dTH.mul), "s"(d.dTH.shift), "s"(d.dTH.d), "s"(d.dW4.mul), "s"(d.dW4.shift), "s"(d.dW4.d), "s"(d.dRow.mul), "s"(d.dRow.shift), "s"(d.dRow.d), "s"(d.dGroup.mul), "s"(d.dGroup.shift), "s"(d.dGroup.d));
    constexpr uint32_t kFar = 0x80000000u;  // tensors stay below 2 GiB: this offset plus any scalar offset is out of range
    typedef Mma<CONV_BF16, 32> mma_t;
    extern __shared__ __attribute__((aligned(16))) float smem[];

    const int PWL = d.PWL, pitch = d.pitch;
    float* const Vs = smem;                  // [16][4][TT][4]
    float* const Rs = smem + CFG::V_FLOATS;  // [16][pitch], then the spare vectors
    float* const Ms = CFG::LOOP ? Rs + 16 * pitch + CFG::SPARE : smem;  // [16][32][MP], of the epilogue

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C16 = (a.C + 15) >> 4, MBK = (a.K + 31) >> 5;
    // An XCD's workgroups share a contiguous run of "groups of 3 channel tiles; within a group all tile groups", workgroup
    // `mine` of `wgs` its tiles mine, mine + wgs, ...
    const int total = d.KT * d.TN, xcd = blockIdx.x & 7, mine = blockIdx.x >> 3;
    const int first = xcd * (total >> 3) + (xcd < (total & 7) ? xcd : (total & 7)), count = (total >> 3) + (xcd < (total & 7) ? 1 : 0);
    const int wgs = ((int)gridDim.x >> 3) + (xcd < ((int)gridDim.x & 7) ? 1 : 0);
    struct Place {
        int t0, m0;
    };
    auto place_of = [&](const WinosGeom& d, int q) {
        uint32_t gr, rem;
        d.dGroup.divmod((uint32_t)(first + q), gr, rem);
        const int left = d.KT - 3 * (int)gr, gs = left < 3 ? left : 3;
        const uint32_t tg = gs == 3 ? rem / 3u : rem >> (gs - 1);
        return Place{(int)tg * TT, (3 * (int)gr + (int)(rem - tg * gs)) * TM};
    };

    // ---- transformed filters: ring of groups (plane of this wave, 32-channel block), three parts each ----------------
    constexpr int GRP = 2 * MB, RING = CFG::RING;
    const __amdgpu_buffer_rsrc_t ru = make_rsrc(a.ws, (uint32_t)C16 * 16u * (uint32_t)MBK * 3072u);
    const uint32_t a_lane = (uint32_t)lane * 16u;
    const uint32_t u_plane = (uint32_t)MBK * 3072u, u_step = u_plane * 16u;
    auto filters_of = [&](const Place& p) { return (uint32_t)(wave * 2) * u_plane + (uint32_t)(p.m0 >> 5) * 3072u; };
    uint4 ar[RING][3];
    auto load_a = [&](auto slot_c, auto grp_c, uint32_t base) {
        constexpr int slot = decltype(slot_c)::value, grp = decltype(grp_c)::value;
        const uint32_t soff = base + (uint32_t)(grp / MB) * u_plane + (uint32_t)(grp % MB) * 3072u;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            // (the part's kilobyte in a scalar or a vector register, whichever kind is short in the loop)
            const u32x4 v = CFG::LOOP ? __builtin_amdgcn_raw_buffer_load_b128(ru, (int)(a_lane + q * 1024u), (int)soff, 0)
                                      : __builtin_amdgcn_raw_buffer_load_b128(ru, (int)a_lane, (int)(soff + q * 1024u), 0);
            ar[slot][q] = make_uint4(v.x, v.y, v.z, v.w);
        }
    };

    // ---- input rows ----------------------------------------------------------------------------------------------------
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    auto stacked_row = [&](const WinosGeom& d, uint32_t tile_row) {
        uint32_t n, ty;
        d.dTH.divmod(tile_row, n, ty);
        return (int)n * d.IR + 2 * (int)ty;
    };
    auto first_row = [&](const WinosGeom& d, int t0) { return __builtin_amdgcn_readfirstlane(stacked_row(d, d.dTW.div((uint32_t)t0))); };
    // task = (channel of the step, staged row, 16-byte vector of the row): the loads of a wave are contiguous runs of rows
    uint32_t r_goff[LBV];
    int r_lds[LBV], r_task[LBV];  // r_task: column, channel << 12, row << 16
#pragma unroll
    for (int i = 0; i < LBV; ++i) {
        uint32_t c, e, ri, xv;
        d.dRow.divmod((uint32_t)(i * NT + tid), c, e);
        d.dW4.divmod(e, ri, xv);
        const int x = (int)xv * 4 < a.W - 4 ? (int)xv * 4 : a.W - 4;
        r_lds[i] = c < 16u ? (int)(ri * (uint32_t)PWL + c * (uint32_t)pitch) + x + a.pad : 16 * pitch + lane * 4;
        r_task[i] = x | (int)(c & 15u) << 12 | (c < 16u ? (int)ri : 0x7fff) << 16;
    }
    // Rows are fetched for tile `row_q`, step `row_step`, up to three steps ahead of the products
    int row_q = mine, row_step = 0;
    auto aim_rows = [&](const WinosArgs& w) {
        if (row_q >= count) {
#pragma unroll
            for (int i = 0; i < LBV; ++i) r_goff[i] = kFar;
            return;
        }
        const ConvArgs& a = w.a;
        const WinosGeom& d = w.d;
        const int t0 = place_of(d, row_q).t0, t_last = (t0 + TT < d.tiles ? t0 + TT : d.tiles) - 1;
        const int s0 = first_row(d, t0), nrows = first_row(d, t_last) + 4 - s0;
#pragma unroll
        for (int i = 0; i < LBV; ++i) {
            const int ri = r_task[i] >> 16, c = r_task[i] >> 12 & 15, x = r_task[i] & 0xfff;
            uint32_t n, yy;
            d.dIR.divmod((uint32_t)(s0 + ri), n, yy);
            const int y = (int)yy - a.pad;
            const bool ok = ri < nrows && (unsigned)y < (unsigned)a.H && (int)n < a.N;
            r_goff[i] = ok ? (uint32_t)((((int)n * a.C + c) * a.H + y) * a.W + x) * 4u : kFar;
        }
    };
    const uint32_t step_bytes = (uint32_t)a.HW * 64u;
    struct Rows {
        f32x4 v[LBV];
    };
    auto load_rows = [&](Rows& r) {  // channels past the last one read as zero
#pragma unroll
        for (int i = 0; i < LBV; ++i)
            r.v[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rin, (int)(row_step * 16 + (r_task[i] >> 12 & 15) < a.C ? r_goff[i] : kFar),
                                                                                     (int)((uint32_t)row_step * step_bytes), 0));
        ++row_step;
        if (CFG::LOOP && row_step == C16) {
            row_step = 0;
            row_q += wgs;
            aim_rows(winos_args_again());
        }
    };
    auto store_rows = [&](const Rows& r) {  // (rows outside the image are written too, as zeros)
#pragma unroll
        for (int i = 0; i < LBV; ++i) {
            float* dst = Rs + r_lds[i];
#pragma unroll
            for (int j = 0; j < 4; ++j) dst[j] = CFG::SCALE_ROWS ? r.v[i][j] * kSplitScale : r.v[i][j];
        }
    };

    // ---- input transform: thread = (tile, channel) ---------------------------------------------------------------------
    const int v_quad = wave & 3, v_sub = lane & 3, v_tile = (wave >> 2) * 16 + (lane >> 2);
    typedef __attribute__((address_space(3))) char* lds_bytes;
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(3))) f32x2* lds_pairs;
    uint32_t v_src[4];  // LDS address of a row each: addresses made in the loop would push its LDS reads behind the products they belong above
    auto aim_transform = [&](const WinosGeom& d, int t0) {
        const int t = (t0 + v_tile < d.tiles) ? t0 + v_tile : t0;  // tiles past the end repeat the first one; never stored
        uint32_t gr, tx;
        d.dTW.divmod((uint32_t)t, gr, tx);
        v_src[0] = (uint32_t)(uintptr_t)(lds_bytes)smem + (uint32_t)(CFG::V_FLOATS + (v_quad * 4 + v_sub) * d.pitch + (stacked_row(d, gr) - first_row(d, t0)) * d.PWL + 2 * (int)tx) * 4u;
#pragma unroll
        for (int r = 1; r < 4; ++r) v_src[r] = v_src[r - 1] + (uint32_t)d.PWL * 4u;
    };
    float* const v_dst = Vs + (v_quad * TT + v_tile) * 4 + v_sub;
    struct Tile {
        float2 lo[4], hi[4];
    };
    auto read_tile = [&]() {
        Tile d;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const lds_pairs src = (lds_pairs)(uintptr_t)v_src[r];
            d.lo[r] = make_float2(src[0][0], src[0][1]);
            d.hi[r] = make_float2(src[1][0], src[1][1]);
        }
        return d;
    };
    auto write_tile = [&](const Tile& b) {
        float d[4][4], t[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            d[r][0] = b.lo[r].x; d[r][1] = b.lo[r].y; d[r][2] = b.hi[r].x; d[r][3] = b.hi[r].y;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            constexpr float sc = CFG::SCALE_ROWS ? 1.0f : kSplitScale;
            const float d1 = d[1][j] * sc, d2 = d[2][j] * sc;
            t[0][j] = __builtin_fmaf(d[0][j], sc, -d2);
            t[1][j] = d1 + d2;
            t[2][j] = d2 - d1;
            t[3][j] = __builtin_fmaf(d[3][j], -sc, d1);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v_dst[(4 * i + 0) * 16 * TT] = t[i][0] - t[i][2];
            v_dst[(4 * i + 1) * 16 * TT] = t[i][1] + t[i][2];
            v_dst[(4 * i + 2) * 16 * TT] = t[i][2] - t[i][1];
            v_dst[(4 * i + 3) * 16 * TT] = t[i][1] - t[i][3];
        }
    };

    typename mma_t::acc_t acc[2][MB];
    auto clear = [&]() {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[x][mb][v] = 0.0f;
    };

    // lane (li, g) feeds column li of a block with channels 8g .. 8g+7 of the step
    struct Plane {
        f32x4 lo, hi;
    };
    auto read_plane = [&](int x) {
        const float* src = Vs + ((wave * 2 + x) * 4 + 2 * g) * TT * 4 + li * 4;
        return Plane{*(const f32x4*)src, *(const f32x4*)&src[TT * 4]};
    };
    auto split_plane = [&](const Plane& p) {
        const float x[8] = {p.lo[0], p.lo[1], p.lo[2], p.lo[3], p.hi[0], p.hi[1], p.hi[2], p.hi[3]};
        return split3(x);
    };
    // the six partial products of plane x, smallest first; the filters of group grp + RING - 1 are fetched meanwhile
    auto multiply = [&](auto xc, const Split3& b, uint32_t now, uint32_t next) {
        constexpr int x = decltype(xc)::value;
        static_for<MB>([&](auto mbc) {
            constexpr int mb = decltype(mbc)::value, grp = x * MB + mb, ahead = grp + RING - 1;
            constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
            load_a(std::integral_constant<int, ahead % RING>{}, std::integral_constant<int, ahead % GRP>{}, ahead < GRP ? now : next);
#pragma unroll
            for (int q = 0; q < 6; ++q) acc[x][mb] = mma_t::run(ar[grp % RING][pa[q]], b.p[pb[q]], acc[x][mb]);
        });
    };
    // asks for one MFMA, then LDS writes and vector work that fit beneath it, and so on through a stage
    auto interleave = [&](auto valu_c, auto dsw_c) {
        constexpr int valu = decltype(valu_c)::value, dsw = decltype(dsw_c)::value;
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
        static_for<6 * MB>([&](auto ic) {
            if constexpr (decltype(ic)::value % 6 == 0) __builtin_amdgcn_sched_group_barrier(0x020, 3, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, valu, 0);
            __builtin_amdgcn_sched_group_barrier(0x200, dsw, 0);
        });
    };
    typedef std::integral_constant<int, 0> c0_t;
    typedef std::integral_constant<int, 1> c1_t;

    // ---- epilogue, 32 channels at a time: planes to LDS, inverse transform, bias + activation, 2x2 stores ---------------
    auto finish = [&](const Place& at) {
        const WinosArgs& w = winos_args_again();
        const ConvArgs& a = w.a;
        const WinosGeom& d = w.d;
        const __amdgpu_buffer_rsrc_t rout = make_rsrc(a.out, a.out_bytes);
        const bool even = (a.OW & 1) == 0;  // a tile's two outputs of a row are 8-byte aligned and both inside
        // thread = (tile, channel of 16): two channels of each block
        const int kr = tid >> 5, t = at.t0 + li;
        const bool in = t < d.tiles;
        uint32_t gr, tx, n, ty;
        d.dTW.divmod(in ? (uint32_t)t : 0u, gr, tx);
        d.dTH.divmod(gr, n, ty);
        const int oy = 2 * (int)ty, ox = 2 * (int)tx;
        const uint32_t base = (uint32_t)(((int)n * a.K + at.m0 + kr) * a.OHW + oy * a.OW + ox) * 4u;
        const uint32_t plane = (uint32_t)a.OHW * 4u, row = (uint32_t)a.OW * 4u;
        const bool in1 = in && oy + 1 < a.OH, right = ox + 1 < a.OW;
        float bias[MB][2];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < 2; ++j) {  // (scalar loads: vector ones would wait for the rows on their way)
                float b0 = 0.0f, b1 = 0.0f;
                if (a.bias) {
                    const int k = at.m0 + mb * 32 + j * 16 + wave * 2, top = a.K - 1;
                    b0 = a.bias[k < top ? k : top], b1 = a.bias[k + 1 < top ? k + 1 : top];
                }
                bias[mb][j] = g ? b1 : b0;
            }
        auto store = [&](uint32_t o, bool ok, bool ok1, const float* y) {
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
                const bool in_row = dy ? ok1 : ok;
                const uint32_t oo = in_row ? o + (dy ? row : 0u) : kOutOfRange;
                if (even) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__builtin_bit_cast(uint32_t, y[2 * dy]), __builtin_bit_cast(uint32_t, y[2 * dy + 1])},
                                                          rout, (int)oo, 0, 0);
                } else {
                    buffer_store_elem<float>(y[2 * dy], rout, oo);
                    buffer_store_elem<float>(y[2 * dy + 1], rout, in_row && right ? oo + 4u : kOutOfRange);
                }
            }
        };
        uint32_t bad = 0;  // bit 2 * block + half: sums that are not finite
        static_for<MB>([&](auto mbc) {
            constexpr int mb = decltype(mbc)::value;
            if constexpr (mb > 0) __syncthreads();
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int v = 0; v < 16; ++v) Ms[((wave * 2 + x) * 32 + acc_row<32>(v, lane)) * MP + li] = acc[x][mb][v];
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int kl = j * 16 + kr;
                const float* src = Ms + kl * MP + li;
                float m[4][4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) m[i][jj] = src[(4 * i + jj) * 32 * MP];
                float r0[4], r1[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    r0[jj] = (m[0][jj] + m[1][jj]) + m[2][jj];
                    r1[jj] = (m[1][jj] - m[2][jj]) - m[3][jj];
                }
                float y[4];
                y[0] = (r0[0] + r0[1]) + r0[2];
                y[1] = (r0[1] - r0[2]) - r0[3];
                y[2] = (r1[0] + r1[1]) + r1[2];
                y[3] = (r1[1] - r1[2]) - r1[3];
                const float big = (__builtin_fabsf(y[0]) + __builtin_fabsf(y[1])) + (__builtin_fabsf(y[2]) + __builtin_fabsf(y[3]));
                const bool fine = big < __builtin_inff();  // no NaN, no infinity in any of the four
                const bool have = at.m0 + mb * 32 + kl < a.K;
                bad |= in && have && !fine ? 1u << (2 * mb + j) : 0u;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    y[q] = __builtin_fmaf(y[q], kSplitUnscale, bias[mb][j]);
                    if (a.relu) y[q] = __builtin_fmaxf(y[q], 0.0f);
                }
                store(base + (uint32_t)(mb * 32 + j * 16) * plane, in && have && fine, in1 && have && fine, y);
            }
        });
        if (__any(bad != 0)) {
#pragma unroll 1
            for (int e = 0; e < 2 * MB; ++e) {
                const uint64_t again = __ballot(bad >> e & 1);
                if (!again) continue;
                const int k = at.m0 + e * 16 + kr;
                float y[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                winos_sum_again(a, lane, again, k, (int)n, oy - a.pad, ox - a.pad, y);
                const bool mine_ = bad >> e & 1;
                const float b = a.bias && mine_ ? a.bias[k] : 0.0f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    y[q] += b;
                    if (a.relu) y[q] = y[q] > 0.0f ? y[q] : 0.0f;
                }
                store(base + (uint32_t)(e * 16) * plane, mine_, mine_ && in1, y);
            }
        }
    };

    // ---- pipeline: entering step i, Vs holds the tiles of step i, `p0` the parts of this wave's first plane and `v1` its
    // second plane, Rs the rows of step i+1, and the rows of step i+2 are in flight.  Every wave holds all it needs of Vs.
    // The steps of a workgroup's tiles follow each other without a gap.
    Rows rows, rows1;
    Place here = place_of(d, mine);
    uint32_t now = filters_of(here);
    aim_rows(w);
    load_rows(rows);
    static_for<RING - 1>([&](auto gc) { load_a(gc, gc, now); });
    load_rows(rows1);
    aim_transform(d, here.t0);
    for (int i = tid; i < 4 * pitch; i += NT) *(f32x4*)&Rs[4 * i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};  // the border stays zero
    __syncthreads();
    store_rows(rows);
    load_rows(rows);
    __syncthreads();
    write_tile(read_tile());
    __syncthreads();
    Split3 p0 = split_plane(read_plane(0)), p1;
    Plane v1 = read_plane(1);
    store_rows(rows1);
    clear();
    __syncthreads();
    auto step = [&](uint32_t next) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(v1.lo), "+v"(v1.hi));  // (its split belongs beneath the products that follow, not to the step before)
        const Tile t = read_tile();  // the step after (past the last one: nobody reads what becomes of it)
        p1 = split_plane(v1);
        multiply(c0_t{}, p0, now, next);
        write_tile(t);
        interleave(std::integral_constant<int, ((CFG::SCALE_ROWS ? 96 : 104) + 6 * MB - 1) / (6 * MB)>{}, std::integral_constant<int, (8 + 6 * MB - 1) / (6 * MB)>{});
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        const Plane v0 = read_plane(0);
        v1 = read_plane(1);
        multiply(c1_t{}, p1, now, next);
        store_rows(rows);
        p0 = split_plane(v0);
        interleave(std::integral_constant<int, (48 + 6 * MB - 1) / (6 * MB)>{}, std::integral_constant<int, (2 * LBV + 6 * MB - 1) / (6 * MB)>{});
        // (nor the split of the first plane behind the branch in load_rows)
        asm volatile("" ::"v"(__builtin_bit_cast(u32x4, p0.p[0])), "v"(__builtin_bit_cast(u32x4, p0.p[1])), "v"(__builtin_bit_cast(u32x4, p0.p[2])));
        __builtin_amdgcn_sched_barrier(0);
        load_rows(rows);
        __syncthreads();
        now = next;
    };
    if constexpr (!CFG::LOOP) {
        for (int i = 0; i < C16; ++i) step(now + u_step);
        finish(here);
        return;
    }
    for (int q = mine;;) {
        for (int i = 1; i < C16; ++i) step(now + u_step);
        // the last step of a tile prepares the first one of the next
        const int qn = q + wgs;
        const WinosGeom& d = winos_args_again().d;
        const Place there = qn < count ? place_of(d, qn) : here;
        if (qn < count) aim_transform(d, there.t0);
        step(filters_of(there));
        finish(here);
        if (qn >= count) break;
        clear();
        here = there, q = qn;
    }
}

template <class CFG>
size_t winos_ws_bytes(const Variant&, const conv_desc& d, int, int)
{
    return winos_filter_bytes(d.K, d.C);
}

template <class CFG>
hipError_t winos_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    WinosArgs w = {a, winos_geom<CFG>(a.N, a.K, a.W, a.OH, a.OW)};
    WinosGeom& g = w.d;
    const size_t lds = winos_lds_bytes<CFG>(g);
    const hipError_t e = ensure_dynamic_lds((const void*)winos_kernel<CFG>, lds);
    if (e != hipSuccess) return e;
    g.dTW = make_fastdiv((uint32_t)g.TW);
    g.dIR = make_fastdiv((uint32_t)g.IR);
    g.dTH = make_fastdiv((uint32_t)g.TH);
    g.dW4 = make_fastdiv((uint32_t)g.W4);
    g.dRow = make_fastdiv((uint32_t)(g.rows_max * g.W4));
    g.dGroup = make_fastdiv((uint32_t)(3 * g.TN));
    hipLaunchKernelGGL(winos_filter_kernel, dim3((unsigned)((a.K + 31) / 32), (unsigned)((a.C + 15) / 16)), dim3(512), 0, s,
                       (const float*)a.filt, (uint4*)a.ws, a.K, a.C);
    const hipError_t e2 = hipGetLastError();
    if (e2 != hipSuccess) return e2;
    const int total = g.TN * g.KT;  // (LOOP: one workgroup per CU, 256 of them)
    hipLaunchKernelGGL(winos_kernel<CFG>, dim3((unsigned)(CFG::LOOP && total > 256 ? 256 : total)), dim3(CFG::NT), lds, s, w);
    return hipGetLastError();
}

template <class CFG>
bool winos_valid(const Variant&, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != CONV_F32 || d.R != 3 || d.S != 3 || d.stride != 1 || d.pad > 1) return false;
    if (d.flags & ~(uint32_t)CONV_FLAG_RELU) return false;  // plain formats and filters, no fused pool
    // a step is 16 channels and a block 32 filters, neither worth it half empty; a row is at least one vector
    if (d.C < 8 || d.K <= 16 || d.W < 4) return false;
    // 32-bit byte offsets beside an out-of-range marker
    const long long lim = 1LL << 31;
    if (((long long)d.N * d.C + 64) * d.H * d.W * 4 >= lim || (long long)d.N * d.K * OH * OW * 4 >= lim) return false;
    if ((long long)winos_filter_bytes(d.K, d.C) * 2 >= lim || (d.C + 15) / 16 > 65535) return false;
    if ((long long)d.N * ((OH + 1) / 2 + 2) * ((OW + 1) / 2 + 1) >= (1LL << 28)) return false;
    const WinosGeom g = winos_geom<CFG>(d.N, d.K, d.W, OH, OW);
    if ((long long)g.rows_max * g.W4 * 16 > CFG::SLOTS) return false;  // every staged vector needs a slot
    if (winos_lds_bytes<CFG>(g) > 160 * 1024) return false;
    if ((long long)((d.K + CFG::TM - 1) / CFG::TM) * ((g.tiles + CFG::TT - 1) / CFG::TT) >= lim) return false;
    return true;
}

template <class CFG>
void winos_register(std::vector<Variant>& out, const TileModel& model)
{
    Variant v;
    char buf[96];
    snprintf(buf, sizeof buf, "winos_f32_M%dT%d_e%d_r%d", CFG::TM, CFG::TT, CFG::LBV, CFG::RING);
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
    v.per_cu = CFG::WPS / 2;
    v.model = model;
    v.valid = &winos_valid<CFG>;
    v.launch = &winos_launch<CFG>;
    v.ws_extra = &winos_ws_bytes<CFG>;
    out.push_back(v);
}

}  // namespace convfwd
