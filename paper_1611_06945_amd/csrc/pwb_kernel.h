// Pointwise (1x1, stride 1, no padding) convolution on the plain formats, fp16 / bf16, for many pixels:
//     Out[K x P] = Filt[K x C] * X[C x P],   X[c][(n,pix)] = in[n][c][pix].
// Such a layer is a stream: input read once, output written once, a few microseconds of matrix work beneath.  What the
// other kernels lose is the transposition: a lane of a 16-bit MFMA feeds 8 consecutive channels of one pixel, which lie a
// plane apart.  Here a lane loads NPX = 2 or 4 neighbouring pixels of its 8 channels (4 or 8 bytes each, a wave reads runs
// of 128 or 256 bytes of a plane) and puts pairs of channels together with one byte permute per operand register: pixel j
// of every lane is column block j of the MFMA, so NPX pixels per lane make NPX column blocks and nothing goes through LDS.
//   * The filters of the workgroup's 32*TMB channels are staged in LDS once (rows padded by 16 bytes); behind that one
//     barrier every wave runs alone, GD groups of 16 channels of input in flight.
//   * All channels of a tile belong to one wave, so every input value is loaded once per 32*TMB output channels.
//   * A lane ends with NPX neighbouring pixels of each channel: stores of 4 or 8 bytes, runs of 128 or 256 bytes.
//   * Biases come from LDS: loaded between the stores they were waited for until the stores ahead of them were done, eight times a
//     wave; a thread's filter vectors are stepped, not divided for (both: 12.2 -> 11.5 us).
// Measured: 64 images of 28x28x256 -> 128 in fp16 (38.5 MB) 11.5 us = 3.3 TB/s, of the 4.7 a large copy reaches, with 64 x 512
// tiles (17.2 us for the best of the other kernels, 32.5 for the one the cost model took).  What is left is start-up: the
// filters' latency, the first groups' latency and the tail of a launch that is little more than one round (two waves or one
// per workgroup, for more workgroups: 13.1 and 13.2 us, before the biases moved).
#pragma once

#include "pwin_kernel.h"

namespace convfwd {

template <int DT_, int TMB_, int NPX_, int GD_>
struct PwbCfg {
    static_assert(DT_ == CONV_F16 || DT_ == CONV_BF16, "16-bit storage only");
    static_assert(NPX_ == 2 || NPX_ == 4, "4- or 8-byte loads");
    static constexpr int DT = DT_, TMB = TMB_, NPX = NPX_, GD = GD_;
    static constexpr int NT = 256;
    static constexpr int TM = 32 * TMB;        // output channels per workgroup
    static constexpr int TNP = 4 * 32 * NPX;   // pixels per workgroup: 32*NPX per wave
    static constexpr int AB = 16;              // staging loads of the filters in flight per thread
};

// filters, then the biases of the tile
inline size_t pwb_lds_bytes(int TM, int C) { return (size_t)TM * (((C + 15) / 16) * 16 + 8) * 2 + (size_t)TM * 4; }

// a.dX divides by the number of channel tiles
template <class CFG>
__global__ __launch_bounds__(CFG::NT, 2) void pwb_kernel(ConvArgs a)
{
    constexpr int DT = CFG::DT, TMB = CFG::TMB, NPX = CFG::NPX, GD = CFG::GD, NT = CFG::NT, TM = CFG::TM, AB = CFG::AB;
    constexpr int W = NPX / 2;  // 32-bit words of a load
    typedef Mma<DT, 32> mma_t;
    extern __shared__ __attribute__((aligned(16))) uint16_t Fs[];

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // ids b, b+8, ... run on one XCD: give each XCD a contiguous run of pixel tiles, the channel tiles of one side by side
    uint32_t pt, mt;
    {
        const int T = (int)gridDim.x, b = blockIdx.x, x = b & 7, per = T >> 3, rem = T & 7;
        a.dX.divmod((uint32_t)(x * per + (x < rem ? x : rem) + (b >> 3)), pt, mt);
    }
    const int m0 = (int)mt * TM, p = (int)pt * CFG::TNP + wave * 32 * NPX + li * NPX;  // this lane's first pixel
    const int G = (a.C + 15) >> 4, C8 = a.C >> 3, pitch = G * 16 + 8;

    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    const __amdgpu_buffer_rsrc_t rfilt = make_rsrc(a.filt, a.filt_bytes);
    uint32_t n, pix;
    a.dHW.divmod((uint32_t)(p < a.P ? p : 0), n, pix);
    // (pixels past the end are pointed beyond the tensor, which stays below 2 GiB: the marker plus any channel offset
    // is out of range too)
    const uint32_t in_off = p < a.P ? (uint32_t)(((int)n * a.C + 8 * g) * a.HW + (int)pix) * 2u : 0x80000000u;
    const uint32_t plane = (uint32_t)a.HW * 2u;

    uint32_t xr[GD][8][W];
    auto load_group = [&](auto slot_c, int grp) {
        constexpr int slot = decltype(slot_c)::value;
        const uint32_t soff = (uint32_t)grp * 16u * plane;
        const uint32_t off = grp * 2 + g < C8 ? in_off : 0x80000000u;  // half a group, or none, behind the last channel
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if constexpr (W == 1) {
                xr[slot][j][0] = __builtin_amdgcn_raw_buffer_load_b32(rin, (int)off, (int)(soff + (uint32_t)j * plane), 0);
            } else {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(rin, (int)off, (int)(soff + (uint32_t)j * plane), 0);
                const uint32_t v0 = v[0], v1 = v[1];
                xr[slot][j][0] = v0;
                xr[slot][j][W - 1] = v1;
            }
        }
    };

    // ---- filters to LDS; the first input groups are requested behind the first batch of filter loads -------------------
    float* const bias_s = (float*)(Fs + TM * pitch);
    const __amdgpu_buffer_rsrc_t rbias = make_rsrc(a.bias, a.bias ? (uint32_t)a.K * 4u : 0u);
    const float bias_r = buffer_load_elem<float>(rbias, tid < TM ? (uint32_t)(m0 + tid) * 4u : kOutOfRange);
    const int vecs = TM * G * 2;  // 16-byte vectors of the tile, channels padded to whole groups with zeros
    // (a thread's vectors are NT apart: rows and columns are stepped, a division each took as long as the loads)
    uint32_t row, c8, row_step, c8_step;
    a.dY.divmod((uint32_t)tid, row, c8);
    a.dY.divmod((uint32_t)NT, row_step, c8_step);
    for (int v0 = 0; v0 < vecs; v0 += AB * NT) {
        uint4 f[AB];
        uint32_t at[AB];
#pragma unroll
        for (int i = 0; i < AB; ++i) {
            const bool ok = row < (uint32_t)TM && m0 + (int)row < a.K && (int)c8 < C8;
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rfilt, (int)(ok ? __umul24(row, (uint32_t)a.C * 2u) + c8 * 16u : 0x80000000u), (int)((uint32_t)(m0 * a.C) * 2u), 0);
            f[i] = make_uint4(v.x, v.y, v.z, v.w);
            at[i] = row < (uint32_t)TM ? __umul24(row, (uint32_t)pitch) + c8 * 8u : kOutOfRange;
            row += row_step, c8 += c8_step;
            if (c8 >= 2u * (uint32_t)G) c8 -= 2u * (uint32_t)G, ++row;
        }
        if (v0 == 0) {
            static_for<GD>([&](auto sc) { load_group(sc, decltype(sc)::value); });
            if (tid < TM) bias_s[tid] = bias_r;
        }
#pragma unroll
        for (int i = 0; i < AB; ++i) {
            if (at[i] != kOutOfRange) *(uint4*)&Fs[at[i]] = f[i];
        }
    }

    typename mma_t::acc_t acc[TMB][NPX];
#pragma unroll
    for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NPX; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.0f;
    __syncthreads();

    const uint16_t* frag = Fs + li * pitch + g * 8;
    // one pass over the ring; in the last, partial one the spare slots are left out (their input is zero, but an infinite
    // filter value times zero would not be)
    auto pass = [&](auto last_c, int grp) {
        constexpr bool LAST = decltype(last_c)::value;
        static_for<GD>([&](auto sc) {
            constexpr int slot = decltype(sc)::value;
            if (LAST && grp + slot >= G) return;
            uint4 b[NPX];
#pragma unroll
            for (int nb = 0; nb < NPX; ++nb) {
                const uint32_t sel = (nb & 1) ? 0x07060302u : 0x05040100u;
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = __builtin_amdgcn_perm(xr[slot][2 * j + 1][nb / 2], xr[slot][2 * j][nb / 2], sel);
                b[nb] = make_uint4(w[0], w[1], w[2], w[3]);
            }
            if constexpr (!LAST) load_group(sc, grp + GD + slot);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mb = 0; mb < TMB; ++mb) {
                const uint4 f = *(const uint4*)(frag + mb * 32 * pitch + (grp + slot) * 16);
#pragma unroll
                for (int nb = 0; nb < NPX; ++nb) acc[mb][nb] = mma_t::run(f, b[nb], acc[mb][nb]);
            }
        });
    };
    int grp = 0;
    for (; grp + GD <= G; grp += GD) pass(std::false_type{}, grp);
    if (grp < G) pass(std::true_type{}, grp);

    // ---- bias + activation + rounding; lane (li, g) holds channels 8i + 4g .. +3 of a block at its NPX pixels -----------
    // (biases from LDS: memory serves a wave in order, and a load between the stores was waited for until those ahead of it were done)
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(a.out, a.out_bytes);
    const uint32_t out_off = (uint32_t)(((int)n * a.K + m0 + 4 * g) * a.HW + (int)pix) * 2u;
    auto store = [&](auto relu_c) {
        auto act = [&](float x) { return decltype(relu_c)::value ? (x > 0.0f ? x : 0.0f) : x; };
#pragma unroll
        for (int mb = 0; mb < TMB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 bs = *(const f32x4*)(bias_s + mb * 32 + 8 * i + 4 * g);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = mb * 32 + 8 * i + r, v = 4 * i + r;
                    const uint32_t o = p < a.P && m0 + row + 4 * g < a.K ? out_off + (uint32_t)row * plane : kOutOfRange;
                    const uint32_t w0 = Prec<DT>::pack2_from_f32(act(acc[mb][0][v] + bs[r]), act(acc[mb][1][v] + bs[r]));
                    if constexpr (NPX == 2) {
                        __builtin_amdgcn_raw_buffer_store_b32(w0, rout, (int)o, 0, 0);
                    } else {
                        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                        const uint32_t w1 = Prec<DT>::pack2_from_f32(act(acc[mb][NPX - 2][v] + bs[r]), act(acc[mb][NPX - 1][v] + bs[r]));
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{w0, w1}, rout, (int)o, 0, 0);
                    }
                }
            }
    };
    if (a.relu)
        store(std::true_type{});
    else
        store(std::false_type{});
}

template <class CFG>
hipError_t pwb_launch(const Variant&, ConvArgs& a, hipStream_t s)
{
    const size_t lds = pwb_lds_bytes(CFG::TM, a.C);
    const hipError_t e = ensure_dynamic_lds((const void*)pwb_kernel<CFG>, lds);
    if (e != hipSuccess) return e;
    const int PT = (a.P + CFG::TNP - 1) / CFG::TNP, MT = (a.K + CFG::TM - 1) / CFG::TM;
    a.dX = make_fastdiv((uint32_t)MT);
    a.dY = make_fastdiv((uint32_t)((a.C + 15) / 16 * 2));
    hipLaunchKernelGGL(pwb_kernel<CFG>, dim3((unsigned)(PT * MT)), dim3(CFG::NT), lds, s, a);
    return hipGetLastError();
}

template <class CFG>
bool pwb_valid(const Variant&, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != CFG::DT || d.R != 1 || d.S != 1 || d.stride != 1 || d.pad != 0) return false;
    if (d.flags & ~(uint32_t)CONV_FLAG_RELU) return false;               // plain formats, no fused pool
    const long long HW = (long long)d.H * d.W, P = HW * d.N;
    if ((d.C % 8) != 0 || (HW % CFG::NPX) != 0) return false;            // rows of filters and pixel groups are aligned
    if (CFG::TM > ((d.K + 31) / 32) * 32 && CFG::TMB > 1) return false;  // an empty channel block only costs time
    if (pwb_lds_bytes(CFG::TM, d.C) > 160 * 1024) return false;
    const long long lim = 1LL << 31;  // 32-bit byte offsets, a look-ahead of GD groups past the last channel included
    if ((long long)d.N * (d.C + 16 * 2 * CFG::GD) * HW * 2 >= lim || P * d.K * 2 >= lim || (long long)d.K * d.C * 2 >= lim) return false;
    return ((P + CFG::TNP - 1) / CFG::TNP) * ((d.K + CFG::TM - 1) / CFG::TM) < lim;
}

template <class CFG>
void pwb_register(std::vector<Variant>& out)
{
    Variant v;
    char buf[160];
    snprintf(buf, sizeof buf, "pwb_%s_M%dN%d_px%d_g%d", dtype_name(CFG::DT), CFG::TM, CFG::TNP, CFG::NPX, CFG::GD);
    v.name = buf;
    v.dtype = CFG::DT;
    v.split = 1;
    v.tm = CFG::TM;
    v.tn = CFG::TNP;
    v.tk = 16;
    v.threads = CFG::NT;
    v.family = FAM_POINTWISE;
    v.specificity = 6;
    v.traits = TRAIT_PIXEL_STREAM;
    v.valid = &pwb_valid<CFG>;
    v.launch = &pwb_launch<CFG>;
    out.push_back(v);
}

template <int DT>
void pwb_register_all(std::vector<Variant>& out)
{
    //                 TMB NPX GD
    pwb_register<PwbCfg<DT, 4, 2, 8>>(out);   // M128 N256
    pwb_register<PwbCfg<DT, 2, 4, 4>>(out);   // M64  N512
    pwb_register<PwbCfg<DT, 2, 2, 8>>(out);   // M64  N256
    pwb_register<PwbCfg<DT, 1, 4, 6>>(out);   // M32  N512
    pwb_register<PwbCfg<DT, 1, 2, 8>>(out);   // M32  N256
}

}  // namespace convfwd
