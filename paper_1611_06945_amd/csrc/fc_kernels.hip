// Fully-connected layers written as convolutions: the window covers the whole input (R == H, S == W, no padding), so
// there is one output pixel per image and
//     out[n][k] = act(bias[k] + sum_q filt[k][q] * in[n][q]),   q = (c, r, s) = the NCHW order of image n.
// The paper lists these layers in its benchmark set (Appendix A: 6x6x256 -> 4096 and 1x1x4096 -> 4096 at batch 5) and
// names them as the outlier its convolution variants do not handle well (Section 4, "Experimental Results").  With a
// handful of images every weight is used only N times: the layer streams the filter tensor once from HBM and is bound
// by that stream, not by arithmetic -- so this kernel is a plain vector-ALU dot product organised around the loads:
//   * a workgroup owns ROWS output channels; its four waves split the reduction axis, every lane walks it with
//     16-byte loads (a wave reads 1 KiB of one filter row per instruction);
//   * the input vectors are read with the same pattern from L2 and reused for all ROWS rows in registers, which keeps
//     the load traffic at (1 + N/ROWS) times the filter bytes;
//   * partial sums are added lane by lane (fixed butterfly order), then wave by wave through LDS: deterministic.
#include "igemm_kernel.h"

namespace convfwd {

namespace {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// acc += dot(w, x) over the VEC elements of one 16-byte vector of each operand, accumulated in fp32.  16-bit pairs go
// through the two-element dot instructions (exact products, fp32 sum), which halves the vector-ALU work per byte.
template <int DT>
struct FcVec;
template <>
struct FcVec<CONV_F32> {
    static constexpr int VEC = 4;
    static __device__ __forceinline__ float mac(const uint4& w, const uint4& x, float acc)
    {
        acc = __builtin_fmaf(__builtin_bit_cast(float, w.x), __builtin_bit_cast(float, x.x), acc);
        acc = __builtin_fmaf(__builtin_bit_cast(float, w.y), __builtin_bit_cast(float, x.y), acc);
        acc = __builtin_fmaf(__builtin_bit_cast(float, w.z), __builtin_bit_cast(float, x.z), acc);
        acc = __builtin_fmaf(__builtin_bit_cast(float, w.w), __builtin_bit_cast(float, x.w), acc);
        return acc;
    }
};
template <>
struct FcVec<CONV_F16> {
    static constexpr int VEC = 8;
    static __device__ __forceinline__ float mac(const uint4& w, const uint4& x, float acc)
    {
        acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w.x), __builtin_bit_cast(f16x2, x.x), acc, false);
        acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w.y), __builtin_bit_cast(f16x2, x.y), acc, false);
        acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w.z), __builtin_bit_cast(f16x2, x.z), acc, false);
        acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w.w), __builtin_bit_cast(f16x2, x.w), acc, false);
        return acc;
    }
};
template <>
struct FcVec<CONV_BF16> {
    static constexpr int VEC = 8;
    static __device__ __forceinline__ float mac(const uint4& w, const uint4& x, float acc)
    {
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.x), __builtin_bit_cast(bf16x2, x.x), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.y), __builtin_bit_cast(bf16x2, x.y), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.z), __builtin_bit_cast(bf16x2, x.z), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.w), __builtin_bit_cast(bf16x2, x.w), acc, false);
        return acc;
    }
};

constexpr int kFcThreads = 256;  // four waves

template <int DT, int ROWS, int NB>
__global__ __launch_bounds__(kFcThreads) void fc_kernel(ConvArgs a)
{
    typedef typename Prec<DT>::elem_t elem_t;
    constexpr int VEC = FcVec<DT>::VEC;
    constexpr uint32_t ES = sizeof(elem_t);
    __shared__ float red[4][ROWS][NB];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k0 = blockIdx.x * ROWS;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    const __amdgpu_buffer_rsrc_t rfilt = make_rsrc(a.filt, a.filt_bytes);

    float acc[ROWS][NB];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[r][n] = 0.0f;

    // byte offsets of this workgroup's filter rows and of the images (rows past K / images past N read as zero)
    uint32_t row_off[ROWS], img_off[NB];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) row_off[r] = (k0 + r < a.K) ? (uint32_t)(k0 + r) * (uint32_t)a.Q * ES : kOutOfRange;
#pragma unroll
    for (int n = 0; n < NB; ++n) img_off[n] = (n < a.N) ? (uint32_t)n * (uint32_t)a.Q * ES : kOutOfRange;

    // the reduction axis in vectors: wave w takes vectors w*64 + lane, + 256, + 512, ...
    const int nvec = a.Q / VEC;
#pragma unroll 2
    for (int v = tid; v < nvec; v += kFcThreads) {
        const uint32_t col = (uint32_t)v * (uint32_t)(VEC * ES);
        uint4 wv[ROWS], xv[NB];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) wv[r] = buffer_load_vec(rfilt, row_off[r] == kOutOfRange ? kOutOfRange : row_off[r] + col);
#pragma unroll
        for (int n = 0; n < NB; ++n) xv[n] = buffer_load_vec(rin, img_off[n] == kOutOfRange ? kOutOfRange : img_off[n] + col);
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[r][n] = FcVec<DT>::mac(wv[r], xv[n], acc[r][n]);
    }

    // lanes of a wave: butterfly over lane distance 32, 16, ..., 1 (the same order in every launch)
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            float x = acc[r][n];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
            acc[r][n] = x;
        }
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int n = 0; n < NB; ++n) red[wave][r][n] = acc[r][n];
    }
    __syncthreads();
    if (tid < ROWS * NB) {
        const int r = tid / NB, n = tid % NB;
        const int k = k0 + r;
        if (k < a.K && n < a.N) {
            float x = ((red[0][r][n] + red[1][r][n]) + red[2][r][n]) + red[3][r][n];
            if (a.bias) x += a.bias[k];
            if (a.relu & 1) x = x > 0.0f ? x : 0.0f;
            ((elem_t*)a.out)[(size_t)n * a.K + k] = Prec<DT>::from_f32(x);
        }
    }
}

template <int DT, int ROWS, int NB>
hipError_t fc_launch(const Variant& v, ConvArgs& a, hipStream_t s)
{
    a.nsplit = 1;
    a.steps_per_split = 0;
    dim3 grid((unsigned)((a.K + ROWS - 1) / ROWS));
    hipLaunchKernelGGL((fc_kernel<DT, ROWS, NB>), grid, dim3(kFcThreads), 0, s, a);
    return hipGetLastError();
}

template <int DT, int ROWS, int NB, int NB_BELOW>
bool fc_valid(const Variant& v, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != DT) return false;
    if (OH != 1 || OW != 1 || d.pad != 0 || d.R != d.H || d.S != d.W) return false;  // the window is the whole image
    const long long Q = (long long)d.C * d.R * d.S;
    if (Q % FcVec<DT>::VEC != 0) return false;              // rows and images start on 16-byte boundaries
    if (d.N > NB || d.N <= NB_BELOW) return false;  // one pass over the weights, in the smallest instantiation that holds N
    if ((long long)d.K > 2147483647LL * ROWS / 2) return false;
    return true;
}

template <int DT, int ROWS, int NB, int NB_BELOW>
void fc_register_one(std::vector<Variant>& out)
{
    Variant v;
    char buf[96];
    snprintf(buf, sizeof buf, "fc_%s_rows%d_n%d", dtype_name(DT), ROWS, NB);
    v.name = buf;
    v.dtype = DT;
    v.split = 1;
    v.tm = ROWS;
    v.tn = NB;
    v.tk = 256 * FcVec<DT>::VEC;
    v.threads = kFcThreads;
    v.family = FAM_FC;
    v.specificity = 6;
    v.valid = &fc_valid<DT, ROWS, NB, NB_BELOW>;
    v.launch = &fc_launch<DT, ROWS, NB>;
    out.push_back(v);
}

// image counts 1, 2, 3-4, 5, 6, 7-8 (5 is the paper's batch); NB_BELOW = the next smaller instantiation
template <int DT, int ROWS>
void fc_register_rows(std::vector<Variant>& out)
{
    fc_register_one<DT, ROWS, 1, 0>(out);
    fc_register_one<DT, ROWS, 2, 1>(out);
    fc_register_one<DT, ROWS, 4, 2>(out);
    fc_register_one<DT, ROWS, 5, 4>(out);
    fc_register_one<DT, ROWS, 6, 5>(out);
    fc_register_one<DT, ROWS, 8, 6>(out);
}
template <int DT>
void fc_register_dtype(std::vector<Variant>& out)
{
    fc_register_rows<DT, 2>(out);
    fc_register_rows<DT, 4>(out);
    fc_register_rows<DT, 8>(out);
}

// More than eight images (or, TAIL, rows that do not start on 16-byte boundaries): the vector-ALU kernel above would multiply for longer than the weights take to arrive, and the
// MFMA tiles of the general kernels are too few to keep the memory busy (128 of 32 rows, each a serial chain of steps).
// Here a workgroup owns 16 output channels and all images; its 16 waves take every 16th step of the reduction (a step is
// 64 bytes of every row, so together they read 1 KB runs), each with DEPTH steps of loads in flight, both operands straight
// from memory into 16x16 MFMA registers: a lane's 16 bytes are 8 (fp32: 4) consecutive reduction elements of one filter row
// or image.  The waves' sums meet in LDS and are added in wave order: deterministic, no workspace, one launch.
// Bound by the stream of the weights (the images come from L2, NB times the weights' traffic at most): 6x6x256 -> 4096 at
// batch 20 in fp16 (75.5 MB) takes 24 us, 16.6 us of which remain without the image loads (16 segments of 64 bytes cost a
// load instruction twice what a contiguous kilobyte does); the best split of the general kernels took 31.9 us, the best
// without a workspace 163.  Layers of few rows split the reduction over four workgroups as well (fp32 partial sums, second
// launch): 51 images, 18032 -> 1000 in fp32 101 -> 37 us.  3 images, 9506 -> 4096 (rows of 38024 bytes) 52 -> 31 us, without a
// workspace 346 -> 31.  3 to 9 steps in flight and a start that differs per workgroup make no difference.
template <int DT, int NB>
struct FcmCfg {
    static constexpr int WAVES = 16, NT = 64 * WAVES;
    static constexpr int VEC = FcVec<DT>::VEC, STEP = 4 * VEC;  // reduction elements per step: 4 lane groups x 16 bytes
    static constexpr int DEPTH = 4;
};

template <int DT, int NB, bool TAIL>
__global__ __launch_bounds__(1024) void fcm_kernel(ConvArgs a)
{
    typedef FcmCfg<DT, NB> CFG;
    typedef typename Prec<DT>::elem_t elem_t;
    typedef Mma<DT, 16> mma_t;
    constexpr int DEPTH = CFG::DEPTH, WAVES = CFG::WAVES;
    constexpr uint32_t ES = sizeof(elem_t);
    __shared__ float red[WAVES][NB * 16][17];

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = blockIdx.x * 16;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    const __amdgpu_buffer_rsrc_t rfilt = make_rsrc(a.filt, a.filt_bytes);

    // byte offsets at this lane's first step; rows past K, images past N and elements past the row's end read as zero
    const int q0 = wave * CFG::STEP + g * CFG::VEC;
    const uint32_t a_off = k0 + li < a.K ? ((uint32_t)(k0 + li) * (uint32_t)a.Q + (uint32_t)q0) * ES : kOutOfRange;
    uint32_t b_off[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) b_off[nb] = nb * 16 + li < a.N ? ((uint32_t)(nb * 16 + li) * (uint32_t)a.Q + (uint32_t)q0) * ES : kOutOfRange;

    constexpr int STRIDE = WAVES * CFG::STEP, kPast = 0x40000000;
    uint4 av[DEPTH], bv[DEPTH][NB];
    auto load = [&](int slot, int i) {
        const bool live = i != kPast && q0 + i * STRIDE < a.Q;
        const uint32_t d = (uint32_t)(i * STRIDE) * ES;
        av[slot] = buffer_load_vec(rfilt, live && a_off != kOutOfRange ? a_off + d : kOutOfRange);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bv[slot][nb] = buffer_load_vec(rin, live && b_off[nb] != kOutOfRange ? b_off[nb] + d : kOutOfRange);
    };
    auto cut = [](uint4 v, int elems) {  // keeps the first `elems` elements (rows hold whole words)
        const int words = elems * (int)ES / 4;
        return make_uint4(words > 0 ? v.x : 0u, words > 1 ? v.y : 0u, words > 2 ? v.z : 0u, words > 3 ? v.w : 0u);
    };
    typename mma_t::acc_t acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = typename mma_t::acc_t{0.0f, 0.0f, 0.0f, 0.0f};
    const int first = (int)blockIdx.y * a.steps_per_split;
    const int steps = (a.Q + STRIDE - 1) / STRIDE, last = first + a.steps_per_split < steps ? first + a.steps_per_split : steps;
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) load(j, first + j < last ? first + j : kPast);
    for (int i = first; i < last; i += DEPTH) {
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (TAIL) {  // the vector that holds a row's end goes on with the next row: cut both operands there
                const int left = a.Q - (q0 + (i + j) * STRIDE);
                if (left > 0 && left < CFG::VEC) {
                    av[j] = cut(av[j], left);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) bv[j][nb] = cut(bv[j][nb], left);
                }
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if constexpr (DT == CONV_F32) {
                    acc[nb] = mma_t::run(__builtin_bit_cast(float, av[j].x), __builtin_bit_cast(float, bv[j][nb].x), acc[nb]);
                    acc[nb] = mma_t::run(__builtin_bit_cast(float, av[j].y), __builtin_bit_cast(float, bv[j][nb].y), acc[nb]);
                    acc[nb] = mma_t::run(__builtin_bit_cast(float, av[j].z), __builtin_bit_cast(float, bv[j][nb].z), acc[nb]);
                    acc[nb] = mma_t::run(__builtin_bit_cast(float, av[j].w), __builtin_bit_cast(float, bv[j][nb].w), acc[nb]);
                } else {
                    acc[nb] = mma_t::run(av[j], bv[j][nb], acc[nb]);
                }
            }
            load(j, i + DEPTH + j < last ? i + DEPTH + j : kPast);
        }
    }
    // lane (li, g): image nb*16 + li, rows 4g .. 4g+3
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][nb * 16 + li][g * 4 + v] = acc[nb][v];
    __syncthreads();
    if (tid < NB * 256) {
        const int r = tid & 15, n = tid >> 4, k = k0 + r;
        if (k < a.K && n < a.N) {
            float x = red[0][n][r];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) x += red[w][n][r];
            if (a.nsplit > 1) {
                a.ws[((size_t)blockIdx.y * a.K + k) * a.P + n] = x;
                return;
            }
            if (a.bias) x += a.bias[k];
            if (a.relu) x = x > 0.0f ? x : 0.0f;
            ((elem_t*)a.out)[(size_t)n * a.K + k] = Prec<DT>::from_f32(x);
        }
    }
}

template <int DT, int NB, bool TAIL>
hipError_t fcm_launch(const Variant& v, ConvArgs& a, hipStream_t s)
{
    constexpr int STRIDE = FcmCfg<DT, NB>::WAVES * FcmCfg<DT, NB>::STEP;
    const int steps = (a.Q + STRIDE - 1) / STRIDE;
    a.nsplit = v.split;
    a.steps_per_split = (steps + v.split - 1) / v.split;
    hipLaunchKernelGGL((fcm_kernel<DT, NB, TAIL>), dim3((unsigned)((a.K + 15) / 16), (unsigned)v.split), dim3(1024), 0, s, a);
    return hipGetLastError();
}

template <int DT, int NB, bool TAIL>
bool fcm_valid(const Variant& v, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != DT) return false;
    if (OH != 1 || OW != 1 || d.pad != 0 || d.R != d.H || d.S != d.W) return false;  // the window is the whole image
    const long long Q = (long long)d.C * d.R * d.S;
    // rows and images start on 16-byte boundaries, or (TAIL) at least on 4-byte ones
    if ((Q % FcVec<DT>::VEC != 0) != TAIL || Q * dtype_size(DT) % 4 != 0) return false;
    constexpr int STRIDE = FcmCfg<DT, NB>::WAVES * FcmCfg<DT, NB>::STEP;
    if (Q > 0x3fffffffLL || (v.split > 1 && (Q + STRIDE - 1) / STRIDE < 4 * v.split)) return false;
    return (TAIL || d.N > 8) && d.N <= NB * 16 && d.N > (NB - 1) * 16;
}

template <int DT, int NB, bool TAIL>
void fcm_register_one(std::vector<Variant>& out, int split)
{
    Variant v;
    char buf[96];
    snprintf(buf, sizeof buf, "fc_%s_mfma_rows16_n%d%s%s", dtype_name(DT), NB * 16, TAIL ? "_t" : "", split > 1 ? "_sk4" : "");
    v.name = buf;
    v.dtype = DT;
    v.split = split;
    v.tm = 16;
    v.tn = NB * 16;
    v.tk = 16 * FcmCfg<DT, NB>::STEP;
    v.threads = 1024;
    v.family = FAM_FC;
    v.specificity = 6;
    v.valid = &fcm_valid<DT, NB, TAIL>;
    v.launch = &fcm_launch<DT, NB, TAIL>;
    out.push_back(v);
}
template <int DT>
void fcm_register_dtype(std::vector<Variant>& out)
{
    for (int split : {1, 4}) {
        fcm_register_one<DT, 1, false>(out, split);
        fcm_register_one<DT, 2, false>(out, split);
        fcm_register_one<DT, 3, false>(out, split);
        fcm_register_one<DT, 4, false>(out, split);
        fcm_register_one<DT, 1, true>(out, split);
        fcm_register_one<DT, 2, true>(out, split);
        fcm_register_one<DT, 3, true>(out, split);
        fcm_register_one<DT, 4, true>(out, split);
    }
}

}  // namespace

void register_fc(std::vector<Variant>& out)
{
    fc_register_dtype<CONV_F32>(out);
    fc_register_dtype<CONV_F16>(out);
    fc_register_dtype<CONV_BF16>(out);
    fcm_register_dtype<CONV_F32>(out);
    fcm_register_dtype<CONV_F16>(out);
    fcm_register_dtype<CONV_BF16>(out);
}

}  // namespace convfwd
