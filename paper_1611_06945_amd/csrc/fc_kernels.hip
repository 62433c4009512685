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

// More than eight images (or, TAIL, rows that do not start on 16-byte boundaries): the vector-ALU kernel above would multiply
// for longer than the weights take to arrive, and the MFMA tiles of the general kernels are too few to keep the memory busy
// (128 of 32 rows, each a serial chain of steps).
// Here a workgroup owns 16 output channels and all images; its 16 waves take every 16th step of the reduction (a step is
// 128 bytes of every row), each with DEPTH steps of loads in flight.  The filters go straight from memory into 16x16 MFMA
// registers.  The images come from L2 in whole lines and change lanes in a piece of LDS that only this wave uses, without a
// barrier: loaded as the MFMA wants them (16 rows of 64 bytes an instruction) they cost 33 clocks an instruction, as much
// time as the filters.  The waves' sums meet in LDS and are added in wave order: deterministic, no workspace, one launch.
// Bound by the stream of the weights.  6x6x256 -> 4096 at batch 20 in fp16 (75.5 MB): 16.1 us = 4.7 TB/s (23.5 with the
// images in MFMA order); the best split of the general kernels took 32, the best without a workspace 163.  Layers of few rows
// split the reduction over four workgroups as well (fp32 partial sums, second launch): 51 images, 18032 -> 1000 in fp32 84 ->
// 34 us.  3 images, 9506 -> 4096 (rows of 38024 bytes), without a workspace 346 -> 29.5 us.
template <int DT, int R8>
struct FcmCfg {
    static constexpr int WAVES = 16, NT = 64 * WAVES;
    static constexpr int NB = (R8 + 1) / 2;                     // blocks of 16 images
    static constexpr int VEC = FcVec<DT>::VEC, STEP = 8 * VEC;  // reduction elements per step: 128 bytes of a row
    static constexpr int DEPTH = R8 <= 4 ? 3 : 2;               // steps in flight
    static constexpr int PITCH = 128 + 16;                      // bytes of an image's piece in LDS: 8 rows on distinct banks
    static constexpr size_t X_BYTES = (size_t)WAVES * NB * 16 * PITCH, RED_BYTES = sizeof(float) * WAVES * NB * 16 * 17;
    static constexpr size_t LDS_BYTES = X_BYTES > RED_BYTES ? X_BYTES : RED_BYTES;
};

template <int DT, int R8, bool TAIL>
__global__ __launch_bounds__(1024) void fcm_kernel(ConvArgs a)
{
    typedef FcmCfg<DT, R8> CFG;
    typedef typename Prec<DT>::elem_t elem_t;
    typedef Mma<DT, 16> mma_t;
    constexpr int DEPTH = CFG::DEPTH, WAVES = CFG::WAVES, NB = CFG::NB, VEC = CFG::VEC, STEP = CFG::STEP, PITCH = CFG::PITCH;
    constexpr uint32_t ES = sizeof(elem_t);
    extern __shared__ __attribute__((aligned(16))) unsigned char fcm_lds[];
    typedef float red_t[NB * 16][17];
    red_t* const red = (red_t*)fcm_lds;

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = blockIdx.x * 16;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    const __amdgpu_buffer_rsrc_t rfilt = make_rsrc(a.filt, a.filt_bytes);

    // A step of a wave is 128 bytes of every row.  Filters: lane (li, g) takes vectors g and 4 + g of row li, as the MFMA
    // wants them.  Images: lane l takes vector l % 8 of image 8j + l / 8, whole lines; they change lanes in LDS.  Rows past
    // K, images past N and elements past the row's end read as zero.
    const int w0 = wave * STEP;
    const int qa = w0 + g * VEC, qx = w0 + (lane & 7) * VEC;
    // (both tensors stay below 2 GiB: kFar plus any scalar offset is out of range)
    constexpr uint32_t kFar = 0x80000000u;
    const uint32_t a_off = k0 + li < a.K ? ((uint32_t)(k0 + li) * (uint32_t)a.Q + (uint32_t)qa) * ES : kFar;
    const uint32_t x_off = ((uint32_t)(lane >> 3) * (uint32_t)a.Q + (uint32_t)qx) * ES, x_rows = (uint32_t)a.Q * 8u * ES;
    const bool x_last = (R8 - 1) * 8 + (lane >> 3) < a.N;  // the other groups of eight images are whole

    constexpr int STRIDE = WAVES * STEP, kPast = 0x40000000;
    uint4 av[DEPTH][2], xv[DEPTH][R8];
    auto fetch = [](__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)soff, 0);
        return make_uint4(v.x, v.y, v.z, v.w);
    };
    auto load = [&](int slot, int i) {
        const bool some = i != kPast;
        const uint32_t d = some ? (uint32_t)(i * STRIDE) * ES : 0u;
        const int left = some ? a.Q - i * STRIDE : 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) av[slot][u] = fetch(rfilt, qa + u * 4 * VEC < left ? a_off : kFar, d + u * 64u);
#pragma unroll
        for (int j = 0; j < R8; ++j)
            xv[slot][j] = fetch(rin, qx < left && (j + 1 < R8 || x_last) ? x_off : kFar, d + (uint32_t)j * x_rows);
    };
    // the vector that holds a row's end goes on with the next row: keeps the elements before index a.Q (rows hold whole words)
    auto cut = [&](uint4 v, int q) {
        const int left = a.Q - q;
        if (left <= 0 || left >= VEC) return v;
        const int words = left * (int)ES / 4;
        return make_uint4(v.x, words > 1 ? v.y : 0u, words > 2 ? v.z : 0u, words > 3 ? v.w : 0u);
    };
    unsigned char* const xs = fcm_lds + (size_t)wave * NB * 16 * PITCH;  // this wave's own piece
    unsigned char* const x_dst = xs + (lane >> 3) * PITCH + (lane & 7) * 16;
    const unsigned char* const x_src = xs + li * PITCH + g * 16;
    // lanes read what other lanes of the wave wrote: LDS serves a wave's accesses in order, the compiler must keep theirs
    auto wave_order = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    typename mma_t::acc_t acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = typename mma_t::acc_t{0.0f, 0.0f, 0.0f, 0.0f};
    const int first = (int)blockIdx.y * a.steps_per_split;
    const int steps = (a.Q + STRIDE - 1) / STRIDE, last = first + a.steps_per_split < steps ? first + a.steps_per_split : steps;
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) load(s, first + s < last ? first + s : kPast);
    for (int i = first; i < last; i += DEPTH) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            if constexpr (TAIL) {
#pragma unroll
                for (int u = 0; u < 2; ++u) av[s][u] = cut(av[s][u], qa + u * 4 * VEC + (i + s) * STRIDE);
#pragma unroll
                for (int j = 0; j < R8; ++j) xv[s][j] = cut(xv[s][j], qx + (i + s) * STRIDE);
            }
            wave_order();
#pragma unroll
            for (int j = 0; j < R8; ++j) *(uint4*)(x_dst + j * 8 * PITCH) = xv[s][j];
            wave_order();
            const uint4 f[2] = {av[s][0], av[s][1]};
            load(s, i + DEPTH + s < last ? i + DEPTH + s : kPast);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const uint4 x = *(const uint4*)(x_src + nb * 16 * PITCH + u * 64);
                    if constexpr (DT == CONV_F32) {
                        acc[nb] = mma_t::run(__builtin_bit_cast(float, f[u].x), __builtin_bit_cast(float, x.x), acc[nb]);
                        acc[nb] = mma_t::run(__builtin_bit_cast(float, f[u].y), __builtin_bit_cast(float, x.y), acc[nb]);
                        acc[nb] = mma_t::run(__builtin_bit_cast(float, f[u].z), __builtin_bit_cast(float, x.z), acc[nb]);
                        acc[nb] = mma_t::run(__builtin_bit_cast(float, f[u].w), __builtin_bit_cast(float, x.w), acc[nb]);
                    } else {
                        acc[nb] = mma_t::run(f[u], x, acc[nb]);
                    }
                }
        }
    }
    __syncthreads();  // the images' pieces are dead: the sums overlay them
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

template <int DT, int R8, bool TAIL>
hipError_t fcm_launch(const Variant& v, ConvArgs& a, hipStream_t s)
{
    const hipError_t e = ensure_dynamic_lds((const void*)fcm_kernel<DT, R8, TAIL>, FcmCfg<DT, R8>::LDS_BYTES);
    if (e != hipSuccess) return e;
    constexpr int STRIDE = FcmCfg<DT, R8>::WAVES * FcmCfg<DT, R8>::STEP;
    const int steps = (a.Q + STRIDE - 1) / STRIDE;
    a.nsplit = v.split;
    a.steps_per_split = (steps + v.split - 1) / v.split;
    constexpr size_t lds = FcmCfg<DT, R8>::LDS_BYTES;
    hipLaunchKernelGGL((fcm_kernel<DT, R8, TAIL>), dim3((unsigned)((a.K + 15) / 16), (unsigned)v.split), dim3(1024), lds, s, a);
    return hipGetLastError();
}

template <int DT, int R8, bool TAIL>
bool fcm_valid(const Variant& v, const conv_desc& d, int OH, int OW)
{
    if (d.dtype != DT) return false;
    if (OH != 1 || OW != 1 || d.pad != 0 || d.R != d.H || d.S != d.W) return false;  // the window is the whole image
    const long long Q = (long long)d.C * d.R * d.S;
    // rows and images start on 16-byte boundaries, or (TAIL) at least on 4-byte ones
    if ((Q % FcVec<DT>::VEC != 0) != TAIL || Q * dtype_size(DT) % 4 != 0) return false;
    if ((long long)d.K * Q * dtype_size(DT) >= (1LL << 31) || (long long)d.N * Q * dtype_size(DT) >= (1LL << 31)) return false;
    constexpr int STRIDE = FcmCfg<DT, R8>::WAVES * FcmCfg<DT, R8>::STEP;
    if (Q > 0x3fffffffLL || (v.split > 1 && (Q + STRIDE - 1) / STRIDE < 2 * v.split)) return false;
    return (TAIL || d.N > 8) && d.N <= R8 * 8 && d.N > (R8 - 1) * 8;
}

template <int DT, int R8, bool TAIL>
void fcm_register_one(std::vector<Variant>& out, int split)
{
    Variant v;
    char buf[96];
    snprintf(buf, sizeof buf, "fc_%s_mfma_rows16_n%d%s%s", dtype_name(DT), R8 * 8, TAIL ? "_t" : "", split > 1 ? "_sk4" : "");
    v.name = buf;
    v.dtype = DT;
    v.split = split;
    v.tm = 16;
    v.tn = R8 * 8;
    v.tk = 16 * FcmCfg<DT, R8>::STEP;
    v.threads = 1024;
    v.family = FAM_FC;
    v.specificity = 6;
    v.valid = &fcm_valid<DT, R8, TAIL>;
    v.launch = &fcm_launch<DT, R8, TAIL>;
    out.push_back(v);
}
template <int DT>
void fcm_register_dtype(std::vector<Variant>& out)
{
    for (int split : {1, 4}) {
        fcm_register_one<DT, 2, false>(out, split);
        fcm_register_one<DT, 3, false>(out, split);
        fcm_register_one<DT, 4, false>(out, split);
        fcm_register_one<DT, 5, false>(out, split);
        fcm_register_one<DT, 6, false>(out, split);
        fcm_register_one<DT, 7, false>(out, split);
        fcm_register_one<DT, 8, false>(out, split);
        fcm_register_one<DT, 1, true>(out, split);
        fcm_register_one<DT, 2, true>(out, split);
        fcm_register_one<DT, 3, true>(out, split);
        fcm_register_one<DT, 4, true>(out, split);
        fcm_register_one<DT, 5, true>(out, split);
        fcm_register_one<DT, 6, true>(out, split);
        fcm_register_one<DT, 7, true>(out, split);
        fcm_register_one<DT, 8, true>(out, split);
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
