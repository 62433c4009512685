// fp32 operands as sums of three bf16 numbers, for kernels that multiply them on the 16-bit matrix units.
#pragma once

#include "igemm_kernel.h"

namespace convfwd {

constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;  // of either operand, and of the sum of their products

struct Split3 {
    uint4 p[3];
};
// two fp32 values -> three pairs of bf16 that add up to them
__device__ __forceinline__ void split3_pair(float a, float b, uint32_t& w0, uint32_t& w1, uint32_t& w2)
{
    w0 = Prec<CONV_BF16>::pack2_from_f32(a, b);
    a -= __builtin_bit_cast(float, w0 << 16);
    b -= __builtin_bit_cast(float, w0 & 0xffff0000u);
    w1 = Prec<CONV_BF16>::pack2_from_f32(a, b);
    a -= __builtin_bit_cast(float, w1 << 16);
    b -= __builtin_bit_cast(float, w1 & 0xffff0000u);
    w2 = Prec<CONV_BF16>::pack2_from_f32(a, b);
}
// eight fp32 values -> the three MFMA operands
__device__ __forceinline__ Split3 split3(const float* x)
{
    Split3 s;
    uint32_t w[3][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) split3_pair(x[2 * j], x[2 * j + 1], w[0][j], w[1][j], w[2][j]);
#pragma unroll
    for (int q = 0; q < 3; ++q) s.p[q] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
    return s;
}

}  // namespace convfwd
