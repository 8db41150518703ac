// Pieces shared by the kernels that generate X on chip: the low-rank part X[i, j] = sum_r A[i,r] (B[j,r] C[k,r]) of a tile is a
// product on the 16x16x32 matrix instruction with every operand value in two 16-bit pieces.
#pragma once
#include <utility>

#include "exat_mode2.h"

namespace exat {

struct GenSplitParams {
    const __bf16 *Asp;  // [NV][Irows][Rpad] bf16 pieces of A, zero padded (rows >= I and columns >= R)
    int64_t Irows;
    int Rpad;
};

// MFMA 16x16x32 bf16: A lane (row l%16, k 8*(l/16)+e), B lane (col l%16, k 8*(l/16)+e),
// C lane (col l%16, rows 4*(l/16)+r).
typedef float f32x4v __attribute__((ext_vector_type(4)));
// The generator's low-rank product runs on the 16x16x32 matrix instruction with every operand value taken as
// the sum of two 16-bit pieces, v = h + m, and the three significant cross terms accumulated in fp32.
// bf16 plans: bf16 pieces (16 significand bits together, below the bf16 rounding of the tile).
// fp32 plans: fp16 pieces (22 significand bits together; the dropped term is 2^-22 of a product; the factors and
// their products are O(1..100), far inside the fp16 range).  Pieces travel as raw 16-bit patterns in bf16x8
// registers whatever their format.
template <typename T> struct gen_piece;
template <> struct gen_piece<__bf16> {
    static constexpr int FMT = 0;
    __device__ static __forceinline__ void split(float v, __bf16 &h, __bf16 &m)
    {
        h = (__bf16)v;
        m = (__bf16)(v - (float)h);
    }
    __device__ static __forceinline__ f32x4v mfma(const bf16x8 &a, const bf16x8 &b, const f32x4v &c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct gen_piece<float> {
    static constexpr int FMT = 1;
    __device__ static __forceinline__ void split(float v, __bf16 &h, __bf16 &m)
    {
        const _Float16 fh = (_Float16)v;
        const _Float16 fm = (_Float16)(v - (float)fh);
        h = __builtin_bit_cast(__bf16, fh);
        m = __builtin_bit_cast(__bf16, fm);
    }
    __device__ static __forceinline__ f32x4v mfma(const bf16x8 &a, const bf16x8 &b, const f32x4v &c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

template <int... Ms, typename F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, Ms...>, F &&f) { (f(ic<Ms>()), ...); }
// f(ic<0>()), ..., f(ic<N-1>()): a loop whose index is a compile-time constant in the body
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) { static_for_seq(std::make_integer_sequence<int, N>(), f); }

// A (I x R, column-major, fp32) -> the generator's two 16-bit pieces [2][Irows][Rpad] (bf16 pieces for bf16 plans,
// fp16 pieces for fp32 plans), zero padded
template <typename T>
__global__ void k_split_a(const float *A, int64_t I, int R, __bf16 *out, int64_t Irows, int Rpad)
{
    const int64_t n = Irows * Rpad;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = idx / Rpad;
        const int r = (int)(idx % Rpad);
        const float v = (i < I && r < R) ? A[i + I * r] : 0.0f;
        __bf16 h, m;
        gen_piece<T>::split(v, h, m);
        out[idx] = h;
        out[n + idx] = m;
    }
}

}  // namespace exat
