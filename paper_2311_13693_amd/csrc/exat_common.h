// Parameter block and MFMA wrappers shared by the mode-1/2 kernels and their common mode-2 phase.
#pragma once
#include "exat_device.h"

namespace exat {

struct Mode12Params {
    const void *U;   // packed [PLpad][Ipad] of T, zero padded
    const float *V;  // packed [P][Mpad][Jpad] fp32, zero padded (bf16-rounded values for bf16 plans)
    float *Q;        // [k1-k0][PLpad][Mpad] fp32
    // materialised source: element (i,j,k) at X[(i-xo_i) + (j-xo_j)*x_sj + (k-xo_k)*x_sk]
    const void *X;
    int64_t x_sj, x_sk, xo_i, xo_j, xo_k;
    int x_vec;  // 16-byte loads of X are aligned
    // materialised source held as separate blocks: xtab[bi + tab_nbi*(bj + tab_nbj*bk)] is the
    // column-major x_dI x dj x dk block (bi, bj, bk) of X (dj, dk shorter in the last block of an axis); X is unused
    const void *const *xtab;
    int64_t x_dI, x_dJ, x_dK;
    int tab_nbi, tab_nbj;
    // generated source
    const float *A, *B, *C;
    int64_t ldA, ldB, ldC;
    int R, a_vec;  // a_vec: 16-byte loads of A rows are aligned
    uint32_t skey;
    float amp2_ln2;  // -2 ln2 sigma^2, 0 when sigma == 0
    int64_t I, Ipad, Jpad;
    int L, PL, PLpad, Mpad, MT, G;
    int row_base;  // first stacked row of row group 0 of this launch (k_mode12_v3; a multiple of 32, else 0)
    int64_t i0, i1, j0, j1, k0, k1;
    // k_mode12 behind k_mode12_mp: it computes the call only if the noted value ranges say so (mp_out_of_range), and then
    // also clears the rows from qzero0 on of every slice's part of Q (the other wave columns' partial results)
    const uint32_t *guard;
    int qzero0;
};

// Words of MpParams::flags, set where a value lies outside the range in which the piece sums of k_mode12_mp hold: of one call (cleared by
// mode 3), and of the factors.
enum { MPF_X = 0, MPF_Z, MPF_CALL_WORDS, MPF_U = 8, MPF_V, MPF_VNORM, MPF_VNZ, MPF_WORDS = 16 };
// The ranges.  Three bf16 pieces hold a value of at least 2^-102 exactly (the last bit of the last piece is 2^-23 of it, and a normal
// bf16 number is at least 2^-126), and of a sum of products of 2^-100 and more nothing above its rounding is lost; so
//   every element of U and V is 0 or at least MP_EMIN, and V's largest at least MP_VMIN;
//   the X that a wave reads of a slice is 0 throughout or its largest at least MP_EMIN;
//   a row of a slice's Z is 0 throughout or its largest at least MP_ZMIN (MP_ZMIN MP_VMIN = 2^-100).
// Elements of X or Z below 2^-102 beside larger ones of the same slice are held to 2^-126 absolutely, 2^-30 of the largest or less.  At
// the upper end a value only has to be finite in bf16, products of it too; the limits stop far below.
// Measured (70 x 140 x 6, one replica's U or V or one slice of X scaled, error of what comes from it alone): 2.0e-7 down to 1e-32, 2.8e-7
// at 1e-33, 1.9e-6 at 1e-34, 1.9e-4 at 1e-36 with pieces; 2.5e-7 throughout with fp32 products, which take over at 2^-96 (1.3e-29).
constexpr float MP_EMIN = 0x1p-96f, MP_XMAX = 0x1p80f, MP_UMAX = 0x1p40f, MP_VMAX = 0x1p20f, MP_VMIN = 0x1p-20f, MP_ZMAX = 0x1p104f, MP_ZMIN = 0x1p-80f;

// true if the products of the call have to be formed in fp32
__device__ __forceinline__ bool mp_out_of_range(const uint32_t *f)
{
    return (f[MPF_X] | f[MPF_Z] | f[MPF_U] | f[MPF_V]) || (f[MPF_VNZ] && !f[MPF_VNORM]);
}

enum { SRC_MATERIALISED = 0, SRC_GENERATED = 1 };

template <typename T> struct mma_frag;
template <> struct mma_frag<float> {
    typedef f32x4 type;
    __device__ static __forceinline__ void mma(f32x16 &c, const f32x4 &a, const f32x4 &b)
    {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0], b[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[1], b[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[2], b[2], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[3], b[3], c, 0, 0, 0);
    }
};
template <> struct mma_frag<__bf16> {
    typedef bf16x8 type;
    __device__ static __forceinline__ void mma(f32x16 &c, const bf16x8 &a, const bf16x8 &b)
    {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

}  // namespace exat
