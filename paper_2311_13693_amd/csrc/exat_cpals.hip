// Batched CP-ALS on the P proxy tensors (paper Alg. 1; Sec. 3 "Decomposition").  Declarations and contracts in
// include/exat.h.
//
// The P problems are independent and small (L, M, N, R <= 64), so latency is what bounds them: a sweep is 3 * 2 L M N R flops per
// replica (1.6 GFLOP at 32 replicas of 64^3, rank 32: 10 us at the fp32 matrix rate) and the rest are short serial steps.  One
// update, e.g. of A, is one launch, k_cpals_step, of NS + 1 workgroups per replica:
//   1. the update before it is finished: the workgroup adds the NS partial MTTKRP results in slab order and multiplies with the inverse
//      of the normal matrix, X = Mx G^{-1}.  Every workgroup of the replica does that for itself (it needs the new factor at once and
//      there is nothing to wait for); the first slab's writes the factor to memory.
//   2. NS workgroups compute their share of this update's MTTKRP, Mx[d0,r] = sum_{d2} (sum_{d1} Y[d0,d1,d2] F1[d1,r]) F2[d2,r], over a
//      slab of the outer contraction index, the inner sum on the bf16 matrix cores with both operands as three bf16 pieces (six of the
//      nine products; what is left out is at most 2^-26 of a product).  F1 is split once.  The inner sum and the pieces need no range record:
//      with Y of the size of A B C, |Y F1| = |F1 F2| |F1 F3| is a root of the product of two normal matrices, so what would leave the range
//      of fp32, or have pieces below the smallest bf16 value (2^-133; a piece is at least 2^-17 of its value), meets a normal matrix that
//      has left it before.  8450 scalings of Y and the start factors by 10^-36 to 10^36: all that worked with fp32 products still do.
//   3. Meanwhile one workgroup forms this update's normal matrix G = (F2^T F2) * (F1^T F1) (Gram matrices on the fp32 matrix cores; G
//      does not depend on the MTTKRP) and inverts it for the next launch.
// The tensor is read where it lies: a lane holds one row of the updated mode, and the order of the contraction indices inside
// a matrix instruction is free, so the first mode reads 128-byte runs along l and the other two 16 bytes of l per lane.
// The normal matrix is inverted by Gauss-Jordan steps without pivoting (it is positive definite; the pivots met are the squared ones of
// its Cholesky factorisation): 256 threads own cyclic blocks of it in registers, a step eliminates four rows and columns, which go through
// LDS, and has one barrier.
// Data, products and sums are fp32, in a fixed order; the inverse and the product with it are fp64.  An inverse rounded to fp32 leaves
// a residual X G - Mx of cond(G) 2^-24 |Mx|, a triangular solve in fp32 one of 2^-24 |Mx|; measured at rank 64, cond(G) = 3.5e4: inverse
// in fp32 1.9e-4, Cholesky factor and two substitutions in fp32 1.7e-7, inverse in fp64 6.5e-8.  The steps wait for LDS and barriers,
// not for arithmetic, so fp64 costs nothing.
// Measured (32 tensors of 64^3, rank 32, ten sweeps, 31 launches): 0.735 ms with the inverse in line in every workgroup, fp32 matrix
// instructions (6 us a launch) and four waves; 0.62 with a workgroup of its own for the inverse, 0.55 with eight waves and 32-bit
// offsets, 0.49 with bf16 pieces, 0.42 with the requests in the order of their use and none under a condition, and with four pivots
// per step (7.2 -> 5 us), 0.385 with a descriptor per outer value in place of scalar offsets (60 to 89 scalars were spilled in the update of
// A).  A launch is now bound by two chains of about 10 us: partial results, product, Gram matrices (4 us), inverse;
// and the tensor's way from the last-level cache (33.5 MB, more than the L2 holds).  Rank 64: 1.34 -> 0.82 ms; 16^3, rank 8: 0.35 -> 0.21.
#include "../../include/exat.h"
#include "exat_lds.h"

#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

constexpr int CP_MAX = 64;   // largest L, M, N and R
constexpr int CP_NS = 8;     // largest number of slabs
constexpr int CP_NW = 8;     // waves per workgroup
constexpr int CP_NT = 64 * CP_NW;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef double f64_a4 __attribute__((aligned(4)));    // the workspace starts at a multiple of 4 bytes
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));   // rows of Y start at multiples of 4 bytes

struct CpStep {
    const float *Y;         // per replica Y[l + L(m + M n)]
    float *F[3];            // A, B, C, per replica column-major D x R
    const float *pin;       // [replica][NSin][d][R]: partial MTTKRP results of the update before this one; replicas `rs` floats apart
    float *pout;            // the same of this update
    int64_t rs;             // the same for every update, whatever its extent: a replica overwrites its own partial results only
    int D[3];               // L, M, N
    int R, NSin, DS;        // slabs of the update before; values of the outer contraction index per slab of this one
    int prev, mode;         // updated factor of the update before and of this one (0, 1, 2), or -1: none
    int32_t *status;        // optional, [replica]: incremented by every update whose normal matrix has a non-positive pivot
    const f64_a4 *gin;      // [replica][16 NB][16 NB]: inverse of the normal matrix of the update before this one
    f64_a4 *gout;           // the same of this update
};

// 1/x to within an ulp or two: the hardware's estimate (more than 20 bits) and two Newton steps.  The pivots come from fp32 values, far
// inside the range of fp64; a zero gives NaN.
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}

// Inverse of the normal matrix G = (F2^T F2) * (F1^T F1) of the factors Fa and Fb, as g[a][b] = element (ty + 16 a, tx + 16 b) of thread
// 16 ty + tx, zero beyond R; the first 256 threads hold it.  All threads call it; `bad` is set if a pivot is not positive.
template <int RC, int NB>
__device__ __forceinline__ bool invert_normal(const float *Fa, const float *Fb, float (*Gt)[1024], float *G, double (*rowb)[64][4], double (*colb)[64][4],
                                              int R, int tid, int w, double (&g)[NB][NB])
{
    constexpr int RS = 32 * RC, RSP = RS + 1;
    const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    // Gram matrices, one 32 x 32 tile of one of them (one tile only: a quarter of its contraction) per job, jobs to the waves in turn
    constexpr int KH = CP_NW / (2 * RC * RC);
    {
        const int t = w / (2 * KH), kh = w % KH;
        const float *F = ((w / KH) & 1 ? Fb : Fa) + kh * (CP_MAX / KH) * RSP + hi * RSP;
        const int ri = 32 * (t / RC) + l32, ci = 32 * (t % RC) + l32;
        f32x16 gt[2];
#pragma unroll
        for (int e = 0; e < 16; e++) gt[0][e] = gt[1][e] = 0.0f;
#pragma unroll
        for (int s = 0; s < CP_MAX / 2 / KH; s++)
            gt[s & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(F[2 * s * RSP + ri], F[2 * s * RSP + ci], gt[s & 1], 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; e++) Gt[w][e * 64 + lane] = gt[0][e] + gt[1][e];
    }
    lds_barrier();
    for (int e = tid; e < RC * RC * 1024; e += CP_NT) {
        const int t = e >> 10, x = e & 1023, r = x >> 6, l = x & 63;
        float g1 = Gt[2 * KH * t][x], g2 = Gt[2 * KH * t + KH][x];
#pragma unroll
        for (int k = 1; k < KH; k++) { g1 += Gt[2 * KH * t + k][x]; g2 += Gt[2 * KH * t + KH + k][x]; }
        G[(32 * (t / RC) + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3)) * RSP + 32 * (t % RC) + (l & 31)] = g1 * g2;
    }
    lds_barrier();
    // Gi <- G^{-1}, in fp64: thread (ty, tx) owns the entries (ty + 16 a, tx + 16 b), extended by the identity beyond R.  A step
    // eliminates four rows and columns, in the order and with the pivots of four single steps.  Four waves do it, the others keep step.
    const bool act = w < 4;
    const int ty = (tid >> 4) & 15, tx = tid & 15;
#pragma unroll
    for (int a = 0; a < NB; a++)
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const int i = ty + 16 * a, c = tx + 16 * b;
            g[a][b] = (i == c && i >= R) ? 1.0 : (double)G[i * RSP + c];
        }
    bool bad = false;   // the same in every thread: all see the same pivots
    double er[4], ec[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        er[k] = (ty & 3) == k ? -1.0 : 0.0;
        ec[k] = (tx & 3) == k ? 1.0 : 0.0;
    }
#pragma unroll
    for (int jb = 0; jb < NB; jb++)
        for (int jt = 0; jt < 16; jt += 4) {
            const int j = 16 * jb + jt, par = (jt >> 2) & 1;
            if (j >= R) break;
            const bool rin = (ty & 12) == jt, cin = (tx & 12) == jt;
            if (act && cin) {
#pragma unroll
                for (int a = 0; a < NB; a++) colb[par][ty + 16 * a][tx & 3] = g[a][jb];
            }
            if (act && rin) {
#pragma unroll
                for (int b = 0; b < NB; b++) rowb[par][tx + 16 * b][ty & 3] = g[jb][b];
            }
            lds_barrier();
            if (!act) continue;
            // the pivot block is symmetric up to rounding: its upper triangle
            const double a00 = rowb[par][j][0], a01 = rowb[par][j + 1][0], a11 = rowb[par][j + 1][1], b00 = rowb[par][j + 2][0],
                         b01 = rowb[par][j + 3][0], b10 = rowb[par][j + 2][1], b11 = rowb[par][j + 3][1], d00 = rowb[par][j + 2][2],
                         d01 = rowb[par][j + 3][2], d11 = rowb[par][j + 3][3];
            double f[NB][4], q[NB][4];
#pragma unroll
            for (int a = 0; a < NB; a++)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    f[a][k] = colb[par][ty + 16 * a][k];
                    q[a][k] = rowb[par][tx + 16 * a][k];
                }
            // its inverse, by every thread for itself, in 2 x 2 blocks: [A B; B^T D], T = A^-1 B, S = D - B^T T, U = T S^-1,
            // [A^-1 + U T^T, -U; -U^T, S^-1].  The squared Cholesky pivots are a00, det A / a00, s00 and det S / s00.
            const double da = fma(a00, a11, -a01 * a01), ia = recip(da), x00 = a11 * ia, x01 = -a01 * ia, x11 = a00 * ia;
            const double t00 = fma(x00, b00, x01 * b10), t01 = fma(x00, b01, x01 * b11), t10 = fma(x01, b00, x11 * b10), t11 = fma(x01, b01, x11 * b11);
            const double s00 = fma(-b00, t00, fma(-b10, t10, d00)), s01 = fma(-b00, t01, fma(-b10, t11, d01)), s11 = fma(-b01, t01, fma(-b11, t11, d11));
            const double ds = fma(s00, s11, -s01 * s01), is = recip(ds), y00 = s11 * is, y01 = -s01 * is, y11 = s00 * is;
            const double u00 = fma(t00, y00, t01 * y01), u01 = fma(t00, y01, t01 * y11), u10 = fma(t10, y00, t11 * y01), u11 = fma(t10, y01, t11 * y11);
            const double z00 = fma(u00, t00, fma(u01, t01, x00)), z01 = fma(u00, t10, fma(u01, t11, x01)), z11 = fma(u10, t10, fma(u11, t11, x11));
            const double pv[4][4] = {{z00, z01, -u00, -u01}, {z01, z11, -u10, -u11}, {-u00, -u10, y00, y01}, {-u01, -u11, y01, y11}};
            // zero, negative or NaN: not positive definite
            bad = bad || !(a00 > 0.0) || (j + 1 < R && !(da > 0.0)) || (j + 2 < R && !(s00 > 0.0)) || (j + 3 < R && !(ds > 0.0));
            // rows outside the block: g - F P^-1 Q, in its columns -F P^-1; its rows: P^-1 Q and P^-1.  With minus the identity for F in its
            // rows, the identity for Q in its columns and zero for g in both this is one formula.
#pragma unroll
            for (int k = 0; k < 4; k++) {
                f[jb][k] = rin ? er[k] : f[jb][k];
                q[jb][k] = cin ? ec[k] : q[jb][k];
            }
#pragma unroll
            for (int a = 0; a < NB; a++) {
                double wv[4];
#pragma unroll
                for (int k = 0; k < 4; k++)
                    wv[k] = fma(f[a][3], pv[3][k], fma(f[a][2], pv[2][k], fma(f[a][1], pv[1][k], f[a][0] * pv[0][k])));
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    double base = g[a][b];
                    if (a == jb) base = rin ? 0.0 : base;
                    if (b == jb) base = cin ? 0.0 : base;
                    g[a][b] = fma(-wv[3], q[b][3], fma(-wv[2], q[b][2], fma(-wv[1], q[b][1], fma(-wv[0], q[b][0], base))));
                }
            }
        }
#pragma unroll
    for (int a = 0; a < NB; a++)
#pragma unroll
        for (int b = 0; b < NB; b++)
            if (ty + 16 * a >= R || tx + 16 * b >= R) g[a][b] = 0.0;
    return bad;
}

// Element i of an array whose start is the same in all lanes: one 32-bit offset per lane, no 64-bit address arithmetic on the vector unit
__device__ __forceinline__ float at(const float *base, int i) { return *(const float *)((const char *)base + 4u * (unsigned)i); }

// eight fp32 values as three bf16 pieces each, x = h + m + l, in operand order: exact (three times eight significand bits) from 2^-110,
// where the last bit of l is the smallest bf16 value, up to the largest bf16 value, 3.39e38, above which h is infinite
__device__ __forceinline__ void split8(const float *x, u32x4 (&w)[3])
{
#pragma unroll
    for (int i = 0; i < 4; i++) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int q = 0; q < 3; q++) {
            typedef float f2 __attribute__((ext_vector_type(2)));
            w[q][i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), bf16x2));   // one packed conversion
            if (q < 2) {   // the residual of a rounding to bf16 is exact in fp32
                a -= __builtin_bit_cast(float, w[q][i] << 16);
                b -= __builtin_bit_cast(float, w[q][i] & 0xffff0000u);
            }
        }
    }
}
__device__ __forceinline__ f32x16 mma(const u32x4 &a, const u32x4 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// RC = 32-column tiles of the rank, NB = 16-wide blocks of it (R <= 16 NB, NB <= 2 RC)
// U: the factor that is updated (in the launch behind the last update: 0).
template <int RC, int NB, bool OWN, int U>
__global__ __launch_bounds__(CP_NT) void k_cpals_step(const CpStep p)
{
    constexpr int RS = 32 * RC, RSP = RS + 1;
    __shared__ float Fs[3][CP_MAX * RSP];     // factors as [d][r], zero beyond D and R
    __shared__ float Mx[CP_MAX * RSP];        // MTTKRP result of the update before
    __shared__ float G[RS * RSP];             // normal matrix
    __shared__ __align__(16) float Gt[CP_NW][1024];   // tiles of the Gram matrices, the inverse of the normal matrix, partial tiles
    double *Gi = (double *)&Gt[0][0];         // [r][c ^ 16 (r & 1)]: neighbouring rows 32 banks apart
    static_assert(RS * RS * 8 <= CP_NW * 4096, "");
    __shared__ __align__(16) double rowb[2][64][4], colb[2][64][4];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t rep = blockIdx.x;
    // unless every workgroup inverts for itself (OWN), the first one of a replica does nothing else
    const bool inv = !OWN && p.mode >= 0 && blockIdx.y == 0;
    const int slab = !OWN && p.mode >= 0 ? (int)blockIdx.y - 1 : (int)blockIdx.y, R = p.R;
    constexpr int RB = 16 * NB;
    auto put_gi = [&](int i, int c, double x) { Gi[i * RS + (c ^ (16 * (i & 1)))] = x; };

    // ---- this workgroup's share of the MTTKRP.  Mode 0: rows l, inner m, outer n; mode 1: rows m, inner l, outer n; mode 2:
    //      rows n, inner l, outer m.  Tile (rt, ct) of the result to wave w mod ntile; the waves of a tile take the values of
    //      the outer index in turn ----
    constexpr int i1 = U == 0 ? 1 : 0, i2 = U == 2 ? 1 : 2;
    const int Du = p.D[U], D1 = p.D[i1], D2 = p.D[i2];
    const int rtn = (Du + 31) / 32, ntile = rtn * RC, kgn = CP_NW / ntile, kg = w / ntile, tile = w % ntile;
    const int row = 32 * (tile / RC) + l32, c = 32 * (tile % RC) + l32;
    // Element (row, d1, d2) of the tensor: each value d2 of the outer index is a buffer of its own, from its first element to the end of the
    // replica (mode 0: of the slice, where the inner index ends too), and a lane's offset.  Every request is made, in a buffer of no bytes or
    // at the offset NONE where there is nothing to read (it reads nothing then): a request under a condition makes the compiler wait for all
    // that are outstanding.  The range check is relied on for the lane's offset alone, the scalar offset is zero everywhere.
    constexpr int NONE = 1 << 30;
    const bool none = p.mode < 0 || inv;
    const int L4 = 4 * p.D[0], LM = p.D[0] * p.D[1], su = U == 0 ? 1 : (U == 1 ? p.D[0] : LM), s2 = U == 2 ? p.D[0] : LM;
    const float *yr = p.Y + rep * LM * p.D[2];
    const int roh = 4 * (row < Du ? row : Du - 1) * su + (U == 0 ? L4 : 16) * hi;
    constexpr int NSTEP = CP_MAX / 2;
    const int nj = (D1 + 15) / 16;         // groups of 16 inner indices
    const int d2a = none ? 0 : slab * p.DS, d2e = d2a + p.DS < D2 ? d2a + p.DS : D2, d2b = none ? 0 : d2e;
    auto load = [&](int d2, f32x4 (&a)[NSTEP / 4]) __attribute__((always_inline)) {
        const int f = d2 < d2b ? d2 * s2 : 0, bytes = U == 0 ? 4 * LM : 4 * (LM * p.D[2] - f);
        const auto yb = __builtin_amdgcn_make_buffer_rsrc((void *)(yr + f), 0, d2 < d2b ? bytes : 0, 0x00020000);
        int vo = roh;
        if (U == 0) asm("" : "+v"(vo));    // the offsets of a slice are made here, one after the other: 32 registers otherwise
#pragma unroll
        for (int q = 0; q < NSTEP / 4; q++) {
            if constexpr (U == 0) {
#pragma unroll
                for (int e = 0; e < 4; e++) {   // inner index 8 q + 2 e + hi: beyond D1 past the slice
                    a[q][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(yb, vo, 0, 0));
                    vo += 2 * L4;
                }
            } else   // four values of l at 8 q + 4 hi: beyond D1 there are the row's neighbours, which `mac` takes out
                a[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(yb, 8 * q < D1 ? vo + 32 * q : NONE, 0, 0));
        }
    };
    constexpr int PF = 2;
    f32x4 ya[PF][NSTEP / 4];
    // Requests in the order of their use: the factors that are fixed in the update before this one (without one: in this update), that
    // update's inverse and the slabs' partial results, then the wave's first PF values of the outer index, most of whose way is gone
    // when the update before is finished.  All of them are made at clamped addresses and masked afterwards.
    const int v = U == 0 && p.prev < 0 ? 0 : (U + 2) % 3;
    const int f1 = v == 0 ? 1 : 0, f2 = v == 2 ? 1 : 2, D0 = p.D[v], st = D0 * R;
    constexpr int FE = CP_MAX * RS / CP_NT, GE = RB * RB < CP_NT ? 1 : RB * RB / CP_NT;
    const float *psrc = p.pin + rep * p.rs;
    auto poff = [&](int x) {
        const int e = tid + CP_NT * x, d = e / RS, r = e % RS;
        return (d < D0 ? d : D0 - 1) * R + (r < R ? r : R - 1);
    };
    float tf[2][FE], tp[FE][CP_NS];
    double gl[GE];
#pragma unroll
    for (int q = 0; q < 2; q++) {
        const int f = q ? f2 : f1, D = p.D[f];
        const float *src = p.F[f] + rep * D * R;
#pragma unroll
        for (int x = 0; x < FE; x++) {
            const int e = tid + CP_NT * x, d = e % CP_MAX, r = e / CP_MAX;
            tf[q][x] = at(src, (d < D ? d : D - 1) + D * (r < R ? r : R - 1));
        }
    }
    if constexpr (!OWN) {
        const f64_a4 *src = p.gin + rep * (RB * RB);
#pragma unroll
        for (int x = 0; x < GE; x++) gl[x] = src[(tid + CP_NT * x) % (RB * RB)];
    }
#pragma unroll
    for (int x = 0; x < FE; x++)
#pragma unroll
        for (int sl = 0; sl < CP_NS; sl++) tp[x][sl] = at(psrc + (sl < p.NSin ? sl : p.NSin - 1) * st, poff(x));
#pragma unroll
    for (int i = 0; i < PF; i++) load(d2a + kg + i * kgn, ya[i]);
#pragma unroll
    for (int q = 0; q < 2; q++) {
        const int f = q ? f2 : f1, D = p.D[f];
#pragma unroll
        for (int x = 0; x < FE; x++) {
            const int e = tid + CP_NT * x, d = e % CP_MAX, r = e / CP_MAX;
            Fs[f][d * RSP + r] = (d < D && r < R) ? tf[q][x] : 0.0f;
        }
    }

    if (p.prev >= 0) {
        // MTTKRP result: the slabs' partial results in slab order
#pragma unroll
        for (int x = 0; x < FE; x++) {
            float sum = 0.0f;
#pragma unroll
            for (int sl = 0; sl < CP_NS; sl++) sum += sl < p.NSin ? tp[x][sl] : 0.0f;
            const int e = tid + CP_NT * x, d = e / RS, r = e % RS;
            Mx[d * RSP + r] = (d < D0 && r < R) ? sum : 0.0f;
        }
        if constexpr (OWN) {
            lds_barrier();
            double gi[NB][NB];
            const bool bad = invert_normal<RC, NB>(Fs[f1], Fs[f2], Gt, G, rowb, colb, R, tid, w, gi);
            if (bad && tid == 0 && slab == 0 && p.status) p.status[rep] += 1;   // launches on one stream: nothing else touches this word now
            lds_barrier();
#pragma unroll
            for (int a = 0; a < NB; a++)
#pragma unroll
                for (int b = 0; b < NB; b++)
                    if (tid < 256) put_gi((tid >> 4) + 16 * a, (tid & 15) + 16 * b, gi[a][b]);
        } else {
#pragma unroll
            for (int x = 0; x < GE; x++)
                if (tid < RB * RB) put_gi((tid + CP_NT * x) / RB, (tid + CP_NT * x) % RB, gl[x]);
        }
        lds_barrier();
        // X = Mx G^{-1}, accumulated in fp64: 16 x 16 tile (rt, ct) to wave (rt NB + ct) mod CP_NW
        const int rtn = (D0 + 15) / 16, l16 = lane & 15, q16 = lane >> 4;
        for (int t = w; t < rtn * NB; t += CP_NW) {
            const int row = 16 * (t / NB) + l16, c = 16 * (t % NB) + l16;
            float mx[4 * NB];
            double gx[4 * NB];
#pragma unroll
            for (int s = 0; s < 4 * NB; s++) {
                const int k = 4 * s + q16;
                mx[s] = Mx[row * RSP + k];
                gx[s] = Gi[k * RS + (c ^ (16 * (k & 1)))];
            }
            f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * NB; s++) x = __builtin_amdgcn_mfma_f64_16x16x4f64((double)mx[s], gx[s], x, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int d = 16 * (t / NB) + 4 * e + q16;
                const float xf = (float)x[e];
                Fs[v][d * RSP + c] = (d < D0 && c < R) ? xf : 0.0f;
                if (slab == 0 && d < D0 && c < R) p.F[v][rep * D0 * R + d + (int64_t)D0 * c] = xf;
            }
        }
        // the unused row tiles, and the columns beyond the blocks of the rank
        for (int e = tid + 16 * rtn * RS; e < CP_MAX * RS; e += CP_NT) Fs[v][(e / RS) * RSP + e % RS] = 0.0f;
        if (16 * NB < RS)
            for (int e = tid; e < 16 * rtn * (RS - 16 * NB); e += CP_NT) Fs[v][(e / (RS - 16 * NB)) * RSP + 16 * NB + e % (RS - 16 * NB)] = 0.0f;
    }
    if (p.mode < 0) return;
    lds_barrier();
    if (!OWN && inv) {
        double gi[NB][NB];
        const bool bad = invert_normal<RC, NB>(Fs[i1], Fs[i2], Gt, G, rowb, colb, R, tid, w, gi);
        if (bad && tid == 0 && p.status) p.status[rep] += 1;   // launches on one stream: nothing else touches this word now
        f64_a4 *dst = p.gout + rep * (RB * RB);
#pragma unroll
        for (int a = 0; a < NB; a++)
#pragma unroll
            for (int b = 0; b < NB; b++)
                if (tid < 256) dst[((tid >> 4) + 16 * a) * RB + (tid & 15) + 16 * b] = gi[a][b];
        return;
    }

    // inner index of step s, lane half hi: mode 0: 2s + hi; else 8 (s/4) + 4 hi + s%4 (a lane's 16 bytes)
    float b1[NSTEP];
    const float *b1s = Fs[i1] + c + (U == 0 ? hi : 4 * hi) * RSP;
    if constexpr (U == 0) {
#pragma unroll
        for (int s = 0; s < NSTEP; s++) b1[s] = b1s[2 * s * RSP];
    } else {
#pragma unroll
        for (int s = 0; s < NSTEP; s++) b1[s] = b1s[(8 * (s >> 2) + (s & 3)) * RSP];
    }
    u32x4 bp[CP_MAX / 16][3];
#pragma unroll
    for (int j = 0; j < CP_MAX / 16; j++) split8(&b1[8 * j], bp[j]);
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.0f;
    // one value of the outer index: the product over the inner one, smallest terms first, then its factor
    auto mac = [&](int d2, const f32x4 (&a)[NSTEP / 4]) __attribute__((always_inline)) {
        const float f2 = Fs[i2][d2 * RSP + c];
        f32x16 t;
#pragma unroll
        for (int e = 0; e < 16; e++) t[e] = 0.0f;
#pragma unroll
        for (int j = 0; j < CP_MAX / 16; j++) {
            if (j < nj) {
                u32x4 ap[3];
                float av[8] = {a[2 * j][0], a[2 * j][1], a[2 * j][2], a[2 * j][3], a[2 * j + 1][0], a[2 * j + 1][1], a[2 * j + 1][2], a[2 * j + 1][3]};
                if (U != 0 && 16 * j + 16 > D1) {
#pragma unroll
                    for (int e = 0; e < 8; e++) av[e] = 16 * j + 8 * (e >> 2) + 4 * hi + (e & 3) < D1 ? av[e] : 0.0f;
                }
                split8(av, ap);
                t = mma(ap[2], bp[j][0], t);
                t = mma(ap[0], bp[j][2], t);
                t = mma(ap[1], bp[j][1], t);
                t = mma(ap[1], bp[j][0], t);
                t = mma(ap[0], bp[j][1], t);
                t = mma(ap[0], bp[j][0], t);
            }
        }
#pragma unroll
        for (int e = 0; e < 16; e++) acc[e] += f2 * t[e];
    };
    for (int d2 = d2a + kg; d2 < d2b; d2 += PF * kgn) {
#pragma unroll
        for (int i = 0; i < PF; i++) {
            if (d2 + i * kgn < d2b) mac(d2 + i * kgn, ya[i]);
            load(d2 + (i + PF) * kgn, ya[i]);
        }
    }
    // the waves of a tile add up in wave order; the inverse is not needed any more
    if (kg > 0) {
#pragma unroll
        for (int e = 0; e < 16; e++) Gt[(kg - 1) * ntile + tile][e * 64 + lane] = acc[e];
    }
    lds_barrier();
    if (kg == 0) {
        for (int k = 0; k < kgn - 1; k++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[e] += Gt[k * ntile + tile][e * 64 + lane];
        float *dst = p.pout + rep * p.rs + (int64_t)slab * Du * R;
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int d = 32 * (tile / RC) + 8 * (e >> 2) + 4 * hi + (e & 3);
            if (d < Du && c < R) dst[d * R + c] = acc[e];
        }
    }
}

// workspace: slabs of 64 x 64 values per replica
inline int slabs_for(int D2, int P)
{
    int ns = (1024 + P - 1) / P;
    return ns < 1 ? 1 : (ns > D2 ? D2 : ns);
}

}  // namespace

extern "C" {

int64_t exat_cpals_workspace_floats(int32_t L, int32_t M, int32_t N, int32_t P)
{
    if (L < 1 || M < 1 || N < 1 || P < 1) return 0;
    // the slabs' partial MTTKRP results, double-buffered, need slabs_for x 64 x 64 values per replica at most; the call documents
    // the larger figure (room for two copies of Y)
    const int maxd = L > M ? (L > N ? L : N) : (M > N ? M : N);
    return 2 * (int64_t)L * M * N * P + (int64_t)P * slabs_for(maxd, P) * CP_MAX * CP_MAX;
}

__global__ void k_cpals_clear_status(int32_t *status, int P)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < P) status[t] = 0;
}

int exat_cpals(const float *Y, int32_t L, int32_t M, int32_t N, int32_t P, int32_t R, int32_t sweeps, float *A, float *B,
               float *C, float *work, void *stream)
{
    return exat_cpals_checked(Y, L, M, N, P, R, sweeps, A, B, C, work, nullptr, stream);
}

int exat_cpals_checked(const float *Y, int32_t L, int32_t M, int32_t N, int32_t P, int32_t R, int32_t sweeps, float *A, float *B,
                       float *C, float *work, int32_t *status, void *stream)
{
    if (!Y || !A || !B || !C || !work) return EXAT_ERR_NULL;
    if (L < 1 || M < 1 || N < 1 || R < 1 || P < 1 || sweeps < 0) return EXAT_ERR_SHAPE;
    if (L > CP_MAX || M > CP_MAX || N > CP_MAX || R > CP_MAX || P > (1 << 20)) return EXAT_ERR_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    if (status) {   // a fill kernel, not a memset: the call may be recorded into a graph
        hipLaunchKernelGGL(k_cpals_clear_status, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, status, P);
        if (hipGetLastError() != hipSuccess) return EXAT_ERR_HIP;
    }
    if (sweeps == 0) return EXAT_OK;
    // Slabs per replica: one workgroup per compute unit with the one that inverts (two do not fit), and no more than CP_NS: the partial
    // results of all slabs are requested at once, and beyond eight the inverse takes longer than a slab (8 tensors of 64^3, rank 32:
    // 0.375 ms with 16 and with 8; 16 of 32^3, rank 16: 0.278, 0.261).  The partial results and the
    // inverses are double-buffered: a workgroup that is ahead writes while others still read.
    // Every workgroup inverts for itself where a replica has a single one (more than 128 replicas; one workgroup that does both keeps
    // the compute unit as busy as two and finishes the update before once: 1000 tensors of 16^3, rank 16: 1.69 -> 1.26 ms, 130 of 64^3, rank
    // 32: 1.37 -> 1.27; at rank 64 the other way round, 300 of 64^3: 5.08, 5.56), which then has read its partial results before it writes
    // there; and for tiny tensors of high rank, where the workspace has no room for the inverses.
    const int maxd = L > M ? (L > N ? L : N) : (M > N ? M : N);
    int NS = 256 / P - 1;
    NS = NS > CP_NS ? CP_NS : (NS < 1 ? 1 : NS);
    const int64_t room = (int64_t)slabs_for(maxd, P) * CP_MAX * CP_MAX, one = (int64_t)maxd * R;
    while (NS > 1 && 2 * NS * one > room) NS--;
    const int64_t RB = R <= 16 ? 16 : (R <= 32 ? 32 : 64);
    const bool own = (P > 128 && R <= 32) || 2 * NS * one + 4 * RB * RB > 2 * (int64_t)L * M * N + room;
    float *part[2] = {work, own && NS == 1 ? work : work + (int64_t)P * NS * one};
    f64_a4 *ginv[2] = {(f64_a4 *)(work + 2 * P * NS * one), (f64_a4 *)(work + 2 * P * NS * one) + P * RB * RB};
    CpStep c;
    c.Y = Y; c.F[0] = A; c.F[1] = B; c.F[2] = C; c.D[0] = L; c.D[1] = M; c.D[2] = N; c.R = R; c.rs = NS * one; c.status = status;
    c.NSin = 1; c.prev = -1;
    auto launch = [&](int ns, bool inverse) {
        const dim3 grid((unsigned)P, (unsigned)(ns + (inverse && !own ? 1 : 0)));
        const int u = c.mode < 0 ? 0 : c.mode;
        auto go = [&](auto k0, auto k1, auto k2) { hipLaunchKernelGGL(u == 0 ? k0 : u == 1 ? k1 : k2, grid, dim3(CP_NT), 0, st, c); };
        if (own && R <= 16) go(k_cpals_step<1, 1, true, 0>, k_cpals_step<1, 1, true, 1>, k_cpals_step<1, 1, true, 2>);
        else if (own && R <= 32) go(k_cpals_step<1, 2, true, 0>, k_cpals_step<1, 2, true, 1>, k_cpals_step<1, 2, true, 2>);
        else if (own) go(k_cpals_step<2, 4, true, 0>, k_cpals_step<2, 4, true, 1>, k_cpals_step<2, 4, true, 2>);
        else if (R <= 16) go(k_cpals_step<1, 1, false, 0>, k_cpals_step<1, 1, false, 1>, k_cpals_step<1, 1, false, 2>);
        else if (R <= 32) go(k_cpals_step<1, 2, false, 0>, k_cpals_step<1, 2, false, 1>, k_cpals_step<1, 2, false, 2>);
        else go(k_cpals_step<2, 4, false, 0>, k_cpals_step<2, 4, false, 1>, k_cpals_step<2, 4, false, 2>);
    };
    // A <- Y_(1) (C kr B) [(C^T C) * (B^T B)]^-1, then B <- Y_(2) (C kr A) [..]^-1, then C <- Y_(3) (B kr A) [..]^-1: the launch of an
    // update finishes the one before it
    for (int t = 0; t < 3 * sweeps; t++) {
        c.mode = t % 3;
        const int D2 = c.mode == 2 ? M : N;
        int ns = NS < D2 ? NS : D2;
        c.DS = (D2 + ns - 1) / ns;
        ns = (D2 + c.DS - 1) / c.DS;
        c.pin = part[(t + 1) & 1]; c.pout = part[t & 1];
        c.gin = ginv[(t + 1) & 1]; c.gout = ginv[t & 1];
        launch(ns, true);
        c.NSin = ns; c.prev = c.mode;
    }
    c.pin = part[(3 * sweeps + 1) & 1]; c.pout = nullptr; c.mode = -1;
    c.gin = ginv[(3 * sweeps + 1) & 1]; c.gout = nullptr;
    launch(1, false);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}

}  // extern "C"

// ---- exat_cpals for callers that cannot allocate: the workspace is a static device array ----
namespace {
constexpr int64_t kScratchFloats = 4LL << 20;   // 16 MiB per GPU, held until the process ends
constexpr int kMaxDevices = 64;
float *g_scratch_ptr[kMaxDevices] = {};         // device address of `scratch` on each GPU (each holds its own copy)
}  // namespace
static __device__ __align__(256) float scratch[kScratchFloats];

extern "C" {

int exat_cpals_noalloc(const float *Y, int32_t L, int32_t M, int32_t N, int32_t P, int32_t R, int32_t sweeps, float *A, float *B,
                       float *C, void *stream)
{
    if (!Y || !A || !B || !C) return EXAT_ERR_NULL;
    if (L < 1 || M < 1 || N < 1 || R < 1 || P < 1 || sweeps < 0) return EXAT_ERR_SHAPE;
    if (L > CP_MAX || M > CP_MAX || N > CP_MAX || R > CP_MAX || P > (1 << 20)) return EXAT_ERR_SHAPE;
    if (exat_cpals_workspace_floats(L, M, N, P) > kScratchFloats) return EXAT_ERR_SHAPE;   // beyond the static workspace
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return EXAT_ERR_HIP;
    if (!g_scratch_ptr[dev]) {
        // in host code the array's name is a stand-in, not a device address: ask the runtime for this GPU's copy, once
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return EXAT_ERR_HIP; }
        g_scratch_ptr[dev] = (float *)ptr;
    }
    // nothing of the workspace has to start at zero: every update writes the partial results that the next launch reads
    return exat_cpals(Y, L, M, N, P, R, sweeps, A, B, C, g_scratch_ptr[dev], stream);
}

}  // extern "C"
