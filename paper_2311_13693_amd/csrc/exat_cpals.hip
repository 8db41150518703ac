// Batched CP-ALS on the P proxy tensors (paper Alg. 1; Sec. 3 "Decomposition").  Declarations and contracts in
// include/exat.h.
//
// The P problems are independent and small (L, M, N, R <= 64), so latency is what bounds them: the tensors stay in the caches,
// a sweep is 3 * 2 L M N R flops per replica (1.6 GFLOP at 32 replicas of 64^3, rank 32: 10 us at the fp32 matrix rate) and the
// rest are short serial steps.  One update, e.g. of A, is one launch, k_cpals_step, of NS workgroups per replica:
//   1. the update before it is finished: the workgroup adds the NS partial MTTKRP results in slab order, forms the normal matrix
//      G = (F2^T F2) * (F1^T F1) (Gram matrices on the fp32 matrix cores), inverts it and multiplies, X = Mx G^{-1}.  Every
//      workgroup of the replica does that for itself (it needs the new factor at once and there is nothing to wait for); the
//      first one writes the factor to memory.
//   2. its share of this update's MTTKRP, Mx[d0,r] = sum_{d2} sum_{d1} Y[d0,d1,d2] F1[d1,r] F2[d2,r]: a product of the
//      unfolded tensor with the Khatri-Rao matrix, whose entries are formed in registers, on the fp32 matrix cores, over a
//      slab of the outer contraction index.
// The tensor is read where it lies: a lane holds one row of the updated mode, and the order of the contraction indices inside
// a matrix instruction is free, so the first mode reads 128-byte runs along l and the other two 16 bytes of l per lane.
// The normal matrix is inverted by Gauss-Jordan steps without pivoting (it is positive definite; the diagonal elements
// met are the squared pivots of its Cholesky factorisation): 256 threads own cyclic blocks of it in registers, a step publishes
// two rows and two columns through LDS and has one barrier.
// Data, products and sums are fp32, in a fixed order; the inverse and the product with it are fp64.  An inverse rounded to fp32 leaves
// a residual X G - Mx of cond(G) 2^-24 |Mx|, a triangular solve in fp32 one of 2^-24 |Mx|; measured at rank 64, cond(G) = 3.5e4: inverse
// in fp32 1.9e-4, Cholesky factor and two substitutions in fp32 1.7e-7, inverse in fp64 7.5e-8.  The steps wait for LDS and barriers,
// not for arithmetic, so fp64 costs nothing (0.746 -> 0.735 ms, with the hardware's reciprocal in place of a guarded division).
// Measured (32 tensors of 64^3, rank 32, ten sweeps): 3.07 ms with two launches per update and permuted copies of the tensor, 0.735 ms
// now.
#include "../../include/exat.h"

#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

constexpr int CP_MAX = 64;   // largest L, M, N and R

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));   // rows of Y start at multiples of 4 bytes

struct CpStep {
    const float *Y;         // per replica Y[l + L(m + M n)]
    float *F[3];            // A, B, C, per replica column-major D x R
    const float *pin;       // [replica][NSin][d][R]: partial MTTKRP results of the update before this one; replicas `rs` floats apart
    float *pout;            // the same of this update
    int64_t rs;             // the same for every update, whatever its extent: a replica overwrites its own partial results only
    int D[3];               // L, M, N
    int R, NSin, NS, DS;    // NS slabs of DS values of the outer contraction index
    int prev, mode;         // updated factor of the update before and of this one (0, 1, 2), or -1: none
    int P;
    int32_t *status;        // optional, [replica]: incremented by every update whose normal matrix has a non-positive pivot
};

// 1/x to within an ulp or two: the hardware's estimate (more than 20 bits) and two Newton steps.  The pivots come from fp32 values, far
// inside the range of fp64; a zero gives NaN.
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}

// RC = 32-column tiles of the rank, NB = 16-wide blocks of it (R <= 16 NB, NB <= 2 RC)
template <int RC, int NB>
__global__ __launch_bounds__(256) void k_cpals_step(const CpStep p)
{
    constexpr int RS = 32 * RC, RSP = RS + 1;
    __shared__ float Fs[3][CP_MAX * RSP];     // factors as [d][r], zero beyond D and R
    __shared__ float Mx[CP_MAX * RSP];        // MTTKRP result of the update before; scratch of the partial tiles
    __shared__ float G[RS * RSP];             // normal matrix
    constexpr int NGT = RC == 1 ? 4 : 8;
    __shared__ __align__(16) float Gt[NGT][1024];   // tiles of the Gram matrices, then the inverse of the normal matrix
    double *Gi = (double *)&Gt[0][0];         // [r][c ^ 16 (r & 1)]: neighbouring rows 32 banks apart
    static_assert(RS * RS * 8 <= NGT * 4096, "");
    __shared__ double rowb[2][2][64], colb[2][2][64];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t rep = blockIdx.x;
    const int slab = blockIdx.y, R = p.R;

    // ---- this workgroup's share of the MTTKRP.  Mode 0: rows l, inner m, outer n; mode 1: rows m, inner l, outer n; mode 2:
    //      rows n, inner l, outer m.  Tile (rt, ct) of the result to wave w mod ntile; the waves of a tile take the values of
    //      the outer index in turn ----
    const int u = p.mode >= 0 ? p.mode : 0, Du = p.D[u], i1 = u == 0 ? 1 : 0, i2 = u == 2 ? 1 : 2, D1 = p.D[i1], D2 = p.D[i2];
    const int rtn = (Du + 31) / 32, ntile = rtn * RC, kgn = 4 / ntile, kg = w / ntile, tile = w % ntile;
    const int row = 32 * (tile / RC) + l32, c = 32 * (tile % RC) + l32;
    // element (row, d1, d2) of the tensor: a wave-uniform pointer to (0, d1, d2) and the lane's 32-bit offset (a replica has at most
    // 2^18 elements)
    const int LM = p.D[0] * p.D[1], su = u == 0 ? 1 : (u == 1 ? p.D[0] : LM), s2 = u == 2 ? p.D[0] : LM;
    const float *yu = p.Y + rep * LM * p.D[2];
    const unsigned ro = (unsigned)((row < Du ? row : Du - 1) * su);
    constexpr int NSTEP = CP_MAX / 2;
    const int nq = (D1 + 7) / 8;           // groups of 8 inner indices
    const int d2a = slab * p.DS, d2b = d2a + p.DS < D2 ? d2a + p.DS : D2;
    auto load = [&](int d2, f32x4 (&a)[NSTEP / 4]) __attribute__((always_inline)) {
        const float *y = yu + d2 * s2;
#pragma unroll
        for (int q = 0; q < NSTEP / 4; q++) {
            if (q < nq) {
                if (u == 0) {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const int d = 8 * q + 2 * e;   // lane half hi: d + hi; beyond D1 the factor is zero and any element will do
                        if (d + 1 < D1) a[q][e] = (y + d * p.D[0])[ro + (unsigned)(hi * p.D[0])];
                        else a[q][e] = (y + (D1 - 1) * p.D[0])[ro];
                    }
                } else if (8 * q + 8 <= D1)
                    a[q] = *(const f32x4_a4 *)((y + 8 * q) + (ro + 4u * hi));
                else {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const int d = 8 * q + 4 * hi + e;
                        a[q][e] = y[ro + (unsigned)(d < D1 ? d : D1 - 1)];
                    }
                }
            }
        }
    };
    // the wave's first PF values of the outer index are requested ahead of everything else: most of its share comes in while the
    // update before is finished
    constexpr int PF = 4;
    f32x4 ya[PF][NSTEP / 4];
    if (p.mode >= 0) {
#pragma unroll
        for (int i = 0; i < PF; i++)
            if (d2a + kg + i * kgn < d2b) load(d2a + kg + i * kgn, ya[i]);
    }

    // The factors that are fixed in the update before this one (without one: in this update).  All loads below are made at clamped
    // addresses and masked afterwards, so that they are in flight together.
    const int v = p.prev >= 0 ? p.prev : p.mode;
    const int f1 = v == 0 ? 1 : 0, f2 = v == 2 ? 1 : 2;
    constexpr int FE = CP_MAX * RS / 256;
    {
        float t[2][FE];
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const int f = q ? f2 : f1, D = p.D[f];
            const float *src = p.F[f] + rep * D * R;
#pragma unroll
            for (int x = 0; x < FE; x++) {
                const int e = tid + 256 * x, d = e % CP_MAX, r = e / CP_MAX;
                t[q][x] = src[(d < D ? d : D - 1) + D * (r < R ? r : R - 1)];
            }
        }
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const int f = q ? f2 : f1, D = p.D[f];
#pragma unroll
            for (int x = 0; x < FE; x++) {
                const int e = tid + 256 * x, d = e % CP_MAX, r = e / CP_MAX;
                Fs[f][d * RSP + r] = (d < D && r < R) ? t[q][x] : 0.0f;
            }
        }
    }

    if (p.prev >= 0) {
        const int D0 = p.D[v];
        // MTTKRP result: the slabs' partial results in slab order
        const float *src = p.pin + rep * p.rs;
        const int st = D0 * R;
        constexpr int XB = FE < 4 ? FE : 4;
#pragma unroll
        for (int x0 = 0; x0 < FE; x0 += XB) {
            const float *q[XB];
            float x[XB];
#pragma unroll
            for (int i = 0; i < XB; i++) {
                const int e = tid + 256 * (x0 + i), d = e / RS, r = e % RS;
                q[i] = src + (d < D0 ? d : D0 - 1) * R + (r < R ? r : R - 1);
                x[i] = 0.0f;
            }
            int sl = 0;
            for (; sl + 8 <= p.NSin; sl += 8) {
                float t[XB][8];
#pragma unroll
                for (int i = 0; i < XB; i++)
#pragma unroll
                    for (int u = 0; u < 8; u++) t[i][u] = q[i][(sl + u) * st];
#pragma unroll
                for (int i = 0; i < XB; i++)
#pragma unroll
                    for (int u = 0; u < 8; u++) x[i] += t[i][u];
            }
            for (; sl < p.NSin; sl++)
#pragma unroll
                for (int i = 0; i < XB; i++) x[i] += q[i][sl * st];
#pragma unroll
            for (int i = 0; i < XB; i++) {
                const int e = tid + 256 * (x0 + i), d = e / RS, r = e % RS;
                Mx[d * RSP + r] = (d < D0 && r < R) ? x[i] : 0.0f;
            }
        }
        __syncthreads();
        // Gram matrices, one 32 x 32 tile of one of them (one tile only: half of its contraction) per job, jobs to the waves in turn
        constexpr int KH = RC == 1 ? 2 : 1, NJ = RC * RC * 2 * KH;
#pragma unroll
        for (int j = w; j < NJ; j += 4) {
            const int t = j / (2 * KH), m = (j / KH) & 1, kh = j % KH;
            const float *F = Fs[m ? f2 : f1];
            const int ri = 32 * (t / RC) + l32, ci = 32 * (t % RC) + l32;
            f32x16 g[2];
#pragma unroll
            for (int e = 0; e < 16; e++) g[0][e] = g[1][e] = 0.0f;
#pragma unroll
            for (int s = 0; s < CP_MAX / 2 / KH; s++) {
                const int d = (2 * (s + kh * (CP_MAX / 2 / KH)) + hi) * RSP;
                g[s & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(F[d + ri], F[d + ci], g[s & 1], 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 16; e++) Gt[j][e * 64 + lane] = g[0][e] + g[1][e];
        }
        __syncthreads();
        for (int e = tid; e < RC * RC * 1024; e += 256) {
            const int t = e >> 10, x = e & 1023, r = x >> 6, l = x & 63;
            float g1 = Gt[2 * KH * t][x], g2 = Gt[2 * KH * t + KH][x];
            if (KH == 2) { g1 += Gt[2 * KH * t + 1][x]; g2 += Gt[2 * KH * t + KH + 1][x]; }
            G[(32 * (t / RC) + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3)) * RSP + 32 * (t % RC) + (l & 31)] = g1 * g2;
        }
        __syncthreads();
        // Gi <- G^{-1}, in fp64: thread (ty, tx) owns the entries (ty + 16 a, tx + 16 b), extended by the identity beyond R.  A step
        // eliminates two rows and columns, in the order and with the pivots of two single steps.
        const int ty = tid >> 4, tx = tid & 15;
        double g[NB][NB];
#pragma unroll
        for (int a = 0; a < NB; a++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const int i = ty + 16 * a, c = tx + 16 * b;
                g[a][b] = (i == c && i >= R) ? 1.0 : (double)G[i * RSP + c];
            }
        bool bad = false;   // the same in every thread: all see the same pivots
#pragma unroll
        for (int jb = 0; jb < NB; jb++)
            for (int jt = 0; jt < 16; jt += 2) {
                const int j = 16 * jb + jt, par = (jt >> 1) & 1;
                if (j >= R) break;
                if ((tx & 14) == jt) {
#pragma unroll
                    for (int a = 0; a < NB; a++) colb[par][tx & 1][ty + 16 * a] = g[a][jb];
                }
                if ((ty & 14) == jt) {
#pragma unroll
                    for (int b = 0; b < NB; b++) rowb[par][ty & 1][tx + 16 * b] = g[jb][b];
                }
                __syncthreads();
                const double p00 = colb[par][0][j], p10 = colb[par][0][j + 1], p01 = colb[par][1][j], p11 = colb[par][1][j + 1];
                const double inv0 = recip(p00), ur = p01 * inv0, lr = p10 * inv0, s = fma(-lr, p01, p11), inv1 = recip(s);
                bad = bad || !(p00 > 0.0) || (j + 1 < R && !(s > 0.0));   // zero, negative or NaN: not positive definite
                double w0[NB], w1[NB], q0[NB], q1[NB];
#pragma unroll
                for (int a = 0; a < NB; a++) {
                    const double f0 = colb[par][0][ty + 16 * a], f1v = colb[par][1][ty + 16 * a];
                    w1[a] = fma(-f0, ur, f1v) * inv1;
                    w0[a] = fma(-w1[a], p10, f0) * inv0;
                    q0[a] = rowb[par][0][tx + 16 * a]; q1[a] = rowb[par][1][tx + 16 * a];
                }
#pragma unroll
                for (int a = 0; a < NB; a++)
#pragma unroll
                    for (int b = 0; b < NB; b++) {
                        double up = fma(-w1[a], q1[b], fma(-w0[a], q0[b], g[a][b]));
                        if (b == jb) up = (tx & 14) == jt ? ((tx & 1) ? -w1[a] : -w0[a]) : up;
                        if (a == jb) {
                            const double r1 = fma(-lr, q0[b], q1[b]) * inv1, r0 = fma(-p01, r1, q0[b]) * inv0;
                            double rr = (ty & 1) ? r1 : r0;
                            if (b == jb) {   // the inverse of the 2 x 2 pivot block
                                const double i01 = -ur * inv1;
                                const double dd = (tx & 1) ? ((ty & 1) ? inv1 : i01) : ((ty & 1) ? -lr * inv1 : fma(-i01, lr, inv0));
                                rr = (tx & 14) == jt ? dd : rr;
                            }
                            up = (ty & 14) == jt ? rr : up;
                        }
                        g[a][b] = up;
                    }
            }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < NB; a++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const int i = ty + 16 * a, c = tx + 16 * b;
                Gi[i * RS + (c ^ (16 * (i & 1)))] = (i < R && c < R) ? g[a][b] : 0.0;
            }
        if (bad && tid == 0 && slab == 0 && p.status) p.status[rep] += 1;   // launches on one stream: nothing else touches this word now
        __syncthreads();
        // X = Mx G^{-1}, accumulated in fp64: 16 x 16 tile (rt, ct) to wave (rt NB + ct) mod 4
        const int rtn = (D0 + 15) / 16, l16 = lane & 15, q16 = lane >> 4;
        for (int t = w; t < rtn * NB; t += 4) {
            const int row = 16 * (t / NB) + l16, c = 16 * (t % NB) + l16;
            f64x4 x = {0.0, 0.0, 0.0, 0.0};
            for (int s = 0; s < 4 * NB; s++) {
                const int k = 4 * s + q16;
                x = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Mx[row * RSP + k], Gi[k * RS + (c ^ (16 * (k & 1)))], x, 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int d = 16 * (t / NB) + 4 * e + q16;
                const float xf = (float)x[e];
                Fs[v][d * RSP + c] = (d < D0 && c < R) ? xf : 0.0f;
                if (slab == 0 && d < D0 && c < R) p.F[v][rep * D0 * R + d + (int64_t)D0 * c] = xf;
            }
        }
        // the unused row tiles, and the columns beyond the blocks of the rank
        for (int e = tid + 16 * rtn * RS; e < CP_MAX * RS; e += 256) Fs[v][(e / RS) * RSP + e % RS] = 0.0f;
        if (16 * NB < RS)
            for (int e = tid; e < 16 * rtn * (RS - 16 * NB); e += 256) Fs[v][(e / (RS - 16 * NB)) * RSP + 16 * NB + e % (RS - 16 * NB)] = 0.0f;
    }
    if (p.mode < 0) return;
    __syncthreads();

    // inner index of step s, lane half hi: mode 0: 2s + hi; else 8 (s/4) + 4 hi + s%4 (a lane's 16 bytes)
    float b1[NSTEP];
#pragma unroll
    for (int s = 0; s < NSTEP; s++) {
        const int d = u == 0 ? 2 * s + hi : 8 * (s >> 2) + 4 * hi + (s & 3);
        b1[s] = Fs[i1][d * RSP + c];
    }
    f32x16 acc[2];
#pragma unroll
    for (int e = 0; e < 16; e++) acc[0][e] = acc[1][e] = 0.0f;
    auto mac = [&](int d2, const f32x4 (&a)[NSTEP / 4]) __attribute__((always_inline)) {
        const float f2 = Fs[i2][d2 * RSP + c];
#pragma unroll
        for (int q = 0; q < NSTEP / 4; q++) {
            if (q < nq) {
#pragma unroll
                for (int e = 0; e < 4; e++) acc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][e], b1[4 * q + e] * f2, acc[e & 1], 0, 0, 0);
            }
        }
    };
    for (int d2 = d2a + kg; d2 < d2b; d2 += PF * kgn) {
#pragma unroll
        for (int i = 0; i < PF; i++) {
            if (d2 + i * kgn < d2b) mac(d2 + i * kgn, ya[i]);
            if (d2 + (i + PF) * kgn < d2b) load(d2 + (i + PF) * kgn, ya[i]);
        }
    }
#pragma unroll
    for (int e = 0; e < 16; e++) acc[0][e] += acc[1][e];
    // the waves of a tile add up in wave order
    for (int k = 1; k < kgn; k++) {
        __syncthreads();
        if (kg == k) {
#pragma unroll
            for (int e = 0; e < 16; e++) Mx[(tile * 16 + e) * 64 + lane] = acc[0][e];
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int e = 0; e < 16; e++) acc[0][e] += Mx[(tile * 16 + e) * 64 + lane];
        }
    }
    if (kg == 0) {
        float *dst = p.pout + rep * p.rs + (int64_t)slab * Du * R;
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int d = 32 * (tile / RC) + 8 * (e >> 2) + 4 * hi + (e & 3);
            if (d < Du && c < R) dst[d * R + c] = acc[0][e];
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
    // Slabs per replica: about one workgroup per compute unit, and no more than 16, since every workgroup adds up all slabs.  The
    // partial results are double-buffered (a workgroup that is ahead writes while others still read) unless a replica has
    // one workgroup only: that one has read all of its replica's partial results before it writes there.
    const int maxd = L > M ? (L > N ? L : N) : (M > N ? M : N);
    int NS = 256 / P;
    NS = NS > 16 ? 16 : (NS < 1 ? 1 : NS);
    const int64_t room = (int64_t)slabs_for(maxd, P) * CP_MAX * CP_MAX, one = (int64_t)maxd * R;
    while (NS > 1 && 2 * NS * one > room) NS--;
    float *part[2] = {work, NS > 1 ? work + (int64_t)P * NS * one : work};
    CpStep c;
    c.Y = Y; c.F[0] = A; c.F[1] = B; c.F[2] = C; c.D[0] = L; c.D[1] = M; c.D[2] = N; c.R = R; c.P = P; c.rs = NS * one; c.status = status;
    c.NSin = 1; c.prev = -1;
    auto launch = [&](int ns) {
        const dim3 grid((unsigned)P, (unsigned)ns);
        if (R <= 16) hipLaunchKernelGGL((k_cpals_step<1, 1>), grid, dim3(256), 0, st, c);
        else if (R <= 32) hipLaunchKernelGGL((k_cpals_step<1, 2>), grid, dim3(256), 0, st, c);
        else hipLaunchKernelGGL((k_cpals_step<2, 4>), grid, dim3(256), 0, st, c);
    };
    // A <- Y_(1) (C kr B) [(C^T C) * (B^T B)]^-1, then B <- Y_(2) (C kr A) [..]^-1, then C <- Y_(3) (B kr A) [..]^-1: the launch of an
    // update finishes the one before it
    for (int t = 0; t < 3 * sweeps; t++) {
        c.mode = t % 3;
        const int D2 = c.mode == 2 ? M : N;
        int ns = NS < D2 ? NS : D2;
        c.DS = (D2 + ns - 1) / ns;
        c.NS = (D2 + c.DS - 1) / c.DS;
        c.pin = part[(t + 1) & 1]; c.pout = part[t & 1];
        launch(c.NS);
        c.NSin = c.NS; c.prev = c.mode;
    }
    c.pin = part[(3 * sweeps + 1) & 1]; c.pout = nullptr; c.mode = -1; c.NS = 1;
    launch(1);
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
