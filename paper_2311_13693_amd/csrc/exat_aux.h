// Small kernels around the fused mode-1/2 kernel: operand packing (stacking, padding,
// bf16 rounding), the mode-3 contraction, the block merge and the stand-alone block generator.
#pragma once
#include <type_traits>

#include "exat_common.h"

namespace exat {

// round a value through the plan's element type (identity for fp32)
template <typename T> __device__ __forceinline__ float round_through(float v) { return (float)elem<T>::from_f32(v); }

// The packing routines are written for block `block` of `nblocks` blocks of 256 threads, so that one launch can hold several.

// Stacked fp32 matrix (rows x cols, leading dimension ld) -> zero-padded [rowspad][colspad] of T.
template <typename T>
__device__ __forceinline__ void pack_u_part(unsigned block, unsigned nblocks, const float *src, int64_t ld, int rows, int64_t cols, T *dst, int rowspad, int64_t colspad)
{
    const int64_t n = (int64_t)rowspad * colspad;
    for (int64_t idx = (int64_t)block * 256 + threadIdx.x; idx < n; idx += (int64_t)nblocks * 256) {
        const int64_t r = idx / colspad, c = idx % colspad;
        const float v = (r < rows && c < cols) ? src[r * ld + c] : 0.0f;
        dst[idx] = elem<T>::from_f32(v);
    }
}
template <typename T>
__global__ __launch_bounds__(256) void k_pack_u(const float *src, int64_t ld, int rows, int64_t cols, T *dst, int rowspad, int64_t colspad) { pack_u_part<T>(blockIdx.x, gridDim.x, src, ld, rows, cols, dst, rowspad, colspad); }

// Stacked fp32 V (P*M x J) -> fp32 [P][Mpad][Jpad], zero padded, values rounded through T.
template <typename T>
__device__ __forceinline__ void pack_v_part(unsigned block, unsigned nblocks, const float *src, int64_t ld, int P, int M, int64_t J, float *dst, int Mpad, int64_t Jpad)
{
    const int64_t n = (int64_t)P * Mpad * Jpad;
    for (int64_t idx = (int64_t)block * 256 + threadIdx.x; idx < n; idx += (int64_t)nblocks * 256) {
        const int64_t j = idx % Jpad, pm = idx / Jpad;
        const int m = (int)(pm % Mpad), pr = (int)(pm / Mpad);
        const float v = (m < M && j < J) ? src[((int64_t)pr * M + m) * ld + j] : 0.0f;
        dst[idx] = round_through<T>(v);
    }
}
template <typename T>
__global__ __launch_bounds__(256) void k_pack_v(const float *src, int64_t ld, int P, int M, int64_t J, float *dst, int Mpad, int64_t Jpad) { pack_v_part<T>(blockIdx.x, gridDim.x, src, ld, P, M, J, dst, Mpad, Jpad); }

// Stacked fp32 W (P*N x K) -> transposed fp32 [P][K][Npad] (n contiguous, zero padded), values
// rounded through T: the layout the mode-3 MFMA reads its B operand from with coalesced loads.
template <typename T>
__device__ __forceinline__ void pack_w_part(unsigned block, unsigned nblocks, const float *src, int64_t ld, int P, int N, int64_t K, float *dst, int Npad)
{
    const int64_t n_all = (int64_t)P * K * Npad;
    for (int64_t idx = (int64_t)block * 256 + threadIdx.x; idx < n_all; idx += (int64_t)nblocks * 256) {
        const int n = (int)(idx % Npad);
        const int64_t pk = idx / Npad, k = pk % K, pr = pk / K;
        const float v = (n < N) ? src[(pr * N + n) * ld + k] : 0.0f;
        dst[idx] = round_through<T>(v);
    }
}
template <typename T>
__global__ __launch_bounds__(256) void k_pack_w(const float *src, int64_t ld, int P, int N, int64_t K, float *dst, int Npad) { pack_w_part<T>(blockIdx.x, gridDim.x, src, ld, P, N, K, dst, Npad); }

// Mode 3: Y[p,l,m,n] (=|+=) sum_{k in [k0,k1)} W_p[n,k] Q[k-k0][p*L+l][m].
// fp32 MFMAs over k in ascending order; the fp32 partial sums go into fp64 totals every KFLUSH values of k so that the
// summation error does not grow with the extent of K.
struct Mode3Params {
    const float *Q;  // [nk << kshift][PLpad][Mpad]
    const float *W;  // [P][K][Npad]
    float *Y;        // Y[l + L*(m + M*(n + N*p))]
    int L, M, N, PL, PLpad, Mpad, Npad;
    int64_t K, k0, k1;
    int accumulate;
    int kshift;           // slice k left 2^kshift partial Q, which follow each other
    uint32_t *ranges;     // if not null, the MPF_CALL_WORDS first words are cleared for the next call
    unsigned char *flag;  // if not null, set to 1 by the launch (block streaming: "this slot holds a partial result")
};

// One workgroup per MP x 32 (q, m) positions of one stacked row x <= 64 columns n; its NW waves split the k range into
// contiguous slabs (the outputs are few and the k range long, so k is where the parallelism is) and their partial
// sums are added in wave order, which keeps the result independent of timing.
// Bound by the loads: Q once from memory, W_p by every workgroup from the caches.  A workgroup that takes all 64 values of m
// (MP = 2) reads W_p half as often; few workgroups with many waves each (NW = 16) shorten the chain of dependent loads of a
// small call.  Workgroup ids are dealt out so that neighbouring rows share an XCD, and full batches of loads carry no
// per-lane conditions.  Measured (before -> now): 4096 rows x 64 x 512 slices 0.333 -> 0.285 ms, 1550 rows x 50 x 1000 slices
// 0.202 -> 0.188 ms; 64 rows x 16 x 512 partial slices 10.2 -> 8.7 us with 16 waves instead of 4.

// NT = 32-column tiles of n per workgroup (1 or 2).  LONGK: a wave's slab of k may exceed KFLUSH values, so the
// fp32 MFMA accumulators are flushed into fp64 sums every KFLUSH values; without it the accumulators themselves
// are the slab's result and no fp64 registers are alive during the loop.
template <int NT, int MP, int NW, bool LONGK>
__global__ __launch_bounds__(64 * NW, NW > 4 ? NW / 4 : (LONGK ? 1 : 2)) void k_mode3(const Mode3Params p)
{
    constexpr int KFLUSH = 512;
    typedef std::conditional_t<LONGK, double, float> part_t;
    extern __shared__ __align__(16) unsigned char m3_smem[];
    part_t *part = (part_t *)m3_smem;   // [NW][MP][NT][16][64]
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
    if (p.flag != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *p.flag = 1;
    if (p.ranges != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < MPF_CALL_WORDS) p.ranges[threadIdx.x] = 0;
    // Workgroup ids go round-robin over the 8 XCDs: each takes a contiguous range of the stacked rows, so that the rows l of one
    // replica, whose results are neighbours in Y, meet in one L2 (and read the same W_p through it).
    const int64_t per = (gridDim.x + 7) >> 3, tile = (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3), pos0 = tile * 32 * MP;
    if (pos0 >= (int64_t)p.PL * p.Mpad) return;  // whole workgroup
    const int q = (int)(pos0 / p.Mpad), m0 = (int)(pos0 % p.Mpad);
    if (m0 >= p.M) return;                       // a tile made of padding columns only (whole workgroup)
    const int pr = q / p.L, l = q % p.L;
    const int n0 = blockIdx.y * 32 * NT;
    const int64_t nkall = (p.k1 - p.k0) << p.kshift, qs = (int64_t)p.PLpad * p.Mpad;
    const int64_t slab = (((nkall + NW - 1) / NW) + 1) & ~(int64_t)1;  // even: lanes 32..63 take odd k
    const int64_t kbeg = wave * slab;
    const int64_t nk = (kbeg >= nkall) ? 0 : ((kbeg + slab < nkall) ? slab : nkall - kbeg);
    const float *qp = p.Q + kbeg * qs + pos0 + l32;                               // + kk*qs (+32 for tile 1)
    const float *wp = p.W + ((int64_t)pr * p.K + p.k0) * p.Npad + n0 + l32;       // + ((kbeg + kk) >> kshift)*Npad (+32 for tile 1)
    double totl[LONGK ? MP * NT : 1][16];   // LONGK only
    f32x16 acc[MP][NT];
#pragma unroll
    for (int t = 0; t < MP * NT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
            acc[t / NT][t % NT][e] = 0.0f;
            if (LONGK) totl[t][e] = 0.0;
        }
    for (int64_t kc = 0; kc < nk; kc += LONGK ? KFLUSH : nk) {
        const int64_t kend = (LONGK && kc + KFLUSH < nk) ? kc + KFLUSH : nk;
        // 16 values of k per batch, two register sets: the loads of the next batch are issued before the MFMAs
        // of the current one (the kernel runs at well under one wave per SIMD, so nothing else hides the latency)
        constexpr int KB = 16, NS = KB / 2;
        float a[2][MP][NS], b[2][NT][NS];
        const float *ql = qp + hi * qs;
        auto load_batch = [&](int set, int64_t kk) __attribute__((always_inline)) {
            if (kk + KB <= kend) {   // no per-lane condition, wave-uniform offsets
#pragma unroll
                for (int t = 0; t < NS; t++) {
                    const float *a0 = ql + (kk + 2 * t) * qs;
                    const float *b0 = wp + (p.kshift ? ((kbeg + kk + 2 * t + hi) >> p.kshift) * p.Npad : (kbeg + kk + 2 * t) * p.Npad + hi * p.Npad);
#pragma unroll
                    for (int m = 0; m < MP; m++) a[set][m][t] = a0[32 * m];
#pragma unroll
                    for (int n = 0; n < NT; n++) b[set][n][t] = b0[32 * n];
                }
                return;
            }
#pragma unroll
            for (int t = 0; t < NS; t++) {
                const int64_t kx = kk + 2 * t + hi;
                const bool ok = kx < kend;
                const int64_t kw = ((kbeg + kx) >> p.kshift) * p.Npad;
#pragma unroll
                for (int m = 0; m < MP; m++) a[set][m][t] = ok ? qp[kx * qs + 32 * m] : 0.0f;
#pragma unroll
                for (int n = 0; n < NT; n++) b[set][n][t] = ok ? wp[kw + 32 * n] : 0.0f;
            }
        };
        auto mma_batch = [&](int set) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NS; t++)
#pragma unroll
                for (int m = 0; m < MP; m++)
#pragma unroll
                    for (int n = 0; n < NT; n++) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[set][m][t], b[set][n][t], acc[m][n], 0, 0, 0);
        };
        load_batch(0, kc);
        for (int64_t kk = kc; kk < kend; kk += 2 * KB) {
            load_batch(1, kk + KB);       // zeros beyond kend
            __builtin_amdgcn_sched_barrier(0);
            mma_batch(0);
            load_batch(0, kk + 2 * KB);
            __builtin_amdgcn_sched_barrier(0);
            mma_batch(1);
        }
        if (LONGK) {
#pragma unroll
            for (int t = 0; t < MP * NT; t++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    totl[t][e] += (double)acc[t / NT][t % NT][e];
                    acc[t / NT][t % NT][e] = 0.0f;
                }
        }
    }
#pragma unroll
    for (int t = 0; t < MP * NT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
            if constexpr (LONGK) part[((wave * MP * NT + t) * 16 + e) * 64 + lane] = totl[t][e];
            else part[((wave * MP * NT + t) * 16 + e) * 64 + lane] = acc[t / NT][t % NT][e];
        }
    __syncthreads();
    // The waves' partial sums in wave order, in fp64; wave w finishes the elements w, w + NW, ... of every tile.
    // C layout: element 4b+r of the accumulator is row (position) 8b + 4*hi + r, column n = l32
#pragma unroll
    for (int t = 0; t < MP * NT; t++)
#pragma unroll
        for (int ee = 0; ee < 16 / NW; ee++) {
            const int e = wave + NW * ee;
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NW; w++) s += (double)part[((w * MP * NT + t) * 16 + e) * 64 + lane];
            const int n = n0 + 32 * (t % NT) + l32, m = m0 + 32 * (t / NT) + 8 * (e >> 2) + 4 * hi + (e & 3);
            if (n < p.N && m < p.M) {
                float *dst = p.Y + l + (int64_t)p.L * (m + (int64_t)p.M * (n + (int64_t)p.N * pr));
                const float v = (float)s;
                *dst = p.accumulate ? *dst + v : v;
            }
        }
}

// Block merge (Fig. 2a): Y = sum over partial slots in ascending slot order (fp64 running sum).
__global__ void k_merge(const float *slots, const unsigned char *used, int nslots, int64_t n, float *Y)
{
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int t = 0; t < nslots; t++)
            if (used[t]) s += (double)slots[(int64_t)t * n + idx];
        Y[idx] = (float)s;
    }
}

// Stand-alone generator of one box of the synthetic tensor, column-major on the box.
struct GenParams {
    const float *A, *B, *C;
    int64_t ldA, ldB, ldC;
    int R;
    uint32_t skey;
    float amp2_ln2;
    int64_t i0, i1, j0, j1, k0, k1;
};

// Bound by the writes and, close behind, by the noise (39 vector instructions per four elements).  A wave owns GB_Q quads of
// four consecutive i (one per lane) of GB_J fibres: a quad of A serves all of them, and what depends on the fibre only -- the
// products B[j,r] C[k,r], the fibre's key -- is formed once per wave (LDS, scalar registers).  Before, a thread made one quad and
// read A, B and C for each.  500^3, R = 5, fp32: 0.595 ms before,
// 0.095 ms now (5.3 TB/s written).
constexpr int GB_Q = 64, GB_J = 8, GB_W = 4;   // quads and fibres per wave, waves per workgroup

template <typename T>
__global__ __launch_bounds__(64 * GB_W) void k_gen_box(const GenParams p, T *out)
{
    extern __shared__ float bcs[];   // [wave][r][GB_J]
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t q0 = p.i0 >> 2, nq = ((p.i1 - 1) >> 2) - q0 + 1;
    const int64_t di = p.i1 - p.i0, dj = p.j1 - p.j0, dk = p.k1 - p.k0;
    const int64_t nqb = (nq + GB_Q - 1) / GB_Q, njb = (dj + GB_J * GB_W - 1) / (GB_J * GB_W), nb = nqb * njb * dk;
    float *bc = bcs + w * p.R * GB_J;
    typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
    typedef T out4 __attribute__((ext_vector_type(4)));
    typedef out4 out4_u __attribute__((aligned(sizeof(T))));
    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const int64_t qb = b % nqb, jb = b / nqb % njb, k = p.k0 + b / (nqb * njb);
        const int64_t jw = p.j0 + (jb * GB_W + w) * GB_J;   // the wave's first fibre; fibres past the box are made and not written
        const int64_t iq = q0 + qb * GB_Q + lane, i = 4 * iq;
        __syncthreads();   // the products of the round before have been read
        for (int e = lane; e < p.R * GB_J; e += 64) {
            const int r = e / GB_J;
            const int64_t j = jw + e % GB_J < p.j1 ? jw + e % GB_J : p.j1 - 1;
            bc[e] = p.B[j + p.ldB * r] * p.C[k + p.ldC * r];
        }
        __syncthreads();
        float x[GB_J][4];
#pragma unroll
        for (int u = 0; u < GB_J; u++)
#pragma unroll
            for (int e = 0; e < 4; e++) x[u][e] = 0.0f;
        const bool whole = i >= p.i0 && i + 4 <= p.i1;
        for (int r = 0; r < p.R; r++) {
            f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f};
            const float *ap = p.A + p.ldA * r;
            if (whole) a = *(const f32x4_a4 *)(ap + i);
            else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (i + e >= p.i0 && i + e < p.i1) a[e] = ap[i + e];
            }
            const f32x4 b0 = *(const f32x4 *)(bc + r * GB_J), b1 = *(const f32x4 *)(bc + r * GB_J + 4);
#pragma unroll
            for (int u = 0; u < GB_J; u++)
#pragma unroll
                for (int e = 0; e < 4; e++) x[u][e] = __builtin_fmaf(a[e], u < 4 ? b0[u & 3] : b1[u & 3], x[u][e]);
        }
        if (p.amp2_ln2 != 0.0f) {
#pragma unroll
            for (int u = 0; u < GB_J; u++) {
                float z[4];
                noise_quad(fibre_key(p.skey, (uint32_t)(jw + u), (uint32_t)k), (uint32_t)iq, p.amp2_ln2, z);
#pragma unroll
                for (int e = 0; e < 4; e++) x[u][e] += z[e];
            }
        }
#pragma unroll
        for (int u = 0; u < GB_J; u++) {
            if (jw + u >= p.j1) break;   // wave-uniform
            T *dst = out + (i - p.i0) + di * ((jw + u - p.j0) + dj * (k - p.k0));
            if (whole) {
                const out4 v = {elem<T>::from_f32(x[u][0]), elem<T>::from_f32(x[u][1]), elem<T>::from_f32(x[u][2]), elem<T>::from_f32(x[u][3])};
                *(out4_u *)dst = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (i + e >= p.i0 && i + e < p.i1) dst[e] = elem<T>::from_f32(x[u][e]);
            }
        }
    }
}

// The same for blocks thin in i or in j, which would leave most lanes of k_gen_box without a quad or most waves without a fibre.  A
// wave takes 2^lq quads, the smallest power of two that holds a fibre (at most 64), of (64 >> lq) GB_J fibres; the fibres are numbered over
// j and k together, and neighbouring lanes write neighbouring fibres.  A lane's fibres are its own, so their products B[j,r] C[k,r] are
// formed in registers, for two r at a time (one at a time waits for the loads: R = 64 takes three times as long).
// Taken up to a quarter of k_gen_box's lanes busy.  2^24 elements, fp32, one quad per thread as it once was, k_gen_box, this one, in us:
//   dI = 4 of long fibres in j  R = 5  47, 569, 25   R = 64  362, 2031, 94        64 x 32 x 8192 (a quarter)  R = 5  88, 43, 25   R = 64  952, 137, 97
//   dI = 32                     R = 5  59, 77, 25    R = 64  532, 247, 93         500 x 4 x 8388              R = 5  88, 64, 30   R = 64  940, 289, 124
// In full blocks k_gen_box takes 13.
template <typename T>
__global__ __launch_bounds__(256) void k_gen_thin(const GenParams p, int lq, T *out)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, FW = 64 >> lq, grp = lane >> lq;
    const int64_t q0 = p.i0 >> 2, nq = ((p.i1 - 1) >> 2) - q0 + 1;
    const int64_t di = p.i1 - p.i0, dj = p.j1 - p.j0, nf = dj * (p.k1 - p.k0), nqb = (nq + (1 << lq) - 1) >> lq, nw = (nf + GB_J * FW - 1) / (GB_J * FW) * nqb;
    const int sj = (int)(FW % dj), sk = (int)(FW / dj);
    typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
    typedef T out4 __attribute__((ext_vector_type(4)));
    typedef out4 out4_u __attribute__((aligned(sizeof(T))));
    for (int64_t wv = (int64_t)blockIdx.x * 4 + w; wv < nw; wv += (int64_t)gridDim.x * 4) {
        const int64_t iq = q0 + (wv % nqb << lq) + (lane & ((1 << lq) - 1)), i = 4 * iq;
        const bool whole = i >= p.i0 && i + 4 <= p.i1;
        const int64_t t0 = wv / nqb * (GB_J * FW) + grp;   // fibre u of the lane is t0 + u FW
        int j[GB_J], k[GB_J];
        j[0] = (int)(t0 % dj); k[0] = (int)(t0 / dj);
#pragma unroll
        for (int u = 1; u < GB_J; u++) {
            j[u] = j[u - 1] + sj; k[u] = k[u - 1] + sk;
            if (j[u] >= dj) { j[u] -= (int)dj; k[u]++; }
        }
        float x[GB_J][4];
#pragma unroll
        for (int u = 0; u < GB_J; u++) {
            if (t0 + u * FW >= nf) { j[u] = 0; k[u] = 0; }   // past the box: made and not written
#pragma unroll
            for (int e = 0; e < 4; e++) x[u][e] = 0.0f;
        }
#pragma unroll 2
        for (int r = 0; r < p.R; r++) {
            f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f};
            const float *ap = p.A + p.ldA * r, *bp = p.B + p.j0 + p.ldB * r, *cp = p.C + p.k0 + p.ldC * r;
            if (whole) a = *(const f32x4_a4 *)(ap + i);
            else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (i + e >= p.i0 && i + e < p.i1) a[e] = ap[i + e];
            }
            float bc[GB_J];
#pragma unroll
            for (int u = 0; u < GB_J; u++) bc[u] = bp[j[u]] * cp[k[u]];
#pragma unroll
            for (int u = 0; u < GB_J; u++)
#pragma unroll
                for (int e = 0; e < 4; e++) x[u][e] = __builtin_fmaf(a[e], bc[u], x[u][e]);
        }
        if (p.amp2_ln2 != 0.0f) {
#pragma unroll
            for (int u = 0; u < GB_J; u++) {
                float z[4];
                noise_quad(fibre_key(p.skey, (uint32_t)(p.j0 + j[u]), (uint32_t)(p.k0 + k[u])), (uint32_t)iq, p.amp2_ln2, z);
#pragma unroll
                for (int e = 0; e < 4; e++) x[u][e] += z[e];
            }
        }
#pragma unroll
        for (int u = 0; u < GB_J; u++) {
            if (t0 + u * FW >= nf) continue;
            T *dst = out + (i - p.i0) + di * (t0 + u * FW);
            if (whole) {
                const out4 v = {elem<T>::from_f32(x[u][0]), elem<T>::from_f32(x[u][1]), elem<T>::from_f32(x[u][2]), elem<T>::from_f32(x[u][3])};
                *(out4_u *)dst = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (i + e >= p.i0 && i + e < p.i1) dst[e] = elem<T>::from_f32(x[u][e]);
            }
        }
    }
}

}  // namespace exat
