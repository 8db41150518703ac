// Fused mode-1 + mode-2 kernel on the 16-bit matrix cores with operands taken as sums of 16-bit pieces; materialised
// source, any extents, any alignment, any sub-box.
//
// NP pieces per operand value:
//   NP = 3  fp32 data, bf16 pieces: x = h + m + l with h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), which is exact
//           (three times eight significand bits), and six of the nine products u_a x_b accumulated in fp32.  The three that
//           are left out are at most 2^-26 of the product, below the rounding of an fp32 multiplication, and a 16-value
//           contraction costs six roundings of the running sum where the fp32 matrix instruction makes eight.
//   NP = 2  fp32 data, fp16 pieces (the residual split of the paper's Eq. 5): three products, error 2^-22; fp16 range.
//   NP = 1  bf16 data.
// What bounds it: the matrix pipe.  The fp32 matrix instruction runs at 1/16 of the bf16 rate, six bf16 products cost 6/16
// of it.
//
// Pieces of a value outside a range are not what the sum above says: an infinity has no finite residual, and the low pieces
// of values near the smallest normal number are lost.  The kernel therefore notes the range of what it multiplies
// (MpParams::flags) and a launch of the generic kernel behind it, which otherwise ends at once, computes the call with fp32
// products when a value lay outside (mp_out_of_range).
//
// Decomposition as in k_mode12: a workgroup owns one slice k and a group of stacked rows, walks the slice in chunks of 128
// fibres with the whole i extent reduced before mode 2.  Eight waves:
//   NWC = 1  every wave holds up to two 32-row tiles x 128 fibres.  The row tiles are dealt to the G groups in quads, as
//            evenly as they go (a quad is one tile per SIMD), and inside a group tile t goes to wave t mod 8; a wave with one
//            tile runs a stage loop of its own.
//   NWC = 2, 4 (at most 8 or 4 row tiles in all)  NWC waves share a row tile and take 128/NWC fibres each; each leaves its
//            own partial Q, which mode 3 adds up as if it were a slice of its own (Mode3Params::kshift).
// X goes HBM -> registers -> (split) -> LDS; U comes in fragment order straight from L2 into registers.  The X tiles sit in a
// ring of NSLOT LDS slots: a stage reads tile s and writes tile s + H, H = NSLOT/2, and the workgroup meets at a barrier
// after every H-th stage only (between two barriers the slots read and the slots written are disjoint).
// Measured (one call, before -> now): 512^3 fp32, 512 stacked rows 1.05 -> 0.67 ms (fp32 matrix instruction before); 1000^3
// fp32, 1550 rows 39.1 -> 18.5 ms and 1000^3 bf16, 2400 rows 25.8 -> 8.3 ms (generic kernel before: 1000 is no multiple of a
// stage); 1024^3 in two fp16 pieces, 2048 rows 14.2 -> 12.0 ms.
#pragma once
#include "exat_mode12_v3.h"

namespace exat {

struct MpParams {
    const void *Uf;    // [PLpad/32][nig][NP][64 lanes][8]: lane l of fragment (rt, ig, piece) holds row 32*rt + l%32,
                       // i = 16*ig + 8*(l/32) .. +7
    int64_t nig;       // Ipad / 16
    const void *Vf;    // [P][Jpad/16][vmt][NV][64 lanes][8]: element e of lane l of fragment (p, j16, mt, piece) holds
                       // V_p[m = 32*mt + l%32, j = 16*j16 + 4*(l/32) + e%4 + 8*(e/4)]
    int vmt;           // 32-row tiles of m in Vf
    int T4;            // quads of row tiles (NWC = 1)
    int64_t ja0;       // first fibre of the first chunk (a multiple of 16, <= j0)
    uint32_t *flags;   // MPF_* words, or null
};

// notes the largest magnitude `mx` a lane has seen: one word per wave and condition, written only if it is not set yet
__device__ __forceinline__ void mp_note(uint32_t *f, int big, int norm, int nz, float mx, float vmin, float vmax)
{
    const bool b = __any(!(mx <= vmax)), n = __any(mx >= vmin), z = __any(mx > 0.0f);
    if ((threadIdx.x & 63) == 0) {
        if (b && !f[big]) f[big] = 1;
        if (n && !f[norm]) f[norm] = 1;
        if (z && !n && !f[nz]) f[nz] = 1;
    }
}

template <int NP> struct mp_terms;   // (X or Z piece, U or V piece) of the products, smallest first
template <> struct mp_terms<1> { static constexpr int N = 1, X[1] = {0}, U[1] = {0}; };
template <> struct mp_terms<2> { static constexpr int N = 3, X[3] = {1, 0, 0}, U[3] = {0, 1, 0}; };
template <> struct mp_terms<3> { static constexpr int N = 6, X[6] = {2, 0, 1, 1, 0, 0}, U[6] = {0, 2, 1, 0, 1, 0}; };
struct mp_terms_z1 { static constexpr int N = 3, X[3] = {2, 1, 0}, U[3] = {0, 0, 0}; };   // bf16 plans, mode 2: Z in three pieces

template <bool F16>
__device__ __forceinline__ f32x16 mp_mma(const u32x4 &a, const u32x4 &b, const f32x16 &c)
{
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// two fp32 values -> NP words of two 16-bit pieces each (value a in the low half)
template <int NP, bool F16, bool RTZ = false>
__device__ __forceinline__ void mp_split2(float a, float b, uint32_t (&w)[NP])
{
    if constexpr (F16) {
        static_assert(NP == 2, "");
        typedef __fp16 h2 __attribute__((ext_vector_type(2)));
        if constexpr (RTZ) {   // packed truncating conversion: a - h is exact, the pair still carries 21 bits
            const h2 h = __builtin_amdgcn_cvt_pkrtz(a, b);
            w[0] = __builtin_bit_cast(uint32_t, h);
            w[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a - (float)h[0], b - (float)h[1]));
        } else {
            typedef _Float16 g2 __attribute__((ext_vector_type(2)));
            const g2 h = {(_Float16)a, (_Float16)b}, l = {(_Float16)(a - (float)h[0]), (_Float16)(b - (float)h[1])};
            w[0] = __builtin_bit_cast(uint32_t, h); w[1] = __builtin_bit_cast(uint32_t, l);
        }
    } else {
#pragma unroll
        for (int q = 0; q < NP; q++) {
            const bf16x2 h = {(__bf16)a, (__bf16)b};
            w[q] = __builtin_bit_cast(uint32_t, h);
            if (q + 1 < NP) {   // the residual of a rounding to bf16 is exact in fp32
                a -= __builtin_bit_cast(float, w[q] << 16);
                b -= __builtin_bit_cast(float, w[q] & 0xffff0000u);
            }
        }
    }
}

template <int NP, int NWC>
struct Mode12MpCfg {
    static constexpr int NW = 8, NWR = NW / NWC, RT = 2, CT = 4 / NWC, COLS = 128, EI = 32;
    static constexpr int ROWB = 80, XBUF = COLS * ROWB, SLOT = NP * XBUF;
    static constexpr int NSLOT = NP == 1 ? 8 : 4, H = NSLOT / 2;
    static constexpr int LDS_BYTES = NSLOT * SLOT;
    static constexpr int DU = NP == 1 ? 2 : 1;                  // register sets of U fragments
    static constexpr int DX = NP == 1 ? 4 : (NP == 2 ? 2 : 1);  // register sets of the X tile in flight
    static constexpr int XD = NP == 1 ? 4 : 2;                  // register sets of X fragments read from LDS
};

// Mode 2 from the accumulators (acc holds Z^T: rows 32 fibres j, columns 32 stacked rows q; see mode2_direct_bf16 for the
// order of the contraction slots), Z split into pieces like X, V packed in pieces.  A tile whose rows belong to several
// replicas is multiplied with each one's V, and a lane keeps the product of its row's replica.  Q[row][m] += Q^T[m][row];
// Qk points to the rows of this slice (and wave column).
template <int NP, int RT, int CT, int MTC, int RSTRIDE>
__device__ __forceinline__ void mode2_mp(const Mode12Params &p, const MpParams &mp, float *Qk, const f32x16 (&acc)[RT][CT], int wrow0, int ntile,
                                         int64_t jc, bool first_chunk, int lane)
{
    constexpr bool F16 = NP == 2;
    constexpr int MP = 32 * MTC, NZ = NP == 2 ? 2 : 3, NV = NP;
    typedef std::conditional_t<NP == 1, mp_terms_z1, mp_terms<NP>> terms;
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
        const int q0 = wrow0 + rt * RSTRIDE;   // wave-uniform
        if (rt < ntile && q0 < p.PL) {
            int ln = lane;
            asm volatile("" : "+v"(ln));       // per-lane addresses are derived here, after the stage loop (see mode2_chunk)
            const int l32 = ln & 31, hi = ln >> 5;
            const int q = q0 + l32;
            const int qlast = (q0 + 31 < p.PL - 1) ? q0 + 31 : p.PL - 1;
            const int pfirst = q0 / p.L, plast = qlast / p.L;
            float *Qt = Qk + (int64_t)q * MP + 4 * hi;   // + 32*mt + 8*b
            for (int pp = pfirst; pp <= plast; pp++) {
                const bool mine = q >= pp * p.L && q < (pp + 1) * p.L && q < p.PL;
                // fragment (ct, t, mt, piece) of this chunk: j16 = jc/16 + 2 ct + t.  Step u = (2 ct + t) * MTC + mt multiplies
                // with one 32-row tile of V; its fragments are requested AHEAD steps before.
                const u32x4 *vz = (const u32x4 *)mp.Vf + ((int64_t)pp * (p.Jpad / 16) + jc / 16) * mp.vmt * NV * 64 + ln;
                constexpr int NU = 2 * CT * MTC, AHEAD = 2;
                u32x4 v[AHEAD + 1][NV], z[NZ];
                f32x16 d[MTC];
#pragma unroll
                for (int mt = 0; mt < MTC; mt++)
#pragma unroll
                    for (int e = 0; e < 16; e++) d[mt][e] = 0.0f;
                auto load_v = [&](int u) __attribute__((always_inline)) {
#pragma unroll
                    for (int c = 0; c < NV; c++) v[u % (AHEAD + 1)][c] = vz[((u / MTC) * mp.vmt + u % MTC) * (NV * 64) + c * 64];
                };
#pragma unroll
                for (int u = 0; u < AHEAD && u < NU; u++) load_v(u);
                f32x4 qold[MTC][4];
#pragma unroll
                for (int u = 0; u < NU; u++) {
                    const int ct = u / (2 * MTC), t = (u / MTC) & 1, mt = u % MTC;
                    if (u + AHEAD < NU) load_v(u + AHEAD);
                    if (u == NU - 1 - AHEAD / 2) {
#pragma unroll
                        for (int m = 0; m < MTC; m++)
#pragma unroll
                            for (int b = 0; b < 4; b++) {
                                qold[m][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                                if (!first_chunk && mine) qold[m][b] = *(const f32x4 *)(Qt + 32 * m + 8 * b);
                            }
                    }
                    __builtin_amdgcn_sched_barrier(0);   // the requests stay ahead of the MFMAs
                    if (mt == 0) {
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            uint32_t w[NZ];
                            // opaque: or the pieces of all accumulators are formed ahead of the loop over the replicas and spilled
                            float za = acc[rt][ct][8 * t + 2 * e], zb = acc[rt][ct][8 * t + 2 * e + 1];
                            asm volatile("" : "+v"(za), "+v"(zb));
                            mp_split2<NZ, F16>(za, zb, w);
#pragma unroll
                            for (int c = 0; c < NZ; c++) z[c][e] = w[c];
                        }
                    }
#pragma unroll
                    for (int n = 0; n < terms::N; n++) d[mt] = mp_mma<F16>(v[u % (AHEAD + 1)][terms::U[n]], z[terms::X[n]], d[mt]);
                }
                if (mine) {
#pragma unroll
                    for (int mt = 0; mt < MTC; mt++)
#pragma unroll
                        for (int b = 0; b < 4; b++) {
                            f32x4 o;
#pragma unroll
                            for (int r = 0; r < 4; r++) o[r] = d[mt][4 * b + r] + qold[mt][b][r];
                            *(f32x4 *)(Qt + 32 * mt + 8 * b) = o;
                        }
                }
            }
        }
    }
}

// a fibre of X starts at a multiple of the element size, not of 16 bytes
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));

// PTR = false: a fibre of X is addressed by a wave-uniform base and a 32-bit offset of the lane (128 fibres of X are less than
// 2^31 bytes apart).  PTR = true: by a 64-bit pointer of the lane, which may come from the table of blocks of a slab.
template <int NP, int NWC, bool PTR>
__global__ __launch_bounds__(512, 2) void k_mode12_mp(const Mode12Params p, const MpParams mp)
{
    typedef Mode12MpCfg<NP, NWC> cfg;
    typedef std::conditional_t<NP == 1, __bf16, float> T;
    typedef mp_terms<NP> terms;
    constexpr bool F16 = NP == 2;
    constexpr int NWR = cfg::NWR, RT = cfg::RT, CT = cfg::CT, EI = cfg::EI, COLS = cfg::COLS, ROWB = cfg::ROWB, XBUF = cfg::XBUF;
    constexpr int SLOT = cfg::SLOT, NSLOT = cfg::NSLOT, H = cfg::H, DU = cfg::DU, DX = cfg::DX, XD = cfg::XD, NF = 2 * CT;
    constexpr int UNR = lcm_i(lcm_i(NSLOT, DU), DX);
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % NWR, wc = wave / NWR;
    const int nk = (int)(p.k1 - p.k0);
    const int bid = blockIdx.x, xcd = bid & 7, t = bid >> 3;
    // the row groups of one slice sit next to each other on one XCD and share the X tiles through its L2
    const int g = t % p.G, kidx = (t / p.G) * 8 + xcd;
    if (kidx >= nk) return;
    const int64_t k = p.k0 + kidx;
    int t0 = 0, nt = 2 * NWR;   // this group's row tiles: t0 .. t0 + nt - 1
    if (NWC == 1) {
        const int per = mp.T4 / p.G, more = mp.T4 % p.G;
        t0 = 4 * (g * per + (g < more ? g : more));
        nt = 4 * (per + (g < more ? 1 : 0));
    }
    const int wrow0 = 32 * (t0 + wr);   // first row of this wave's tile 0; tile 1 is NWR tiles further
    const bool two = wr + NWR < nt && wrow0 + 32 * NWR < p.PL;
    const int64_t ia0 = p.i0 & ~(int64_t)(EI - 1);
    const int nstage = (int)((p.i1 - ia0 + EI - 1) / EI);
    const int64_t u_tile = mp.nig * (NP * 1024);   // bytes of one row tile of Uf

    u32x4 ufr[DU][2][RT][NP];
    u32x4 xr[DX][NP == 1 ? 1 : 2];
    float xmax = 0.0f, zmax = 0.0f;

    for (int64_t jc = mp.ja0; jc < p.j1; jc += COLS) {
        int tidc = tid;
        asm volatile("" : "+v"(tidc));   // per-lane offsets are derived again in every chunk (not kept live over mode 2)
        const int lane = tidc & 63, l32 = lane & 31, hi = lane >> 5;
        const int col = tidc >> 2, part = tidc & 3;        // this thread's piece of the X tile: 8 values of i of one fibre
        const int xs_w = col * ROWB + part * 16;
        const int xs_r = (wc * CT * 32 + l32) * ROWB + hi * 16;   // + ct*32*ROWB + g2*32 + piece*XBUF
        const bool full = jc >= p.j0 && jc + COLS <= p.j1;
        const bool cok = jc + col >= p.j0 && jc + col < p.j1;
        const int64_t jb = jc > p.j0 ? jc : p.j0, j = cok ? jc + col : jb;   // a lane outside the box reads the chunk's first fibre
        // the thread's values of the stage that starts at i: plain layout at xu + (i - ia0) + xo
        const T *xu = nullptr;       // wave-uniform
        unsigned xo = 0;             // bytes
        const T *xp = nullptr;       // PTR: the lane's pointer for i = ia0
        int64_t tab_end = 0, tab_in = 0;   // table: first i beyond the current block; offset of the fibre inside a block
        const void *const *tabrow = nullptr;
        if constexpr (PTR) {
            if (p.xtab) {
                const int64_t bj = j / p.x_dJ, bk = k / p.x_dK, jb0 = bj * p.x_dJ, djb = (p.j1 - jb0 < p.x_dJ) ? p.j1 - jb0 : p.x_dJ;
                tabrow = p.xtab + (bk * p.tab_nbj + bj) * p.tab_nbi;
                tab_in = (j - jb0) * p.x_dI + (k - bk * p.x_dK) * p.x_dI * djb;
            } else
                xp = (const T *)p.X + (ia0 + 8 * part - p.xo_i) + (j - p.xo_j) * p.x_sj + (k - p.xo_k) * p.x_sk;
        } else {
            xu = (const T *)p.X + (ia0 - p.xo_i) + (jb - p.xo_j) * p.x_sj + (k - p.xo_k) * p.x_sk;
            xo = ((unsigned)(j - jb) * (unsigned)p.x_sj + 8u * (unsigned)part) * (unsigned)sizeof(T);
        }

        f32x16 acc[RT][CT];
        float zero = 0.0f;
        asm volatile("" : "+v"(zero));   // a zero the compiler cannot keep as a 16-register vector across the chunks
#pragma unroll
        for (int rt = 0; rt < RT; rt++)
#pragma unroll
            for (int ct = 0; ct < CT; ct++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[rt][ct][e] = zero;

        // requests this thread's 8 values of stage s (calls come in the order of the stages)
        auto request_x = [&](int s, u32x4 *dst) __attribute__((always_inline)) {
            s = s < nstage ? s : nstage - 1;
            const int64_t ib = ia0 + (int64_t)s * EI;
            const T *a;
            if constexpr (PTR) {
                if (p.xtab) {
                    int64_t i = ib + 8 * part;
                    i = i < p.i1 ? i : p.i1 - 1;
                    if (__any(i >= tab_end)) {   // a block boundary: dI is a multiple of 16, a thread's 8 values lie in one block
                        const int64_t bi = i / p.x_dI;
                        xp = (const T *)tabrow[bi] + tab_in + (8 * part - bi * p.x_dI);
                        tab_end = (bi + 1) * p.x_dI;
                    }
                }
                a = xp + (ib - ia0);
            } else
                a = (const T *)((const char *)(xu + (ib - ia0)) + xo);
            typedef const __attribute__((address_space(1))) T *gp;   // X is device memory whatever the pointer's origin
            if (__builtin_expect(ib >= p.i0 && ib + EI <= p.i1, 1)) {
                if constexpr (NP == 1) dst[0] = *(const __attribute__((address_space(1))) u32x4_a2 *)(gp)a;
                else {
                    dst[0] = *(const __attribute__((address_space(1))) u32x4_a4 *)(gp)a;
                    dst[1] = *(const __attribute__((address_space(1))) u32x4_a4 *)(gp)(a + 4);
                }
            } else {   // first or last stage of a box that does not fill it: value by value, zero outside
                const int64_t i = ib + 8 * part;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const bool ok = i + e >= p.i0 && i + e < p.i1;
                    if constexpr (NP == 1) {
                        const uint32_t v = ok ? (uint32_t)*(const __attribute__((address_space(1))) uint16_t *)(gp)(a + e) : 0u;
                        dst[0][e >> 1] = (e & 1) ? (dst[0][e >> 1] | (v << 16)) : v;
                    } else
                        dst[e >> 2][e & 3] = ok ? *(const __attribute__((address_space(1))) uint32_t *)(gp)(a + e) : 0u;
                }
            }
        };
        uint32_t xw[4][NP];   // the pieces of the tile on its way to LDS
        // splits values 2e, 2e+1 of the requested tile
        auto split_pair = [&](int e, const u32x4 *src) __attribute__((always_inline)) {
            if constexpr (NP > 1) {
                const uint32_t ua = src[e >> 1][2 * (e & 1)], ub = src[e >> 1][2 * (e & 1) + 1];
                const float a = __builtin_bit_cast(float, ua), b = __builtin_bit_cast(float, ub);
                if (NP == 3) xmax = fmaxf(fmaxf(xmax, fabsf(a)), fabsf(b));
                mp_split2<NP, F16, true>(a, b, xw[e]);
            }
        };
        auto store_x = [&](unsigned char *base, const u32x4 *src) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < NP; c++) {
                u32x4 v;
                if constexpr (NP == 1) v = src[0];
                else v = u32x4{xw[0][c], xw[1][c], xw[2][c], xw[3][c]};
                if (!full) v = cok ? v : u32x4{0u, 0u, 0u, 0u};
                *(u32x4 *)(base + c * XBUF + xs_w) = v;
            }
        };
        const int u_lane = lane * 16;
        auto load_u = [&](int rt, int s, int g2, u32x4 *dst) __attribute__((always_inline)) {
            s = s < nstage ? s : nstage - 1;
            const char *b = (const char *)mp.Uf + (int64_t)((wrow0 >> 5) + rt * NWR) * u_tile + ((ia0 >> 4) + 2 * (int64_t)s + g2) * (NP * 1024);
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)b, 0, NP * 1024, 0x00020000);
#pragma unroll
            for (int c = 0; c < NP; c++) dst[c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, u_lane, c * 1024, 0));
        };

        // One stage: the MFMAs of stage s, the tile of stage s+H split and written to its slot, the requests of later stages
        auto stage = [&](auto sic, auto rac, int s) __attribute__((always_inline)) {
            constexpr int SI = decltype(sic)::value, RA = decltype(rac)::value;
            constexpr int US = SI % DU, XS = (SI + H) % DX;
            const unsigned char *cur = smem + (SI % NSLOT) * SLOT;
            unsigned char *oth = smem + ((SI + H) % NSLOT) * SLOT;
            constexpr int NSP = NF < 4 ? NF : 4;   // fragments behind which the split of the tile is dealt out
            u32x4 bx[XD][NP];
            auto load_bx = [&](int f, u32x4 *dst) __attribute__((always_inline)) {
#pragma unroll
                for (int c = 0; c < NP; c++) dst[c] = *(const u32x4 *)(cur + c * XBUF + xs_r + (f % CT) * 32 * ROWB + (f / CT) * 32);
            };
#pragma unroll
            for (int f = 0; f < XD - 1 && f < NF; f++) load_bx(f, bx[f]);
            static_for<NF>([&](auto fc) {
                constexpr int f = decltype(fc)::value, g2 = f / CT, ct = f % CT;
                if constexpr (f + XD - 1 < NF) load_bx(f + XD - 1, bx[(f + XD - 1) % XD]);
                __builtin_amdgcn_sched_barrier(0);
                static_for<terms::N>([&](auto nc) {
                    constexpr int n = decltype(nc)::value;
#pragma unroll
                    for (int rt = 0; rt < RA; rt++) acc[rt][ct] = mp_mma<F16>(bx[f % XD][terms::X[n]], ufr[US][g2][rt][terms::U[n]], acc[rt][ct]);
                });
                if constexpr (ct == CT - 1) {   // last use of these U fragments this stage: refill for stage s+DU
#pragma unroll
                    for (int rt = 0; rt < RA; rt++) load_u(rt, s + DU, g2, ufr[US][g2][rt]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (f < NSP) {
#pragma unroll
                    for (int e = f * 4 / NSP; e < (f + 1) * 4 / NSP; e++) split_pair(e, xr[XS]);
                    if constexpr (f == NSP - 1) {
                        store_x(oth, xr[XS]);
                        request_x(s + H + DX, xr[XS]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        };

        auto run = [&](auto rac) __attribute__((always_inline)) {
            constexpr int RA = decltype(rac)::value;
            // prologue: tiles 0 .. H-1 into the ring, tiles H .. H+DX-1 requested, U of the first stages requested
            {
                u32x4 x0[H][NP == 1 ? 1 : 2];
#pragma unroll
                for (int d = 0; d < H; d++) request_x(d, x0[d]);
#pragma unroll
                for (int d = 0; d < DU; d++)
#pragma unroll
                    for (int g2 = 0; g2 < 2; g2++)
#pragma unroll
                        for (int rt = 0; rt < RA; rt++) load_u(rt, d, g2, ufr[d][g2][rt]);
#pragma unroll
                for (int d = 0; d < DX; d++) request_x(H + d, xr[(H + d) % DX]);
                __syncthreads();   // every wave is done with the slots of the previous chunk
#pragma unroll
                for (int d = 0; d < H; d++) {
#pragma unroll
                    for (int e = 0; e < 4; e++) split_pair(e, x0[d]);
                    store_x(smem + d * SLOT, x0[d]);
                }
                __syncthreads();
            }
            int s = 0;
            auto chain = [&](auto self, auto cc) __attribute__((always_inline)) -> bool {
                constexpr int c = decltype(cc)::value;
                stage(cc, rac, s);
                if (++s >= nstage) return false;
                if constexpr ((c + 1) % H == 0) __syncthreads();
                if constexpr (c + 1 < UNR) return self(self, ic<c + 1>());
                else return true;
            };
            while (chain(chain, ic<0>())) {}
        };
        if (RT == 2 && two) run(ic<2>()); else run(ic<1>());

        if (NP != 2 && mp.flags) {
#pragma unroll
            for (int rt = 0; rt < RT; rt++)
#pragma unroll
                for (int ct = 0; ct < CT; ct++)
#pragma unroll
                    for (int e = 0; e < 16; e += 2) zmax = fmaxf(fmaxf(zmax, fabsf(acc[rt][ct][e])), fabsf(acc[rt][ct][e + 1]));
        }
        const bool first_chunk = (jc == mp.ja0);
        float *Qk = p.Q + ((int64_t)kidx * NWC + wc) * (p.PLpad / NWC) * p.Mpad;
        const int64_t jw = jc + wc * CT * 32;
        const int ntile = two ? 2 : 1;
        if (p.MT == 2) mode2_mp<NP, RT, CT, 2, 32 * NWR>(p, mp, Qk, acc, wrow0, ntile, jw, first_chunk, tid & 63);
        else mode2_mp<NP, RT, CT, 1, 32 * NWR>(p, mp, Qk, acc, wrow0, ntile, jw, first_chunk, tid & 63);
    }
    if (NP != 2 && mp.flags) {
        if (NP == 3) mp_note(mp.flags, MPF_XBIG, MPF_XNORM, MPF_XNZ, xmax, MP_XMIN, MP_XMAX);
        mp_note(mp.flags, MPF_ZBIG, MPF_ZNORM, MPF_ZNZ, zmax, MP_ZMIN, MP_ZMAX);
    }
}

// Stacked fp32 U (rows x cols, leading dimension ld) -> MpParams::Uf, zero padded; a thread makes the 8 values of one lane.
template <int NP>
__global__ __launch_bounds__(256) void k_pack_u_mp(const float *src, int64_t ld, int rows, int64_t cols, u32x4 *dst, int rowtiles, int64_t nig, uint32_t *flags)
{
    float mx = 0.0f;
    const int64_t n = (int64_t)rowtiles * nig * 64;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * 256) {
        const int l = (int)(idx & 63);
        const int64_t f = idx >> 6, ig = f % nig, r = f / nig * 32 + (l & 31), c = ig * 16 + (l >> 5) * 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = (r < rows && c + e < cols) ? src[r * ld + c + e] : 0.0f;
        u32x4 o[NP];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            mx = fmaxf(fmaxf(mx, fabsf(v[2 * e])), fabsf(v[2 * e + 1]));
            uint32_t w[NP];
            mp_split2<NP, NP == 2>(v[2 * e], v[2 * e + 1], w);
#pragma unroll
            for (int q = 0; q < NP; q++) o[q][e] = w[q];
        }
#pragma unroll
        for (int q = 0; q < NP; q++) dst[(f * NP + q) * 64 + l] = o[q];
    }
    if (flags) mp_note(flags, MPF_UBIG, MPF_UNORM, MPF_UNZ, mx, MP_UMIN, MP_UMAX);
}

// Stacked fp32 V (P*M x J) -> MpParams::Vf with vmt = MT, zero padded.
template <int NP>
__global__ __launch_bounds__(256) void k_pack_v_mp(const float *src, int64_t ld, int P, int M, int64_t J, u32x4 *dst, int MT, int64_t nj16, uint32_t *flags)
{
    float mx = 0.0f;
    const int64_t n = (int64_t)P * nj16 * MT * 64;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * 256) {
        const int l = (int)(idx & 63);
        const int64_t f = idx >> 6, mt = f % MT, j16 = f / MT % nj16, pr = f / (MT * nj16), j = 16 * j16 + 4 * (l >> 5);
        const int m = 32 * (int)mt + (l & 31);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int64_t je = j + (e & 3) + 8 * (e >> 2);
            v[e] = (m < M && je < J) ? src[(pr * M + m) * ld + je] : 0.0f;
        }
        u32x4 o[NP];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            mx = fmaxf(fmaxf(mx, fabsf(v[2 * e])), fabsf(v[2 * e + 1]));
            uint32_t w[NP];
            mp_split2<NP, NP == 2>(v[2 * e], v[2 * e + 1], w);
#pragma unroll
            for (int q = 0; q < NP; q++) o[q][e] = w[q];
        }
#pragma unroll
        for (int q = 0; q < NP; q++) dst[(f * NP + q) * 64 + l] = o[q];
    }
    if (flags) mp_note(flags, MPF_VBIG, MPF_VNORM, MPF_VNZ, mx, MP_VMIN, MP_VMAX);
}

}  // namespace exat
