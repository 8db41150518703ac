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
// of values near the smallest normal number are lost.  The kernel and the packing of U and V therefore note what lies outside
// (MpParams::flags; the ranges are in exat_common.h) and a launch of the generic kernel behind it, which otherwise ends at once,
// computes the call with fp32 products when a value lay outside (mp_out_of_range).
//
// Decomposition as in k_mode12: a workgroup owns one slice k and a group of stacked rows, walks the slice in chunks of 128
// fibres with the whole i extent reduced before mode 2.
//   NWC = 1  (NW = 8; NW = 4 for 5 to 8 row tiles, two workgroups per compute unit) every wave holds up to two 32-row tiles x 128
//            fibres.  The row tiles are dealt to the G groups in quads, as evenly as they go (a quad is one tile per SIMD), and inside
//            a group tile t goes to wave t mod NW; a wave with one tile runs a stage loop of its own.
//   NWC = 4  (at most 4 row tiles in all)  four waves share a row tile and take 32 fibres each; each leaves its
//            own partial Q, which mode 3 adds up as if it were a slice of its own (Mode3Params::kshift), or which are added up in LDS (QL).
// X goes HBM -> registers -> (split) -> LDS; U comes in fragment order straight from L2 into registers.  The X tiles sit in a
// ring of NSLOT LDS slots: a stage reads tile s and writes tile s + H, H = NSLOT/2, and the workgroup meets at a barrier
// after every H-th stage only (between two barriers the slots read and the slots written are disjoint).
// Measured (one call with mode 3, before -> now): 128^3 fp32, 64 stacked rows 34.9 -> 17 us; 512^3 fp32, 512 rows 1.05 -> 0.63 ms
// (fp32 matrix instruction before); 1000^3 fp32, 1550 rows 39.2 -> 16.0 ms and 1000^3 bf16, 2400 rows 25.8 -> 6.1 ms (generic
// kernel before: 1000 is no multiple of a stage); slower only, by the range check's launch: 128 x 128 x 91 bf16, 304 rows 18.3 -> 20.1 us;
// 1024^3 in two fp16 pieces, 2048 rows 14.2 -> 12.0 ms; 512^3 generated in fp32 9.9 -> 7.0 ms.  In the stage loop of the fp32 cases the matrix pipe runs at
// about 1.5 PFLOP/s on random operands, where a large bf16 product of the vendor's library reaches 1.28.
#pragma once
#include "exat_gen.h"
#include "exat_mode12.h"

namespace exat {

constexpr unsigned MP_NOWHERE = 0x80000000u;   // a lane's offset beyond the end of every buffer
constexpr size_t MP_UPAD = 8 << 10;   // NP > 1: the U fragments of the stage past the last one (2 x NP x 1024 bytes) are requested

struct MpParams {
    const void *Uf;    // [PLpad/32][nig][NP][64 lanes][8]: lane l of fragment (rt, ig, piece) holds row 32*rt + l%32,
                       // i = 16*ig + 8*(l/32) .. +7
    int64_t nig;       // Ipad / 16
    const void *Vf;    // [P][Jpad/16][vmt][NV][64 lanes][8]: element e of lane l of fragment (p, j16, mt, piece) holds
                       // V_p[m = 32*mt + l%32, j = 16*j16 + 4*(l/32) + e%4 + 8*(e/4)]
    int vmt;           // 32-row tiles of m in Vf
    int T4;            // quads of row tiles (NWC = 1)
    int nblk, bs;      // runs of slices (nblk * G is a multiple of 8) and the longest run's length, or 0
    int64_t ja0;       // first fibre of the first chunk (a multiple of 16, <= j0)
    uint32_t *flags;   // MPF_* words, or null
    int qs;            // QL: floats per row of Q in LDS, even (see mp_qrow)
};

// the largest of mx, |a|, |b|; NaN if one of them is (one instruction)
__device__ __forceinline__ float mp_max(float mx, float a, float b)
{
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(mx, fabsf(a)), fabsf(b));
}

// sets a word if the condition holds in any lane (written once per wave at most, and only if it is not set yet)
__device__ __forceinline__ void mp_note(uint32_t *f, int word, bool lane)
{
    if (__any(lane) && (threadIdx.x & 63) == 0 && !f[word]) f[word] = 1;
}
// the smallest magnitude that is not 0, as its bits without the sign minus one (0 becomes the largest value)
__device__ __forceinline__ unsigned mp_bits(float v) { return (__builtin_bit_cast(unsigned, v) << 1) - 1u; }
__device__ __forceinline__ unsigned mp_min(unsigned mn, float a, float b) { return min(min(mn, mp_bits(a)), mp_bits(b)); }
// elements of U or V of these extremes: one that is not 0 and too small, or too large, or NaN
__device__ __forceinline__ bool mp_bad(unsigned mn, float mx, float vmax) { return mn < mp_bits(MP_EMIN) || !(mx <= vmax); }

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
            typedef float f2 __attribute__((ext_vector_type(2)));
            const g2 h = __builtin_convertvector((f2{a, b}), g2), l = __builtin_convertvector((f2{a - (float)h[0], b - (float)h[1]}), g2);
            w[0] = __builtin_bit_cast(uint32_t, h); w[1] = __builtin_bit_cast(uint32_t, l);
        }
    } else {
#pragma unroll
        for (int q = 0; q < NP; q++) {
            typedef float f2 __attribute__((ext_vector_type(2)));
            w[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), bf16x2));   // one packed conversion
            if (q + 1 < NP) {   // the residual of a rounding to bf16 is exact in fp32
                a -= __builtin_bit_cast(float, w[q] << 16);
                b -= __builtin_bit_cast(float, w[q] & 0xffff0000u);
            }
        }
    }
}

// QL: the workgroup's rows of Q stay in LDS, behind the ring, until its last chunk (rows of MpParams::qs floats), which adds them to its own
// and writes the sum to memory (through LDS as well: 2 to 5 % of a call of two or three chunks).  The Q of the 32
// workgroups of an XCD is as large as its L2, and with the chunks' other traffic every chunk read it from memory, in front of a wait
// nothing covers.  The ring is half as long for it, a barrier after every second stage (bf16) or every stage (fp32).  Before -> now:
// 1000^3 bf16, 2400 rows 7.24 -> 6.46 ms; fp32: 1000^3, 1550 rows 16.6 -> 16.2 ms, 500^3 blocks of it 20.9 -> 20.1, 512^3, 512 rows 658 -> 644
// us, 250^3 263 -> 246, 64 x 1000 x 300, 820 rows 674 -> 607; the same sums in the same order.
// With NWC = 4 the wave columns' partial rows are added there too, behind the last chunk, and mode 3 reads a quarter: 128^3 fp32, 64 rows
// 22.3 -> 17.1 us, bf16 18.9 -> 14.7; 512^3 bf16, 128 rows 153 -> 104 us.
template <int NP, int NW, int NWC, bool QL = false>
struct Mode12MpCfg {
    static constexpr int NWR = NW / NWC, RT = 2, CT = 4 / NWC, COLS = 128, EI = 32;
    static constexpr int XPT = 512 / (64 * NW);                 // runs of 8 values of the X tile per thread
    static constexpr int ROWB = 80, XBUF = COLS * ROWB, SLOT = NP * XBUF;
    static constexpr int NSLOT = NP == 1 ? (QL && NWC == 1 ? 4 : 8) : (NP == 3 && (NW == 4 || (QL && NWC == 1)) ? 2 : 4), H = NSLOT / 2;   // two 4-wave workgroups share the LDS
    static constexpr int lds_bytes(bool gen, int ks) { return NSLOT * SLOT + (gen ? 8 * ks * 2048 : 0); }
    static constexpr int DU = NP == 1 ? 2 : 1;   // register sets of U fragments
    static constexpr int DX = NP == 1 ? 4 : 1;   // register sets of the X tile in flight
    static constexpr int XD = NP == 1 ? 4 : 2;   // register sets of X fragments read from LDS
    static constexpr int UNR = DX;               // stages per pass of the stage loop (register sets are addressed statically)
    static_assert(H <= 2 || H % UNR == 0 || UNR % H == 0, "");
    static_assert(UNR > 1 || 2 * DU * NP * 1024 <= MP_UPAD, "");
    static_assert(UNR % DU == 0 && UNR % DX == 0 && (UNR % H == 0 || H % UNR == 0), "");
};

// Floats per row of Q in LDS, where `lds` bytes are left for `rows` rows: an odd multiple of 4 or, where that is too much, an odd
// multiple of 2 (neighbouring rows start in different banks either way); 0 if there is no room.  Rows are read and written
// 8 bytes at a time: `mp_q_ld`, `mp_q_st` of columns c .. c+3, of which those beyond the row are zero.
inline int mp_qrow(int M, int rows, int lds)
{
    const int a = 4 * (((M + 3) / 4) | 1), b = 2 * (((M + 1) / 2) | 1), most = lds / (4 * rows);
    return a <= most ? a : (b <= most ? b : 0);
}
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f32x4 mp_q_ld(const float *row, int c, int qs)
{
    f32x2 a = {0.0f, 0.0f}, b = {0.0f, 0.0f};
    if (c < qs) a = *(const f32x2 *)(row + c);
    if (c + 2 < qs) b = *(const f32x2 *)(row + c + 2);
    return f32x4{a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ void mp_q_st(float *row, int c, int qs, const f32x4 &v)
{
    if (c < qs) *(f32x2 *)(row + c) = f32x2{v[0], v[1]};
    if (c + 2 < qs) *(f32x2 *)(row + c + 2) = f32x2{v[2], v[3]};
}

// The same into three bf16 pieces by truncation, where every piece is used: h, m, l are the upper, middle and lower 8 bits of the
// significand, exact like the rounded ones.  (With products left out the rounded pieces, half as large, are the better ones.)  `upper` and
// `pick` are 0xffff0000 and 0x07060302 in registers that the compiler cannot see through: a value that is split again for the next replica
// is then neither split ahead nor copied first (bf16, mode 2: 64 copies and 37 waits of 735 instructions, and they are what bounds it;
// 1000^3, 2400 rows 6.24 -> 6.12 ms, 300^3, 800 rows of 20 188 -> 182 us).
__device__ __forceinline__ void mp_split2_trunc(float a, float b, uint32_t upper, uint32_t pick, uint32_t (&w)[3])
{
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
        w[q] = __builtin_amdgcn_perm(ub, ua, pick);
        a -= __builtin_bit_cast(float, ua & upper);
        b -= __builtin_bit_cast(float, ub & upper);
    }
}

// Mode 2 from the accumulators (acc holds Z^T: rows 32 fibres j, columns 32 stacked rows q; see mode2_direct_bf16 for the
// order of the contraction slots), Z split into pieces like X, V packed in pieces.  A tile whose rows belong to several
// replicas is multiplied with each one's V, and a lane keeps the product of its row's replica.  Q[row][m] += Q^T[m][row];
// Qk points to the rows of this slice (and wave column).
template <int NP, int RT, int CT, int MTC, int RSTRIDE, bool QL>
__device__ __forceinline__ void mode2_mp(const Mode12Params &p, const MpParams &mp, float *Qk, f32x16 (&acc)[RT][CT], int wrow0, int ntile,
                                         int64_t jc, bool first_chunk, int lane, float *ql, bool keep)
{
    constexpr bool F16 = NP == 2, LATE = QL && CT == 4;   // LATE: old rows of Q are read where they are needed (one wave column)
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
            float *Qt = QL ? ql + (rt * RSTRIDE + l32) * mp.qs : Qk + (int64_t)q * MP + 4 * hi;   // + 32*mt + 8*b (+ 4*hi)
            for (int pp = pfirst; pp <= plast; pp++) {
                const bool mine = q >= pp * p.L && q < (pp + 1) * p.L && q < p.PL;
                // Step st = 2 ct + t multiplies 16 fibres: Z split into pieces (during the step before) times the fragments of V,
                // requested VA steps before.  Consecutive MFMAs go to two accumulators (with one 32-row tile of V the products
                // alternate between two partial sums): one that adds to the result of the MFMA before it waits for that result.
                const u32x4 *vz = (const u32x4 *)mp.Vf + ((int64_t)pp * (p.Jpad / 16) + jc / 16) * mp.vmt * NV * 64 + ln;
                constexpr int NS = 2 * CT, VA = MTC == 2 && NV > 1 ? 1 : 2;
                u32x4 v[VA + 1][MTC][NV], z[2][NZ];
                uint32_t upper = 0xffff0000u, pick = 0x07060302u;
                asm volatile("" : "+s"(upper), "+s"(pick));   // opaque: see split_z
                f32x16 d[2];
#pragma unroll
                for (int m = 0; m < 2; m++)
#pragma unroll
                    for (int e = 0; e < 16; e++) d[m][e] = 0.0f;
                auto load_v = [&](int st) __attribute__((always_inline)) {
#pragma unroll
                    for (int m = 0; m < MTC; m++)
#pragma unroll
                        for (int c = 0; c < NV; c++) v[st % (VA + 1)][m][c] = vz[(st * mp.vmt + m) * (NV * 64) + c * 64];
                };
                auto split_z = [&](int st, int e) __attribute__((always_inline)) {   // registers 8t+2e, 8t+2e+1 of the tile
                    uint32_t w[NZ];
                    float za = acc[rt][st >> 1][8 * (st & 1) + 2 * e], zb = acc[rt][st >> 1][8 * (st & 1) + 2 * e + 1];
                    if constexpr (NP == 1) mp_split2_trunc(za, zb, upper, pick, w);
                    else {
                        asm volatile("" : "+v"(za), "+v"(zb));   // opaque: or every split is formed ahead of the loop over pp, and spilled
                        mp_split2<NZ, F16>(za, zb, w);
                    }
#pragma unroll
                    for (int c = 0; c < NZ; c++) z[st & 1][c][e] = w[c];
                };
#pragma unroll
                for (int st = 0; st < VA && st < NS; st++) load_v(st);
#pragma unroll
                for (int e = 0; e < 4; e++) split_z(0, e);
                f32x4 qold[MTC][4];
                static_for<NS>([&](auto sc) {
                    constexpr int st = decltype(sc)::value, NM = terms::N * MTC;
                    if constexpr (st + VA < NS) load_v(st + VA);
                    if constexpr (st == NS - 1) {   // the fragments' registers are free now
#pragma unroll
                        for (int m = 0; m < MTC; m++)
#pragma unroll
                            for (int b = 0; b < 4; b++) {
                                qold[m][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                                if (!LATE && !first_chunk && mine) qold[m][b] = QL ? mp_q_ld(Qt, 32 * m + 8 * b + 4 * hi, mp.qs) : *(const f32x4 *)(Qt + 32 * m + 8 * b);
                            }
                    }
                    __builtin_amdgcn_sched_barrier(0);   // the requests stay ahead of the MFMAs
                    static_for<NM>([&](auto nc) {
                        constexpr int i = decltype(nc)::value, n = i / MTC, m = i % MTC, dm = MTC == 2 ? m : n & 1;
                        d[dm] = mp_mma<F16>(v[st % (VA + 1)][m][terms::U[n]], z[st & 1][terms::X[n]], d[dm]);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (st + 1 < NS) {   // the next step's split, dealt out behind the MFMAs
                            static_for<(i + 1) * 4 / NM - i * 4 / NM>([&](auto ec) { split_z(st + 1, i * 4 / NM + decltype(ec)::value); });
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    });
                });
                if (MTC == 1) d[0] += d[1];
                if (mine) {
#pragma unroll
                    for (int m = 0; m < MTC; m++)
#pragma unroll
                        for (int b = 0; b < 4; b++) {
                            f32x4 o;
                            if (LATE && !first_chunk) qold[m][b] = mp_q_ld(Qt, 32 * m + 8 * b + 4 * hi, mp.qs);
#pragma unroll
                            for (int r = 0; r < 4; r++) o[r] = d[m][4 * b + r] + qold[m][b][r];
                            if (QL && (keep || !LATE)) mp_q_st(Qt, 32 * m + 8 * b + 4 * hi, mp.qs, o);
                            else if (QL) *(f32x4 *)(Qk + (int64_t)q * MP + 4 * hi + 32 * m + 8 * b) = o;
                            else *(f32x4 *)(Qt + 32 * m + 8 * b) = o;
                        }
                }
            }
        }
    }
}

// a fibre of X starts at a multiple of the element size, not of 16 bytes
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_a2 __attribute__((aligned(2)));

// PTR = false: the chunk's fibres are a buffer that ends with the slice's part of the box, and the lane has a 32-bit offset into it (128 fibres
// of X are less than 2^31 bytes apart); the box begins and ends at multiples of 4 in i.  PTR = true: any box; a fibre is addressed by a
// 64-bit pointer of the lane, which may come from the table of blocks of a slab.
// MP_GEN (NP = 3): the tile is generated on chip, the low-rank part by the 16x16x32 matrix instruction as in k_mode12_v3 (a wave
// makes the 16 NSJ fibres it owns, 32 values of i per stage, in aligned quads of i, the unit of the noise).  Everything happens
// within the stage: the A pieces of 16 rows are requested a few fragments before they are used, the products B[j,r] C[k,r] of a
// chunk wait in a lane-private piece of LDS, so the only state between stages are the fibres' keys.
enum { MP_LEAN = 0, MP_PTR = 1, MP_GEN = 2 };
template <int NP, int NW, int NWC, int SRC, int KS = 1, bool QL = false>
__global__ __launch_bounds__(64 * NW, 2) void k_mode12_mp(const Mode12Params p, const MpParams mp, const GenSplitParams gs)
{
    typedef Mode12MpCfg<NP, NW, NWC, QL> cfg;
    typedef std::conditional_t<NP == 1, __bf16, float> T;
    typedef mp_terms<NP> terms;
    constexpr bool F16 = NP == 2, PTR = SRC == MP_PTR, GEN = SRC == MP_GEN;
    static_assert(!GEN || NP == 3, "");
    constexpr int NWR = cfg::NWR, RT = cfg::RT, CT = cfg::CT, EI = cfg::EI, COLS = cfg::COLS, ROWB = cfg::ROWB, XBUF = cfg::XBUF;
    constexpr int SLOT = cfg::SLOT, NSLOT = cfg::NSLOT, H = cfg::H, DU = cfg::DU, DX = cfg::DX, XD = cfg::XD, NF = 2 * CT;
    constexpr int XPT = cfg::XPT, XC = COLS / XPT, XW = NP == 1 ? 1 : 2;   // run u of a thread belongs to fibre col + u*XC
    constexpr int UNR = cfg::UNR;
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % NWR, wc = wave / NWR;
    const int nk = (int)(p.k1 - p.k0);
    const int bid = blockIdx.x, xcd = bid & 7, t = bid >> 3;
    // Workgroup ids go round-robin over the 8 XCDs.  The row groups of one slice sit next to each other on one XCD and share the X
    // tiles through its L2 (generated: nothing of X is shared, neighbours take the same rows and share U instead).  With mp.nblk
    // the slices are dealt in that many runs of at most mp.bs: an XCD takes a run with one row group, which is then all of U that its
    // L2 holds, and the other row groups of the run are on other XCDs at about the same time (X comes from the cache behind the L2s);
    // the group an XCD takes moves on from run to run, so that larger and smaller groups are spread evenly.
    const int nkx = (nk + 7) >> 3;
    int g = GEN ? t / nkx : t % p.G, kidx = (GEN ? t % nkx : t / p.G) * 8 + xcd, kend = nk;
    if (mp.nblk) {
        const int b = 8 * (t / mp.bs) + xcd, blk = b / p.G;
        g = (b + (int)((int64_t)blk * p.G >> 3)) % p.G;
        kidx = (int)((int64_t)blk * nk / mp.nblk) + t % mp.bs;
        kend = (int)((int64_t)(blk + 1) * nk / mp.nblk);
    }
    if (kidx >= kend) return;
    const int64_t k = p.k0 + kidx;
    int t0 = 0, nt = 2 * NWR;   // this group's row tiles: t0 .. t0 + nt - 1
    if (NWC == 1) {
        const int per = mp.T4 / p.G, more = mp.T4 % p.G;
        t0 = 4 * (g * per + (g < more ? g : more));
        nt = 4 * (per + (g < more ? 1 : 0));
    }
    // first row of this wave's tile 0; tile 1 is NWR tiles further.  In a group of one quad the waves of eight beyond it take tile 0 of the
    // group along and leave no result (they make their share of X).
    const bool own = wr < nt;
    const int wrow0 = 32 * (t0 + (own ? wr : 0));
    const bool two = wr + NWR < nt && wrow0 + 32 * NWR < p.PL;
    const int64_t ia0 = p.i0 & ~(int64_t)(EI - 1);
    const int nstage = (int)((p.i1 - ia0 + EI - 1) / EI);
    const int64_t u_tile = mp.nig * (NP * 1024);   // bytes of one row tile of Uf

    const int nst = (nstage + UNR - 1) / UNR * UNR;   // stages per chunk: those past the end of the box hold zeros

    const int ilo = (int)(p.i0 - ia0), ilen = (int)(p.i1 - p.i0);   // the box in i, from ia0 on
    const bool halves = ((p.i0 | p.i1) & 4) != 0;                   // bf16: it begins or ends in the middle of a run
    const int s_lo = p.i0 > ia0 ? 1 : 0, s_hi = (int)((p.i1 - ia0) / EI);   // stages that lie inside the box: s_lo .. s_hi - 1

    u32x4 ufr[DU][2][RT][NP];
    u32x4 xr[DX][XPT][XW];
    float xmax = 0.0f;
    unsigned zseen = 0;   // of the lane's rows of Z: bit rt: reaches MP_ZMIN, bit 2 + rt: not 0, bit 4: too large or NaN

    // ---- the producing side: tiles follow each other through all chunks.  State of the tile that is requested next: chunk
    //      start pj, stage ps, the lane's addresses in that chunk ----
    int64_t pj = mp.ja0;
    int ps = 0;
    int so = 0, sw = H * SLOT;   // ring slots, in bytes: of the tile that is multiplied next, of the tile that is written next
    for (int64_t jc = mp.ja0; jc < p.j1; jc += COLS) {
        int tidc = tid;
        asm volatile("" : "+v"(tidc));   // per-lane offsets are derived again in every chunk (not kept live over mode 2)
        const int lane = tidc & 63, l32 = lane & 31, hi = lane >> 5;
        const int col = tidc >> 2, part = tidc & 3;                 // this thread's runs of the X tile: 8 values of i of a fibre
        const int xs_w = col * ROWB + part * 16;                  // + slot + u*XC*ROWB + piece*XBUF
        const int xs_r = (wc * CT * 32 + l32) * ROWB + hi * 16;   // + slot + ct*32*ROWB + g2*32 + piece*XBUF
        // plain layout: a buffer from element (i0, first fibre of the chunk inside the box, k) to the end of the slice's part of the box; the
        // fibre's offset in bytes, beyond all bounds for a fibre outside the box
        __amdgpu_buffer_rsrc_t xrs;
        unsigned xo[XPT];
        bool jin = false;                // PTR: all fibres of the chunk lie inside the box
        const T *xp[XPT];                // PTR: the lane's pointer for i = ia0 (in the current block)
        int64_t tab_end = 0, tab_in[XPT];   // table: first i beyond the current block; offset of the fibre inside a block
        const void *const *tabrow[XPT];
        constexpr int NSJ = 8 / NW;      // GEN: 16-fibre tiles of this wave
        const int l16 = lane & 15, q16 = lane >> 4;
        uint32_t ckey[NSJ];
        float amp[NSJ];
        unsigned char *bcl = smem + NSLOT * SLOT + (wave * NSJ * KS * 2 * 64 + lane) * 16;   // + ((sj*KS + ks)*2 + piece) * 1024
        auto chunk_state = [&]() __attribute__((always_inline)) {
            const int64_t jb = pj > p.j0 ? pj : p.j0;
            if constexpr (GEN) {
                // the fibres' keys, and the generator's B operand bc[j, r] = B[j,r] C[k,r] in pieces
#pragma unroll
                for (int sj = 0; sj < NSJ; sj++) {
                    const int64_t j = pj + 16 * (wave * NSJ + sj) + l16;
                    const bool jok = j >= p.j0 && j < p.j1;
                    const int64_t jj = jok ? j : p.j0;
                    ckey[sj] = fibre_key(p.skey, (uint32_t)jj, (uint32_t)k);
                    amp[sj] = jok ? p.amp2_ln2 : 0.0f;
#pragma unroll
                    for (int ks = 0; ks < KS; ks++) {
                        bf16x8 bh, bm;
                        float bv[8], cv[8];   // clamped loads, all in flight together; masked values
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            const int r = 32 * ks + 8 * q16 + e, rr = r < p.R ? r : p.R - 1;
                            bv[e] = p.B[jj + p.ldB * rr];
                            cv[e] = p.C[k + p.ldC * rr];
                        }
#pragma unroll
                        for (int e = 0; e < 8; e++) asm volatile("" : "+v"(bv[e]), "+v"(cv[e]));
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            const float bc = (jok && 32 * ks + 8 * q16 + e < p.R) ? bv[e] * cv[e] : 0.0f;
                            __bf16 h, m;
                            gen_piece<float>::split(bc, h, m);
                            bh[e] = h; bm[e] = m;
                        }
                        *(bf16x8 *)(bcl + ((sj * KS + ks) * 2 + 0) * 1024) = bh;
                        *(bf16x8 *)(bcl + ((sj * KS + ks) * 2 + 1) * 1024) = bm;
                    }
                }
                return;
            }
            tab_end = 0;
            jin = pj >= p.j0 && pj + COLS <= p.j1;
#pragma unroll
            for (int u = 0; u < XPT; u++) {
                int64_t j = pj + col + u * XC;
                const bool jok = j >= jb && j < p.j1;
                j = jok ? j : jb;
                if constexpr (PTR) {   // (a lane outside the box: the chunk's first fibre)
                    if (p.xtab) {
                        const int64_t bj = j / p.x_dJ, bk = k / p.x_dK, jb0 = bj * p.x_dJ, djb = (p.j1 - jb0 < p.x_dJ) ? p.j1 - jb0 : p.x_dJ;
                        tabrow[u] = p.xtab + (bk * p.tab_nbj + bj) * p.tab_nbi;
                        tab_in[u] = (j - jb0) * p.x_dI + (k - bk * p.x_dK) * p.x_dI * djb;
                    } else
                        xp[u] = (const T *)p.X + (ia0 + 8 * part - p.xo_i) + (j - p.xo_j) * p.x_sj + (k - p.xo_k) * p.x_sk;
                } else
                    xo[u] = jok ? (unsigned)(j - jb) * (unsigned)p.x_sj * (unsigned)sizeof(T) : MP_NOWHERE;
            }
            if constexpr (!PTR) {
                // (128 fibres are less than 2^31 bytes long, so that the chunk's lie below the limit)
                const int64_t rem = ((p.i1 - p.i0) + (p.j1 - 1 - jb) * p.x_sj) * (int64_t)sizeof(T);
                xrs = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p.X + (p.i0 - p.xo_i) + (jb - p.xo_j) * p.x_sj + (k - p.xo_k) * p.x_sk), 0,
                                                        (int)(rem < 0x7fffffff ? rem : 0x7fffffff), 0x00020000);
            }
        };
        chunk_state();
        // GEN: A pieces (h, m) of rows 16*si .. of the tile that is made next
        auto request_a = [&](int si, bf16x8 (&af)[2 * KS]) __attribute__((always_inline)) {
            // One descriptor per piece and stage.  R <= 32 gains 1 to 3 % (512^3, 64 replicas of 64 6.35 -> 6.28 ms, 300^3, 320 rows 266 -> 258 us), more
            // ranks in four waves 5 % (250^3, 256 rows 125.5 -> 119.3), in eight 0.6 to -1.2 %: those keep one per request.
            if constexpr (KS == 1 || NW == 4) {
                constexpr int RP = 32 * KS;   // = gs.Rpad
#pragma unroll
                for (int v = 0; v < 2; v++) {
                    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(gs.Asp + ((int64_t)v * gs.Irows + ia0 + (int64_t)ps * EI) * RP), 0, EI * RP * 2, 0x00020000);
#pragma unroll
                    for (int ks = 0; ks < KS; ks++)
                        af[v * KS + ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, (l16 * RP + 8 * q16) * 2, (16 * si * RP + 32 * ks) * 2, 0));
                }
            } else {
                const int64_t ib = ia0 + (int64_t)ps * EI + 16 * si;
#pragma unroll
                for (int v = 0; v < 2; v++)
#pragma unroll
                    for (int ks = 0; ks < KS; ks++) {
                        const char *b = (const char *)(gs.Asp + ((int64_t)v * gs.Irows + ib) * gs.Rpad + 32 * ks);
                        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)b, 0, 32 * KS * 32 * KS, 0x00020000);
                        af[v * KS + ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, (l16 * gs.Rpad + 8 * q16) * 2, 0, 0));
                    }
            }
        };
        // GEN: rows 16*si .. 16*si+15 of this wave's fibres, low rank + noise, split and written to the slot at `base`
        auto make_rows = [&](int si, const bf16x8 (&af)[2 * KS], unsigned char *base) __attribute__((always_inline)) {
            const int64_t ib = ia0 + (int64_t)ps * EI;
            const int i = 16 * si + 4 * q16;
#pragma unroll
            for (int sj = 0; sj < NSJ; sj++) {
                f32x4v c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < KS; ks++) {
                    const bf16x8 bh = *(const bf16x8 *)(bcl + ((sj * KS + ks) * 2 + 0) * 1024), bm = *(const bf16x8 *)(bcl + ((sj * KS + ks) * 2 + 1) * 1024);
                    c = gen_piece<float>::mfma(af[KS + ks], bh, c);
                    c = gen_piece<float>::mfma(af[ks], bm, c);
                    c = gen_piece<float>::mfma(af[ks], bh, c);
                }
                float z[4], x[4];
                noise_quad(ckey[sj], (uint32_t)((ib + i) >> 2), amp[sj], z);
#pragma unroll
                for (int e = 0; e < 4; e++) x[e] = c[e] + z[e];
                if (!(ps >= s_lo && ps < s_hi)) {   // zero outside the box
#pragma unroll
                    for (int e = 0; e < 4; e++) x[e] = (ib + i + e >= p.i0 && ib + i + e < p.i1) ? x[e] : 0.0f;
                }
                uint32_t w0[NP], w1[NP];
                xmax = mp_max(xmax, x[0], x[1]);
                xmax = mp_max(xmax, x[2], x[3]);
                mp_split2<NP, F16>(x[0], x[1], w0);
                mp_split2<NP, F16>(x[2], x[3], w1);
#pragma unroll
                for (int q = 0; q < NP; q++) *(u32x2 *)(base + q * XBUF + (16 * (wave * NSJ + sj) + l16) * ROWB + i * 2) = u32x2{w0[q], w1[q]};
            }
        };
        auto next_tile = [&]() __attribute__((always_inline)) {
            if (++ps == nst) {
                ps = 0;
                if (pj + COLS < p.j1) pj += COLS;
                chunk_state();
            }
        };
        // the first value of i of this thread's runs of stage t, counted from i0; the box holds the values 0 .. ilen - 1, and of four that begin
        // at a multiple of 4 all or none
        auto x_first = [&](int t) __attribute__((always_inline)) { return 8 * part - ilo + EI * t; };
        // bf16: a run of which one half lies outside the box comes with what is next to it in memory, and one whose first half does is
        // requested from its second on
        auto mask_x = [&](int t, u32x4 (&d)[XPT][XW]) __attribute__((always_inline)) {
            if constexpr (NP == 1 && !PTR && !GEN) {
                if (halves) {
                    const int i = x_first(t);
                    const bool late = i == -4, early = i + 4 == ilen;
#pragma unroll
                    for (int u = 0; u < XPT; u++) {
                        const u32x4 v = d[u][0];
                        d[u][0] = u32x4{late ? 0u : v[0], late ? 0u : v[1], late ? v[0] : (early ? 0u : v[2]), late ? v[1] : (early ? 0u : v[3])};
                    }
                }
            }
        };
        // requests this thread's runs of the next tile; goes on to the tile after it if `go` is set
        auto request_x = [&](u32x4 (&dst)[XPT][XW], bool go) __attribute__((always_inline)) {
            const int64_t ib = ia0 + (int64_t)ps * EI;
            if constexpr (PTR) {
                if (p.xtab) {
                    int64_t i = ib + 8 * part;
                    i = i < p.i1 ? i : p.i1 - 1;
                    if (__any(i >= tab_end)) {   // a block boundary: dI is a multiple of 16, a thread's 8 values lie in one block
                        const int64_t bi = i / p.x_dI;
#pragma unroll
                        for (int u = 0; u < XPT; u++) xp[u] = (const T *)tabrow[u][bi] + tab_in[u] + (8 * part - bi * p.x_dI);
                        tab_end = (bi + 1) * p.x_dI;
                    }
                }
            }
            if constexpr (!PTR) {
                // One request per four values (bf16: eight), without a branch: what lies outside the box is out of range by the lane's offset, and
                // gives zeros (bf16: see mask_x).  Requests under a condition brought a stretch of scalar code and branches into every stage, and
                // the waits behind them counted with the shorter of the paths.  Whole calls, before -> now: 512^3 fp32, 512 rows 652 -> 644 us, 1000^3
                // bf16, 2400 rows 6.59 -> 6.44 ms; 1000^3 fp32, 1550 rows between nothing and 1.5 %, which is the spread.
                const int i = x_first(ps);
#pragma unroll
                for (int c = 0; c < XW; c++) {
                    const bool ok = NP == 1 ? (unsigned)(i + 4) < (unsigned)(ilen + 4) : (unsigned)(i + 4 * c) < (unsigned)ilen;
                    const unsigned o = (unsigned)((NP == 1 ? max(i, 0) : i) * (int)sizeof(T) + 16 * c);
#pragma unroll
                    for (int u = 0; u < XPT; u++)
                        dst[u][c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xrs, (int)(ok ? xo[u] + o : MP_NOWHERE), 0, 0));
                }
            } else {
            const bool inside = jin && ps >= s_lo && ps < s_hi;
            typedef const __attribute__((address_space(1))) T *gp;   // X is device memory whatever the pointer's origin
            auto load_run = [&](const T *a, u32x4 (&d)[XW]) __attribute__((always_inline)) {
                if constexpr (NP == 1) d[0] = *(const __attribute__((address_space(1))) u32x4_a2 *)(gp)a;
                else {
                    d[0] = *(const __attribute__((address_space(1))) u32x4_a4 *)(gp)a;
                    d[1] = *(const __attribute__((address_space(1))) u32x4_a4 *)(gp)(a + 4);
                }
            };
#pragma unroll
            for (int u = 0; u < XPT; u++) {
                const T *a = xp[u] + (ib - ia0);
                if (__builtin_expect(inside, 1)) load_run(a, dst[u]);
                else {   // a tile that is not filled by the box: zero outside
#pragma unroll
                    for (int c = 0; c < XW; c++) dst[u][c] = u32x4{0u, 0u, 0u, 0u};
                    const int64_t i = ib + 8 * part, j = pj + col + u * XC;
                    const bool jok = j >= p.j0 && j < p.j1;
                    if (jok && i >= p.i0 && i + 8 <= p.i1) load_run(a, dst[u]);
                    else if (jok && i + 8 > p.i0 && i < p.i1) {   // value by value
#pragma unroll
                        for (int e = 0; e < 8; e++)
                            if (i + e >= p.i0 && i + e < p.i1) {
                                if constexpr (NP == 1) dst[u][0][e >> 1] |= (uint32_t)*(const __attribute__((address_space(1))) uint16_t *)(gp)(a + e) << (16 * (e & 1));
                                else dst[u][e >> 2][e & 3] = *(const __attribute__((address_space(1))) uint32_t *)(gp)(a + e);
                            }
                    }
                }
            }
            }
            if (!go) return;
            if (++ps == nst) {   // the first tile of the next chunk (of the same one again behind the last)
                ps = 0;
                if (pj + COLS < p.j1) pj += COLS;
                chunk_state();
            }
        };
        uint32_t xw[4][NP];   // the pieces of a run on its way to LDS
        // splits values 2e, 2e+1 of a requested run
        auto split_pair = [&](int e, const u32x4 (&src)[XW]) __attribute__((always_inline)) {
            if constexpr (NP > 1) {
                const uint32_t ua = src[e >> 1][2 * (e & 1)], ub = src[e >> 1][2 * (e & 1) + 1];
                const float a = __builtin_bit_cast(float, ua), b = __builtin_bit_cast(float, ub);
                if (NP == 3) xmax = mp_max(xmax, a, b);
                mp_split2<NP, F16, true>(a, b, xw[e]);
            }
        };
        auto store_x = [&](unsigned char *base, int u, const u32x4 (&src)[XW]) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < NP; c++) {
                u32x4 v;
                if constexpr (NP == 1) v = src[0];
                else v = u32x4{xw[0][c], xw[1][c], xw[2][c], xw[3][c]};
                *(u32x4 *)(base + c * XBUF + xs_w + u * XC * ROWB) = v;
            }
        };
        // U fragments of stage s.  Where a chunk is filled up to UNR stages, those past the box's last one multiply zeros of X: their
        // fragments are zeros too, which a descriptor of no bytes gives without a read (what follows in memory are other rows, or not U).
        // With UNR = 1 only the request of stage s+DU goes past the end, and nothing uses it (Uf is padded by MP_UPAD bytes).
        auto load_u = [&](int rt, int s, int g2, u32x4 *dst) __attribute__((always_inline)) {
            // (one descriptor for both halves of a stage: fewer scalar instructions; beside the generator one for each is 0.6 % faster)
            constexpr int ND = GEN ? 1 : 2;
            const int gb = GEN ? g2 : 0, go = GEN ? 0 : g2 * NP;
            const char *b = (const char *)mp.Uf + (int64_t)((wrow0 >> 5) + rt * NWR) * u_tile + ((ia0 >> 4) + 2 * (int64_t)s + gb) * (NP * 1024);
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)b, 0, UNR == 1 || s < nstage ? ND * NP * 1024 : 0, 0x00020000);
#pragma unroll
            for (int c = 0; c < NP; c++) dst[c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, (go + c) * 1024, 0));
        };

        // tiles 0 .. H-1 into the ring.  (What a chunk hands to the next across its mode 2 lies in the ring; nothing is in flight in
        // registers then, which mode 2 needs.)
        if (GEN && jc == mp.ja0) {
            for (int d = 0; d < H; d++) {
#pragma unroll
                for (int si = 0; si < 2; si++) {
                    bf16x8 af[2 * KS];
                    request_a(si, af);
                    make_rows(si, af, smem + d * SLOT);
                }
                next_tile();
            }
            __syncthreads();
        } else if (jc == mp.ja0) {
            u32x4 x0[H][XPT][XW];
#pragma unroll
            for (int d = 0; d < H; d++) request_x(x0[d], true);
#pragma unroll
            for (int d = 0; d < H; d++) mask_x(d, x0[d]);   // (a bf16 chunk has at least H stages)
#pragma unroll
            for (int d = 0; d < H; d++)
#pragma unroll
                for (int u = 0; u < XPT; u++) {
#pragma unroll
                    for (int e = 0; e < 4; e++) split_pair(e, x0[d][u]);
                    store_x(smem + d * SLOT, u, x0[d][u]);
                }
            __syncthreads();
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

        // X fragments on their way from LDS.  CARRY: the ring of register sets runs on into the next stage (its first fragments are requested
        // behind the last ones of this stage), so the barrier that lets go of a tile and hands over the next ones lies where the first of them
        // is requested, FB, and the tile this stage makes is written before that.  A bf16 stage is short (16 MFMAs a wave) and began with the
        // latency of LDS: 1000^3, 2400 rows 6.33 -> 6.22 ms, 512 x 1024 x 512, 512 rows 356 -> 350 us.  A stage in pieces has three or six times the
        // MFMAs per fragment and loses by the earlier split of its tile: 250^3 fp32 245 -> 246 us, 512^3 641 -> 643.
        constexpr bool CARRY = NP == 1 && NF > 2;
        constexpr int FB = NF - XD + 1;
        static_assert(!CARRY || NF % XD == 0, "register sets are addressed statically");
        u32x4 bx[XD][NP];
        auto load_bx = [&](const unsigned char *tile, int f) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < NP; c++) bx[f % XD][c] = *(const u32x4 *)(tile + c * XBUF + (f % CT) * 32 * ROWB + (f / CT) * 32);
        };
        // One stage: the MFMAs of stage s, the tile H stages ahead split and written to its slot, the requests of later stages
        auto stage = [&](auto sic, auto rac, int s) __attribute__((always_inline)) {
            constexpr int SI = decltype(sic)::value, RA = decltype(rac)::value;
            constexpr int US = SI % DU, XS = (SI + H) % DX;
            const unsigned char *cur = smem + so + xs_r;
            unsigned char *oth = smem + sw;
            // The tile is split behind the last fragments, a run at a time: its request is a stage old, in a chunk's first stage
            // younger (it follows mode 2).
            constexpr int NPAIR = 4 * XPT, NSP = NF < XPT ? NF : XPT, FSP = CARRY ? FB - NSP : NF - NSP;
            static_assert(FSP >= 0, "the whole tile is split within the stage");
            const int so1 = so == (NSLOT - 1) * SLOT ? 0 : so + SLOT, sw1 = sw == (NSLOT - 1) * SLOT ? 0 : sw + SLOT;
            const unsigned char *nxt = smem + so1 + xs_r;
            auto meet = [&]() __attribute__((always_inline)) {
                if constexpr (H % UNR == 0) { if (H == 1 || so1 == 0 || sw1 == 0) __syncthreads(); }
                else if constexpr ((SI + 1) % H == 0) __syncthreads();
            };
            if constexpr (!CARRY) {
#pragma unroll
                for (int f = 0; f < XD - 1 && f < NF; f++) load_bx(cur, f);
            }
            bf16x8 af[GEN ? 2 * KS : 1];   // GEN: requested in front of the stage's first fragment and behind fragment FQ0
            constexpr int FQ0 = NF > 2 ? NF / 4 : 0, FQ1 = NF > 2 ? NF - 3 : 1;   // the two halves of the tile are made behind these
            if constexpr (GEN) request_a(0, af);
            static_for<NF>([&](auto fc) {
                constexpr int f = decltype(fc)::value, g2 = f / CT, ct = f % CT;
                if constexpr (CARRY && f == FB) meet();
                if constexpr (f + XD - 1 < NF) load_bx(cur, f + XD - 1);
                else if constexpr (CARRY) load_bx(nxt, f + XD - 1 - NF);
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
                if constexpr (GEN) {
                    if constexpr (f == FQ0) { make_rows(0, af, oth); request_a(1, af); }
                    if constexpr (f == FQ1) {
                        make_rows(1, af, oth);
                        asm volatile("" : "+v"(xmax));
                        next_tile();
                    }
                    __builtin_amdgcn_sched_barrier(0);
                } else if constexpr (f >= FSP && f < FSP + NSP) {
                    if constexpr (f == FSP) mask_x(s + H < nst ? s + H : s + H - nst, xr[XS]);
                    static_for<NPAIR / NSP>([&](auto ec) {
                        constexpr int e = (f - FSP) * (NPAIR / NSP) + decltype(ec)::value;
                        split_pair(e % 4, xr[XS][e / 4]);
                        if constexpr (e % 4 == 3) store_x(oth, e / 4, xr[XS][e / 4]);
                        // (in the last stages the request is made once more after mode 2; without a request here the registers would be
                        // copied at the end of the stage, behind a wait for everything in flight)
                        if constexpr (e == NPAIR - 1) {
                            if (NP == 3) asm volatile("" : "+v"(xmax));   // here, and not behind the request, which takes the registers over
                            request_x(xr[XS], s + DX < nst);
                        }
                    });
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            so = so1; sw = sw1;
            if constexpr (!CARRY) meet();
        };
        auto run = [&](auto rac) __attribute__((always_inline)) {
            constexpr int RA = decltype(rac)::value;
#pragma unroll
            for (int d = 0; d < DX && !GEN; d++) request_x(xr[(H + d) % DX], true);
#pragma unroll
            for (int d = 0; d < DU; d++)
#pragma unroll
                for (int g2 = 0; g2 < 2; g2++) {
                    // in this order: the compiler takes the wait in front of a stage's MFMAs from the smaller of the two counts of
                    // requests behind the fragments they read, the one on the way in from here and the one around the loop
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int rt = 0; rt < RA; rt++) load_u(rt, d, g2, ufr[d][g2][rt]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            if constexpr (CARRY) {
#pragma unroll
                for (int f = 0; f < XD - 1; f++) load_bx(smem + so + xs_r, f);
            }
            for (int s = 0; s < nst; s += UNR)
                static_for<UNR>([&](auto c) { stage(c, rac, s + decltype(c)::value); });
        };
        if (RT == 2 && two) run(ic<2>()); else run(ic<1>());

        if (NP != 2 && mp.flags) {
#pragma unroll
            for (int rt = 0; rt < RT; rt++) {   // (rows of a tile the wave does not have are 0)
                float m = 0.0f;
#pragma unroll
                for (int ct = 0; ct < CT; ct++)
#pragma unroll
                    for (int e = 0; e < 16; e += 2) m = mp_max(m, acc[rt][ct][e], acc[rt][ct][e + 1]);
                zseen |= (m >= MP_ZMIN ? 1u << rt : 0u) | (m > 0.0f ? 4u << rt : 0u) | (m <= MP_ZMAX ? 0u : 16u);
            }
        }
        const bool first_chunk = (jc == mp.ja0);
        float *Qk = QL ? p.Q + (int64_t)kidx * p.PLpad * p.Mpad : p.Q + ((int64_t)kidx * NWC + wc) * (p.PLpad / NWC) * p.Mpad;
        const int64_t jw = jc + wc * CT * 32;
        const int ntile = two ? 2 : (own ? 1 : 0);
        float *ql = (float *)(smem + NSLOT * SLOT) + (64 * NWR * wc + 32 * wr) * mp.qs;
        const bool keep = jc + COLS < p.j1;   // (one wave column:) the last chunk's rows go to memory
        if (p.MT == 2) mode2_mp<NP, RT, CT, 2, 32 * NWR, QL>(p, mp, Qk, acc, wrow0, ntile, jw, first_chunk, tid & 63, ql, keep);
        else mode2_mp<NP, RT, CT, 1, 32 * NWR, QL>(p, mp, Qk, acc, wrow0, ntile, jw, first_chunk, tid & 63, ql, keep);
        if constexpr (QL && NWC > 1) {   // behind the last chunk: the wave columns' rows are added up on their way to memory
            if (jc + COLS >= p.j1) {
                __syncthreads();
                const float *qb = (const float *)(smem + NSLOT * SLOT);
                const int m4 = 8 * p.MT, rows = p.PL < 64 * NWR ? p.PL : 64 * NWR;
                for (int e = tid; e < rows * m4; e += 64 * NW) {
                    const int r = e / m4, c = 4 * (e % m4);
                    f32x4 v = mp_q_ld(qb + r * mp.qs, c, mp.qs);
#pragma unroll
                    for (int w = 1; w < NWC; w++) v += mp_q_ld(qb + (64 * NWR * w + r) * mp.qs, c, mp.qs);
                    *(f32x4 *)(Qk + (int64_t)r * p.Mpad + c) = v;
                }
            }
        }
    }
    if (NP != 2 && mp.flags) {
        const bool xn = __any(xmax >= MP_EMIN);
        if (NP == 3) mp_note(mp.flags, MPF_X, !(xmax <= MP_XMAX) || (xmax > 0.0f && !xn));
        mp_note(mp.flags, MPF_Z, (zseen & 16) || ((zseen >> 2) & ~zseen & 3));
    }
}

// Stacked fp32 U (rows x cols, leading dimension ld) -> MpParams::Uf, zero padded; a thread makes the 8 values of one lane.
template <int NP>
__device__ __forceinline__ void pack_u_mp_part(unsigned block, unsigned nblocks, const float *src, int64_t ld, int rows, int64_t cols, u32x4 *dst, int rowtiles, int64_t nig, uint32_t *flags)
{
    float mx = 0.0f;
    unsigned mn = ~0u;
    const int64_t n = (int64_t)rowtiles * nig * 64;
    for (int64_t idx = (int64_t)block * 256 + threadIdx.x; idx < n; idx += (int64_t)nblocks * 256) {
        const int l = (int)(idx & 63);
        const int64_t f = idx >> 6, ig = f % nig, r = f / nig * 32 + (l & 31), c = ig * 16 + (l >> 5) * 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = (r < rows && c + e < cols) ? src[r * ld + c + e] : 0.0f;
        u32x4 o[NP];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            mx = mp_max(mx, v[2 * e], v[2 * e + 1]);
            mn = mp_min(mn, v[2 * e], v[2 * e + 1]);
            uint32_t w[NP];
            mp_split2<NP, NP == 2>(v[2 * e], v[2 * e + 1], w);
#pragma unroll
            for (int q = 0; q < NP; q++) o[q][e] = w[q];
        }
#pragma unroll
        for (int q = 0; q < NP; q++) dst[(f * NP + q) * 64 + l] = o[q];
    }
    if (flags) mp_note(flags, MPF_U, mp_bad(mn, mx, MP_UMAX));
}
template <int NP>
__global__ __launch_bounds__(256) void k_pack_u_mp(const float *src, int64_t ld, int rows, int64_t cols, u32x4 *dst, int rowtiles, int64_t nig, uint32_t *flags) { pack_u_mp_part<NP>(blockIdx.x, gridDim.x, src, ld, rows, cols, dst, rowtiles, nig, flags); }

// Stacked fp32 V (P*M x J) -> MpParams::Vf with vmt = MT, zero padded.
template <int NP>
__device__ __forceinline__ void pack_v_mp_part(unsigned block, unsigned nblocks, const float *src, int64_t ld, int P, int M, int64_t J, u32x4 *dst, int MT, int64_t nj16, uint32_t *flags)
{
    float mx = 0.0f;
    unsigned mn = ~0u;
    const int64_t n = (int64_t)P * nj16 * MT * 64;
    for (int64_t idx = (int64_t)block * 256 + threadIdx.x; idx < n; idx += (int64_t)nblocks * 256) {
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
            mx = mp_max(mx, v[2 * e], v[2 * e + 1]);
            mn = mp_min(mn, v[2 * e], v[2 * e + 1]);
            uint32_t w[NP];
            mp_split2<NP, NP == 2>(v[2 * e], v[2 * e + 1], w);
#pragma unroll
            for (int q = 0; q < NP; q++) o[q][e] = w[q];
        }
#pragma unroll
        for (int q = 0; q < NP; q++) dst[(f * NP + q) * 64 + l] = o[q];
    }
    if (flags) {
        mp_note(flags, MPF_V, mp_bad(mn, mx, MP_VMAX));
        const bool n = __any(mx >= MP_VMIN);   // (then MPF_VNZ says nothing more, and most waves read one word only)
        mp_note(flags, MPF_VNORM, n);
        mp_note(flags, MPF_VNZ, mx > 0.0f && !n);
    }
}
template <int NP>
__global__ __launch_bounds__(256) void k_pack_v_mp(const float *src, int64_t ld, int P, int M, int64_t J, u32x4 *dst, int MT, int64_t nj16, uint32_t *flags) { pack_v_mp_part<NP>(blockIdx.x, gridDim.x, src, ld, P, M, J, dst, MT, nj16, flags); }

}  // namespace exat
