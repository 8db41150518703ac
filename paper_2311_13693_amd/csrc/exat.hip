// C ABI of the exat library (declarations and contracts in include/exat.h): argument
// validation, plan/workspace management and kernel launches.  No compute happens on the host.
#include "../../include/exat.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "exat_aux.h"
#include "exat_mode12.h"
#include "exat_mode12_v3.h"
#include "exat_mode12_v4.h"
#include "exat_mode12_mp.h"

using namespace exat;

namespace {

constexpr int64_t kMaxExtent = 2147483647LL - 64;
constexpr int64_t kSlotBudgetBytes = 4LL << 30;

}  // namespace

struct exat_plan_s {
    exat_desc_t d;
    int PL, PLpad, Mpad, MT, Npad;
    int64_t Ipad, Jpad;
    void *arena = nullptr;  // the allocation that holds the arrays below up to Q, the range words and Asplit
    void *Upack = nullptr;
    void *Ufrag = nullptr;  // bf16 plans: U in MFMA fragment order (k_pack_u_frag), same size as Upack
    void *Vfragz = nullptr; // bf16 plans: V in the fragment order of mode2_direct_bf16 (k_pack_v_frag with perm = 1)
    void *Vfrag = nullptr;  // bf16 plans: V in bf16 MFMA fragment order (k_pack_v_frag)
    void *Ump = nullptr, *Vmp = nullptr;   // fp32 plans: three bf16 pieces of U and V (MpParams)
    void *Usp = nullptr, *Vsp = nullptr;   // split plans: two fp16 pieces
    uint32_t *ranges = nullptr;            // value ranges noted by the pack kernels and k_mode12_mp (MPF_*)
    float *Vpack = nullptr, *Wpack = nullptr, *Q = nullptr;
    bool factors_set = false;
    // block-streamed state
    float *slots = nullptr;
    unsigned char *used_dev = nullptr;
    int nslots = 0;
    int64_t nblocks = 0, ysize = 0;
    std::vector<unsigned char> submitted, slot_used;
    int64_t nsubmitted = 0;
    const void **xtab = nullptr;   // device: one pointer per block of X (exat_compress_blocks), [nbk][nbj][nbi]
    // host-streamed compression: ring of device block buffers, a copy stream, and per buffer an event "copy done"
    // (recorded on the copy stream) and an event "buffer consumed" (recorded on the compute stream)
    static constexpr int kRing = 3;
    void *ring[kRing] = {nullptr, nullptr, nullptr};
    hipStream_t copy_stream = nullptr;
    hipEvent_t ev_copied[kRing] = {nullptr, nullptr, nullptr}, ev_free[kRing] = {nullptr, nullptr, nullptr};
    bool ring_used[kRing] = {false, false, false};
    // optional per-kernel timing
    // a ring of event triples, one per compress call, so that a caller can time many calls without waiting in between
    static constexpr int kTimeRing = 128;
    bool timing = false;
    int64_t timed_calls = 0;
    hipEvent_t evr[kTimeRing][3] = {};
    __bf16 *Asplit = nullptr;  // the two 16-bit pieces of the generator's A factor (bf16 or fp16 bit patterns), [2][Ipad][64]
};

namespace {

inline int64_t ceil_to(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
// extent of block b along an axis of length n cut into pieces of d (the last piece may be shorter)
inline int64_t blk_ext(int64_t n, int64_t d, int64_t b) { return (b + 1) * d <= n ? d : n - b * d; }
inline size_t esize(int dt) { return dt == EXAT_BF16 ? 2 : 4; }

int env_int(const char *name, int dflt)
{
    const char *s = getenv(name);
    return s ? atoi(s) : dflt;
}

// row-tile count per wave of the mode-1/2 kernel (workgroup rows = 128*rt)
int choose_rt(const exat_plan_s *pl, bool generated)
{
    const int forced = env_int("EXAT_RT", 0);
    if (pl->d.in_dtype == EXAT_BF16) {
        if (forced == 2 || forced == 5) return forced;
        return pl->PL > 512 ? 5 : 2;
    }
    if (forced == 1 || forced == 2 || forced == 4) return forced;
    if (pl->PL <= 128) return 1;
    if (generated && pl->PL >= 512) return 4;
    return 2;
}

int validate_desc(const exat_desc_t *d)
{
    if (!d) return EXAT_ERR_NULL;
    if (d->in_dtype != EXAT_F32 && d->in_dtype != EXAT_BF16 && d->in_dtype != EXAT_F32_SPLIT) return EXAT_ERR_DTYPE;
    if (d->I < 1 || d->J < 1 || d->K < 1 || d->I > kMaxExtent || d->J > kMaxExtent || d->K > kMaxExtent) return EXAT_ERR_SHAPE;
    if (d->L < 1 || d->M < 1 || d->N < 1 || d->P < 1 || d->M > 64) return EXAT_ERR_SHAPE;
    if ((int64_t)d->P * d->L >= (1 << 24) || (int64_t)d->P * d->N >= (1 << 24)) return EXAT_ERR_SHAPE;
    if (d->dI < 1 || d->dJ < 1 || d->dK < 1) return EXAT_ERR_SHAPE;
    if (d->dI > d->I || d->dJ > d->J || d->dK > d->K) return EXAT_ERR_SHAPE;
    return EXAT_OK;
}

int validate_gen(const exat_gen_t *g)
{
    if (!g || !g->A || !g->B || !g->C) return EXAT_ERR_NULL;
    if (g->R < 1 || g->R > 256) return EXAT_ERR_SHAPE;
    if (!(g->sigma >= 0.0f) || !(g->sigma < 1e18f)) return EXAT_ERR_SHAPE;
    return EXAT_OK;
}

unsigned grid_for(int64_t n) { int64_t g = (n + 255) / 256; return (unsigned)(g > 65536 ? 65536 : (g < 1 ? 1 : g)); }

float amp2_ln2_of(float sigma) { return sigma == 0.0f ? 0.0f : (float)(-2.0 * 0.69314718055994530942 * (double)sigma * (double)sigma); }

template <typename T, int RT, int CT, int SRC>
int launch_mode12_inst(const Mode12Params &mp, int nk, hipStream_t st)
{
    typedef Mode12Cfg<T, RT, CT> cfg;
    auto kern = k_mode12<T, RT, CT, SRC>;
    static bool attr_done = false;  // per instantiation; setting it twice is harmless
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, cfg::LDS_BYTES) != hipSuccess) return EXAT_ERR_HIP;
        attr_done = true;
    }
    const int64_t grid = 8LL * ((nk + 7) / 8) * mp.G;
    if (grid > 2147483647LL) return EXAT_ERR_SHAPE;
    hipLaunchKernelGGL(kern, dim3((unsigned)(mp.guard && grid > 512 ? 512 : grid)), dim3(256), cfg::LDS_BYTES, st, mp);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}

template <int SRC>
int launch_mode12_f32(int rt, const Mode12Params &mp, int nk, hipStream_t st)
{
    switch (rt) {
    case 1: return launch_mode12_inst<float, 1, 4, SRC>(mp, nk, st);
    case 2: return launch_mode12_inst<float, 2, 4, SRC>(mp, nk, st);
    default: return launch_mode12_inst<float, 4, 4, SRC>(mp, nk, st);
    }
}
template <int SRC>
int launch_mode12_bf16(int rt, const Mode12Params &mp, int nk, hipStream_t st)
{
    switch (rt) {
    case 2: return launch_mode12_inst<__bf16, 2, 4, SRC>(mp, nk, st);
    default: return launch_mode12_inst<__bf16, 5, 4, SRC>(mp, nk, st);
    }
}

// bf16 generated source, 4 waves x RT row tiles
template <int RT, int KS, bool BOXED>
int launch_v3_inst(const Mode12Params &mp, const GenSplitParams &gs, const UFragParams &uf, int nk, hipStream_t st)
{
    typedef Mode12V3Cfg<4, RT> cfg;
    auto kern = k_mode12_v3<4, RT, KS, BOXED, 2>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, cfg::LDS_BYTES) != hipSuccess) return EXAT_ERR_HIP;
        attr_done = true;
    }
    const int64_t grid = 8LL * ((nk + 7) / 8) * mp.G;
    if (grid > 2147483647LL) return EXAT_ERR_SHAPE;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), cfg::LDS_BYTES, st, mp, gs, uf);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}
template <int RT>
int launch_v3_gen_bf16(const Mode12Params &mp, const GenSplitParams &gs, const UFragParams &uf, int ks, bool boxed, int nk, hipStream_t st)
{
    if (ks == 1) return boxed ? launch_v3_inst<RT, 1, true>(mp, gs, uf, nk, st) : launch_v3_inst<RT, 1, false>(mp, gs, uf, nk, st);
    return boxed ? launch_v3_inst<RT, 2, true>(mp, gs, uf, nk, st) : launch_v3_inst<RT, 2, false>(mp, gs, uf, nk, st);
}

// bf16 generated source, 8 waves x 2 row tiles (512 stacked rows per group), k_mode12_v4
template <bool BOXED>
int launch_v4_inst(const Mode12Params &mp, const GenSplitParams &gs, const UFragParams &uf, int nk, hipStream_t st)
{
    typedef Mode12V4Cfg<8, 2> cfg;
    auto kern = k_mode12_v4<8, 2, 1, BOXED, 2, 1, 8>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, cfg::LDS_BYTES) != hipSuccess) return EXAT_ERR_HIP;
        attr_done = true;
    }
    const int64_t grid = 8LL * ((nk + 7) / 8) * mp.G;
    if (grid > 2147483647LL) return EXAT_ERR_SHAPE;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), cfg::LDS_BYTES, st, mp, gs, uf);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}
int launch_v4_gen_bf16(const Mode12Params &mp, const GenSplitParams &gs, const UFragParams &uf, bool boxed, int nk, hipStream_t st)
{
    return boxed ? launch_v4_inst<true>(mp, gs, uf, nk, st) : launch_v4_inst<false>(mp, gs, uf, nk, st);
}

template <int NP, int NW, int NWC, int SRC, int KS = 1, bool QL = false>
int launch_mp_inst(const Mode12Params &mp, const MpParams &q, const GenSplitParams &gs, int nk, hipStream_t st)
{
    typedef Mode12MpCfg<NP, NW, NWC, QL> cfg;
    auto kern = k_mode12_mp<NP, NW, NWC, SRC, KS, QL>;
    constexpr int ring = cfg::lds_bytes(SRC == MP_GEN, KS), most = QL ? 160 * 1024 : ring;
    static_assert(ring <= 160 * 1024, "LDS of a compute unit");
    const int lds = ring + (QL ? 2 * 32 * NW * q.qs * 4 : 0);
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, most) != hipSuccess) return EXAT_ERR_HIP;
        attr_done = true;
    }
    const int64_t grid = q.nblk ? (int64_t)q.nblk * mp.G * q.bs : 8LL * ((nk + 7) / 8) * mp.G;
    if (grid > 2147483647LL) return EXAT_ERR_SHAPE;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW), lds, st, mp, q, gs);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}
template <int NP, int NW, int NWC>
int launch_mp_nwc(const Mode12Params &mp, const MpParams &q, const GenSplitParams &gs, bool generated, int nk, hipStream_t st)
{
    if constexpr (NP == 3)
        if (generated) return gs.Rpad == 32 ? launch_mp_inst<NP, NW, NWC, MP_GEN, 1>(mp, q, gs, nk, st) : launch_mp_inst<NP, NW, NWC, MP_GEN, 2>(mp, q, gs, nk, st);
    // the lean build unless X is a set of blocks, the box has odd ends in i, or the fibres are millions of values long
    const bool ptr = mp.xtab || mp.i0 % 4 != 0 || mp.i1 % 4 != 0 || mp.x_sj > (1LL << 31) / (128 * (NP == 1 ? 2 : 4)) - 64;
    if constexpr (NP != 2 && NW == 8)
        if (q.qs) return ptr ? launch_mp_inst<NP, NW, NWC, MP_PTR, 1, true>(mp, q, gs, nk, st) : launch_mp_inst<NP, NW, NWC, MP_LEAN, 1, true>(mp, q, gs, nk, st);
    return ptr ? launch_mp_inst<NP, NW, NWC, MP_PTR>(mp, q, gs, nk, st) : launch_mp_inst<NP, NW, NWC, MP_LEAN>(mp, q, gs, nk, st);
}
template <int NP>
int launch_mp(const Mode12Params &mp, const MpParams &q, const GenSplitParams &gs, bool generated, int nw, int nwc, int nk, hipStream_t st)
{
    if (nwc == 4) return launch_mp_nwc<NP, 8, 4>(mp, q, gs, generated, nk, st);
    return nw == 8 ? launch_mp_nwc<NP, 8, 1>(mp, q, gs, generated, nk, st) : launch_mp_nwc<NP, 4, 1>(mp, q, gs, generated, nk, st);
}

// Number of row groups of k_mode12_mp for T4 quads of row tiles and nk slices: a workgroup holds two to four quads, the
// groups take the quads as evenly as they go, and a compute unit runs one workgroup of eight waves or two of four at a time.
int choose_groups(int T4, int64_t nk, int nw)
{
    int best = 1;
    double cost = 0.0;
    const int mx = nw / 2, mn = nw / 4;
    const double slots = nw == 8 ? 256 : 512;
    for (int G = (T4 + mx - 1) / mx; G <= (T4 + mn - 1) / mn; G++) {
        const double c = std::max(std::ceil((double)nk * G / slots), (double)nk * G / slots) * ((double)T4 / G + 0.5);
        if (G == (T4 + mx - 1) / mx || c < 0.97 * cost) { best = G; cost = c; }
    }
    return best;
}

// Whether rows of Q that fit stay in LDS over the chunks.  They save a read of Q per chunk and halve the ring of X tiles.  2600 calls
// of 33 to 512 values in i, 129 to 768 in j, 40 to 400 slices and 384 to 2048 rows, both builds in turn (speed with over without): with
// more than 32 columns of Q the saving is the larger part (fp32 1.06, never below 1; bf16 1.05), except for bf16 in two chunks of fewer
// than six stages in one round of workgroups that fills the chip (1.0, down to 0.95) and in chunks of two stages where half the compute
// units are idle.  With up to 32 columns Q is half as large: fp32 gains (1.03) but in two chunks of small slices of a single group (0.94
// to 0.98); bf16 gains from 57000 values a slice on (512 rows, 100 by 300: 0.95; 192 by 300: 1.02) or, with replicas of at least a row
// tile and from three stages on, with idle compute units (1.02) or many rows (1280 rows, 1.04).  Where more than two replicas share a
// row tile (each a pass over its rows of Q) it gains from 120000 values on (replicas of 20 rows: 0.96 to 1.02 below, 0.99 to 1.08
// above).  Where i ends inside a piece of four the read of the last stage waits: bf16 gains (1.05, five stages 1.2) unless that is the
// third of four stages (0.85 to 0.98).
bool mp_keep_q(const Mode12Params &mp, const MpParams &q, bool bf, int64_t nk)
{
    const int64_t nj = mp.j1 - q.ja0, ni = mp.i1 - (mp.i0 & ~(int64_t)31), nstage = cdiv(ni, 32);
    if (nj <= 128) return false;
    const bool full = nk * mp.G > 128;
    if (!bf) return mp.MT == 2 || !full || mp.G > 1 || nj > 256 || ni * nj >= 16000;
    if (mp.i0 % 4 != 0 || mp.i1 % 4 != 0) return nstage != 3;
    if (mp.MT == 2) return full ? nj > 256 || nstage >= 6 || nk * mp.G <= 200 || nk * mp.G > 256 : nstage >= 3;
    const int64_t least = mp.L >= 32 || mp.L == 16 ? 57000 : 120000;
    return ni * nj >= least || (mp.L >= 32 && nstage >= 3 && (!full || (q.T4 >= 10 && ni * nj >= 20000)));
}

// Runs of about 32 slices (a workgroup per compute unit of an XCD), as many as give every XCD the same number of (run, row group)
// pairs.
void slice_runs(int G, int64_t nk, int *nblk, int *bs)
{
    int mul = 8;   // the fewest runs whose pairs can be dealt evenly to 8 XCDs: 8 / gcd(G, 8)
    while (mul > 1 && G % (16 / mul) == 0) mul /= 2;
    *nblk = (int)(mul * cdiv(nk, 32 * mul));
    *bs = (int)cdiv(nk, *nblk);
}

template <int NT, int MP, int NW, bool LONGK>
int launch_mode3_inst(const Mode3Params &m3, dim3 grid, size_t lds, hipStream_t st)
{
    auto kern = k_mode3<NT, MP, NW, LONGK>;
    static bool attr_done = false;
    if (lds > 64 * 1024 && !attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return EXAT_ERR_HIP;
        attr_done = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3(64 * NW), lds, st, m3);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}

// mode 3 over the slices of a call whose mode-1/2 launches left 2^kshift partial Q per slice
int run_mode3(exat_plan_s *pl, const Mode12Params &mp, int kshift, float *Yout, int accumulate, unsigned char *flag, hipStream_t st)
{
    Mode3Params m3;
    m3.kshift = kshift; m3.ranges = pl->ranges;
    m3.Q = pl->Q; m3.W = pl->Wpack; m3.Y = Yout;
    m3.L = pl->d.L; m3.M = pl->d.M; m3.N = pl->d.N; m3.PL = pl->PL; m3.PLpad = pl->PLpad >> kshift; m3.Mpad = pl->Mpad;
    m3.Npad = pl->Npad;
    m3.K = pl->d.K; m3.k0 = mp.k0; m3.k1 = mp.k1; m3.accumulate = accumulate; m3.flag = flag;
    // 64-column tiles of n unless that would carry an idle second tile.  Up to one workgroup of one m tile per compute unit and
    // with 16 values of k and more per wave a workgroup gets 16 waves (64 tiles, 512 slices: 10.2 -> 8.7 us; 304 tiles, 91 slices took 16 us
    // with 16 waves, in two rounds that mostly add up), else it takes both m tiles (64 values of m) where there are two.
    const int nt = pl->Npad % 64 == 0 ? 2 : 1, ny = pl->Npad / (32 * nt);
    const int64_t ntile = (int64_t)pl->PL * pl->MT, nkk = (m3.k1 - m3.k0) << kshift;
    const bool many = ntile * ny <= 256 && nkk >= 256 && nkk <= 8000;   // (8000: no slab of 16 waves is longer than 512)
    const int mp2 = !many && pl->MT == 2, nw = many ? 16 : 4;
    const bool longk = !many && nkk > 512LL * nw - 2 * nw;   // a wave's slab (rounded up to even) may exceed 512
    const dim3 grid((unsigned)((ntile / (1 + mp2) + 7) / 8 * 8), (unsigned)ny);
    const size_t lds = (size_t)nw * nt * (1 + mp2) * (longk ? 8192 : 4096);
    int rc;
    if (many) rc = nt == 2 ? launch_mode3_inst<2, 1, 16, false>(m3, grid, lds, st) : launch_mode3_inst<1, 1, 16, false>(m3, grid, lds, st);
    else if (longk && mp2) rc = nt == 2 ? launch_mode3_inst<2, 2, 4, true>(m3, grid, lds, st) : launch_mode3_inst<1, 2, 4, true>(m3, grid, lds, st);
    else if (longk) rc = nt == 2 ? launch_mode3_inst<2, 1, 4, true>(m3, grid, lds, st) : launch_mode3_inst<1, 1, 4, true>(m3, grid, lds, st);
    else if (mp2) rc = nt == 2 ? launch_mode3_inst<2, 2, 4, false>(m3, grid, lds, st) : launch_mode3_inst<1, 2, 4, false>(m3, grid, lds, st);
    else rc = nt == 2 ? launch_mode3_inst<2, 1, 4, false>(m3, grid, lds, st) : launch_mode3_inst<1, 1, 4, false>(m3, grid, lds, st);
    if (rc != EXAT_OK) return rc;
    if (hipGetLastError() != hipSuccess) return EXAT_ERR_HIP;
    if (pl->timing) {
        if (hipEventRecord(pl->evr[pl->timed_calls % exat_plan_s::kTimeRing][2], st) != hipSuccess) return EXAT_ERR_HIP;
        pl->timed_calls++;
    }
    return EXAT_OK;
}

// materialised X, and generated X of fp32 plans: modes 1 and 2 (k_mode12_mp, and behind it the generic kernel for values outside the
// ranges of the piece sums), then mode 3
int run_pieces(exat_plan_s *pl, Mode12Params mp, bool generated, bool pipelined, float *Yout, int accumulate, hipStream_t st, unsigned char *flag)
{
    const bool bf = pl->d.in_dtype == EXAT_BF16;
    const int64_t nk = mp.k1 - mp.k0;
    GenSplitParams gs;
    gs.Asp = pl->Asplit; gs.Irows = pl->Ipad; gs.Rpad = 32 * ((mp.R + 31) / 32);
    if (generated && pipelined) {
        hipLaunchKernelGGL(k_split_a<float>, dim3(grid_for(gs.Irows * gs.Rpad)), dim3(256), 0, st, mp.A, pl->d.I, mp.R, pl->Asplit, gs.Irows, gs.Rpad);
        if (hipGetLastError() != hipSuccess) return EXAT_ERR_HIP;
    }
    mp.U = pl->Upack; mp.V = pl->Vpack; mp.Q = pl->Q;
    mp.I = pl->d.I; mp.Ipad = pl->Ipad; mp.Jpad = pl->Jpad;
    mp.L = pl->d.L; mp.PL = pl->PL; mp.PLpad = pl->PLpad; mp.Mpad = pl->Mpad; mp.MT = pl->MT;
    hipEvent_t *ev = pl->evr[pl->timed_calls % exat_plan_s::kTimeRing];
    if (pl->timing && hipEventRecord(ev[0], st) != hipSuccess) return EXAT_ERR_HIP;
    int rc = EXAT_OK, kshift = 0;
    if (pipelined) {
        // split-precision plans take the fp16 pieces for aligned tensors and blocks with whole 32-value stages of i, and the
        // fp32 path's pieces (no range limit) for the rest
        const bool split = pl->d.in_dtype == EXAT_F32_SPLIT && !generated && mp.x_vec && (mp.i0 % 32 == 0) && ((mp.i1 - mp.i0) % 32 == 0);
        const int T = (pl->PL + 31) / 32;
        // Up to 4 row tiles: 8 waves, four of which share a tile's fibres (with a tile per wave half of them would have nothing to
        // do).  Up to 8: two 4-wave workgroups per compute unit, one's mode 2 under the other's stages (512^3, 256 rows: 0.40 ms with
        // one 8-wave workgroup of one tile per wave, 0.35 ms so).  Else groups of 8 to 16 tiles, one 8-wave workgroup per compute unit:
        // with two of four each would read and split every X tile (the stage took longer).
        const int nwc = T <= 4 ? 4 : 1, nw = T > 4 && T <= 8 ? 4 : 8;
        kshift = nwc == 4 ? 2 : 0;
        MpParams q;
        q.nig = pl->Ipad / 16; q.T4 = (T + 3) / 4;
        q.Uf = bf ? pl->Ufrag : (split ? pl->Usp : pl->Ump);
        q.Vf = bf ? pl->Vfragz : (split ? pl->Vsp : pl->Vmp);
        q.vmt = bf ? 2 : pl->MT;
        q.flags = split ? nullptr : pl->ranges;
        // chunks of 128 fibres from j0 down to a multiple of 16, as long as V's padding covers the last one
        q.ja0 = mp.j0 & ~(int64_t)15;
        if (q.ja0 + 128 * cdiv(mp.j1 - q.ja0, 128) > pl->Jpad) q.ja0 = mp.j0 & ~(int64_t)127;
        mp.G = nwc > 1 ? 1 : choose_groups(q.T4, nk, nw);
        // Q in LDS where the workgroup has its own compute unit, 512 rows of it fit beside the ring and more than one chunk adds to it (up
        // to 50 columns m for fp32, 60 for bf16; see mp_keep_q) or four wave columns do (beside the whole ring, short calls need it: 20
        // and 40); generated sources need the room for their operands, two fp16 pieces have longer rows in the configurations they are
        // used in
        auto room = [&](auto c1, auto c3) { return 160 * 1024 - (bf ? decltype(c1)::lds_bytes(false, 1) : decltype(c3)::lds_bytes(false, 1)); };
        q.qs = 0;
        if (!split && !generated && nwc == 4) q.qs = mp_qrow(pl->d.M, 512, room(Mode12MpCfg<1, 8, 4, true>(), Mode12MpCfg<3, 8, 4, true>()));
        if (!split && !generated && nw == 8 && nwc == 1 && mp_keep_q(mp, q, bf, nk))
            q.qs = mp_qrow(pl->d.M, 512, room(Mode12MpCfg<1, 8, 1, true>(), Mode12MpCfg<3, 8, 1, true>()));
        if (q.qs) kshift = 0;
        q.nblk = q.bs = 0;
        // Row groups of different size drift apart and then neither share X tiles nor leave room for U in the L2 (2400 rows, 1000^3
        // bf16: 37 GB fetched past the L2 in 7.7 ms slice by slice, 17 GB in 7.2 ms in runs): slices in runs, one group per XCD at a time.  Both orders measured, slice by
        // slice -> runs: 1000^3 fp32, 1550 rows 17.9 -> 16.3 ms; 700^3, 2624 rows 11.6 -> 10.7; 1000^3 bf16, 2400 rows 7.48 -> 7.08;
        // 300^3 1.156 -> 1.140; but 250 x 250 x 64 0.154 -> 0.156 (the set-up of a workgroup weighs more).  Equal groups stay in step and
        // gain nothing (1024^3 in four groups 20.8 -> 21.1), two or three groups lose as often as they gain.
        if (!generated && mp.G >= 4 && q.T4 % mp.G != 0 && mp.i1 - mp.i0 >= 288) slice_runs(mp.G, nk, &q.nblk, &q.bs);
        rc = bf ? launch_mp<1>(mp, q, gs, false, nw, nwc, (int)nk, st) : (split ? launch_mp<2>(mp, q, gs, false, nw, nwc, (int)nk, st) : launch_mp<3>(mp, q, gs, generated, nw, nwc, (int)nk, st));
        if (rc != EXAT_OK) return rc;
        mp.guard = q.flags;
        mp.qzero0 = pl->PLpad >> kshift;
    }
    if (!pipelined || mp.guard) {
        const int rt = choose_rt(pl, generated);
        mp.G = (pl->PL + 128 * rt - 1) / (128 * rt);
        if (bf) rc = launch_mode12_bf16<SRC_MATERIALISED>(rt, mp, (int)nk, st);
        else rc = generated ? launch_mode12_f32<SRC_GENERATED>(rt, mp, (int)nk, st) : launch_mode12_f32<SRC_MATERIALISED>(rt, mp, (int)nk, st);
        if (rc != EXAT_OK) return rc;
    }
    if (pl->timing && hipEventRecord(ev[1], st) != hipSuccess) return EXAT_ERR_HIP;
    return run_mode3(pl, mp, kshift, Yout, accumulate, flag, st);
}

// generated source of a bf16 plan: the pipelined generating kernels (or the generic one), then mode 3
int run_generated_bf16(exat_plan_s *pl, Mode12Params mp, bool pipelined, float *Yout, hipStream_t st)
{
    int rt = choose_rt(pl, true);
    if (pipelined) {
        // rt = 128-row units of the workgroup tile: 2 = 4 waves x 2 row tiles, 3 = 4 waves x 3 (384 stacked rows, one wave per SIMD)
        const int forced = env_int("EXAT_RT", 0);
        rt = forced == 2 || (forced != 4 && pl->PL <= 256) ? 2 : 3;
    }
    const int rows = 128 * rt;
    mp.U = pl->Upack; mp.V = pl->Vpack; mp.Q = pl->Q;
    mp.I = pl->d.I; mp.Ipad = pl->Ipad; mp.Jpad = pl->Jpad;
    mp.L = pl->d.L; mp.PL = pl->PL; mp.PLpad = pl->PLpad; mp.Mpad = pl->Mpad; mp.MT = pl->MT;
    mp.G = (pl->PL + rows - 1) / rows;
    const int nk = (int)(mp.k1 - mp.k0);
    int rc;
    GenSplitParams gs;
    gs.Asp = pl->Asplit; gs.Irows = pl->Ipad; gs.Rpad = 32 * ((mp.R + 31) / 32);
    if (pipelined) {
        hipLaunchKernelGGL(k_split_a<__bf16>, dim3(grid_for(gs.Irows * gs.Rpad)), dim3(256), 0, st, mp.A, pl->d.I, mp.R, pl->Asplit, gs.Irows, gs.Rpad);
        if (hipGetLastError() != hipSuccess) return EXAT_ERR_HIP;
    }
    hipEvent_t *ev = pl->evr[pl->timed_calls % exat_plan_s::kTimeRing];
    if (pl->timing && hipEventRecord(ev[0], st) != hipSuccess) return EXAT_ERR_HIP;
    if (pipelined) {
        const bool boxed = (mp.i0 != 0 || mp.i1 != pl->d.I);
        const int ks = gs.Rpad / 32;
        UFragParams uf;
        uf.Uf = pl->Ufrag; uf.nig = pl->Ipad / 16; uf.Vf = pl->Vfrag; uf.Vz = pl->Vfragz;
        if (pl->PL > 256 && ks == 1 && env_int("EXAT_RT", 0) == 0 && pl->Ipad < (1LL << 21)) {
            // 512-row groups, two waves per SIMD (k_mode12_v4): the tile is generated once per group, so large groups
            // are what keeps the generator's vector work below the MFMA work.  Factor ranks above 32 would need twice
            // the generator registers, which this build does not have: they take the 384-row kernel below.  The kernel
            // addresses U and the generator's A pieces with 32-bit byte offsets (a wave's two row tiles are 8 tiles, 576
            // bytes per padded column, apart): 2^21 padded columns and more take the 384-row kernel as well.
            mp.G = (pl->PL + 511) / 512;
            rc = launch_v4_gen_bf16(mp, gs, uf, boxed, nk, st);
        } else if (rt == 3) {
            // 384-row groups; a remainder of at most 256 rows gets a launch of its own with a smaller tile
            // instead of a mostly empty group (the generator's vector work per group does not shrink with
            // the rows, the MFMA work does)
            const int full = pl->PL / 384, rem = pl->PL - 384 * full;
            rc = EXAT_OK;
            if (full > 0 && (rem == 0 || rem <= 256)) {
                mp.G = full;
                rc = launch_v3_gen_bf16<3>(mp, gs, uf, ks, boxed, nk, st);
                if (rc == EXAT_OK && rem > 0) {
                    mp.row_base = 384 * full; mp.G = 1;
                    rc = rem <= 128 ? launch_v3_gen_bf16<1>(mp, gs, uf, ks, boxed, nk, st) : launch_v3_gen_bf16<2>(mp, gs, uf, ks, boxed, nk, st);
                }
            } else
                rc = launch_v3_gen_bf16<3>(mp, gs, uf, ks, boxed, nk, st);
        } else
            rc = launch_v3_gen_bf16<2>(mp, gs, uf, ks, boxed, nk, st);
    } else
        rc = launch_mode12_bf16<SRC_GENERATED>(rt, mp, nk, st);
    if (rc != EXAT_OK) return rc;
    if (pl->timing && hipEventRecord(ev[1], st) != hipSuccess) return EXAT_ERR_HIP;
    return run_mode3(pl, mp, 0, Yout, 0, nullptr, st);
}

// Materialised sources run k_mode12_mp at any size and alignment, and so do generated sources of fp32 plans if the factor rank
// fits the generator; generated sources of bf16 plans run kernels of their own under the same condition; everything else
// runs the generic kernel.  EXAT_PIPELINED=0 forces the generic kernel (a testing aid).
int run_chain(exat_plan_s *pl, const Mode12Params &mp, bool generated, float *Yout, int accumulate, hipStream_t st, unsigned char *flag = nullptr)
{
    const bool pipelined = env_int("EXAT_PIPELINED", 1) != 0 && !(generated && mp.R > 64);
    if (generated && pl->d.in_dtype == EXAT_BF16) return run_generated_bf16(pl, mp, pipelined, Yout, st);
    return run_pieces(pl, mp, generated, pipelined, Yout, accumulate, st, flag);
}

__global__ void k_clear_flags(unsigned char *flags, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) flags[i] = 0;
}

// All operand copies of an fp32 plan in one launch: each copy has a range of blocks.  Bound by the launches: five of 4 to 5 us in a row
// for the matrices of a 250^3 tensor with 1550 rows before (set_factors and compress 274 -> 265 us).
struct PackF32 {
    const float *U, *V, *W;
    int64_t ldU, ldV, ldW, I, J, K, Ipad, Jpad;
    int P, M, N, PL, PLpad, MT, Npad;
    u32x4 *Ump, *Vmp;
    float *Upack, *Vpack, *Wpack;
    uint32_t *ranges;
    unsigned nb[5];   // blocks of Ump, Vmp, Upack, Vpack, Wpack
};
__global__ __launch_bounds__(256) void k_pack_f32(const PackF32 p)
{
    unsigned b = blockIdx.x;
    if (b < p.nb[0]) { pack_u_mp_part<3>(b, p.nb[0], p.U, p.ldU, p.PL, p.I, p.Ump, p.PLpad / 32, p.Ipad / 16, p.ranges); return; }
    b -= p.nb[0];
    if (b < p.nb[1]) { pack_v_mp_part<3>(b, p.nb[1], p.V, p.ldV, p.P, p.M, p.J, p.Vmp, p.MT, p.Jpad / 16, p.ranges); return; }
    b -= p.nb[1];
    if (b < p.nb[2]) { pack_u_part<float>(b, p.nb[2], p.U, p.ldU, p.PL, p.I, p.Upack, p.PLpad, p.Ipad); return; }
    b -= p.nb[2];
    if (b < p.nb[3]) { pack_v_part<float>(b, p.nb[3], p.V, p.ldV, p.P, p.M, p.J, p.Vpack, 32 * p.MT, p.Jpad); return; }
    b -= p.nb[3];
    pack_w_part<float>(b, p.nb[4], p.W, p.ldW, p.P, p.N, p.K, p.Wpack, p.Npad);
}

__global__ void k_clear_words(uint32_t *w, int n)
{
    if ((int)threadIdx.x < n) w[threadIdx.x] = 0;
}

// up to 32 entries of the block-pointer table per launch, carried in the kernel arguments
struct PtrChunk { const void *p[32]; int64_t idx[32]; };
__global__ void k_set_ptrs(const void **tab, PtrChunk c, int n)
{
    const int t = threadIdx.x;
    if (t < n) tab[c.idx[t]] = c.p[t];
}

// the partial-result slots of the block-streamed calls, allocated at their first use with a plan
int ensure_slots(exat_plan_s *pl, hipStream_t st)
{
    if (pl->slots) return EXAT_OK;
    int64_t ns = kSlotBudgetBytes / (pl->ysize * 4);
    if (ns < 1) ns = 1;
    if (ns > pl->nblocks) ns = pl->nblocks;
    if (ns > (1 << 20)) ns = 1 << 20;
    if (hipMalloc((void **)&pl->slots, (size_t)ns * pl->ysize * 4) != hipSuccess || hipMalloc((void **)&pl->used_dev, (size_t)ns) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(pl->slots); (void)hipFree(pl->used_dev);
        pl->slots = nullptr; pl->used_dev = nullptr;
        return EXAT_ERR_ALLOC;
    }
    pl->nslots = (int)ns;
    pl->submitted.assign((size_t)pl->nblocks, 0);
    pl->slot_used.assign((size_t)ns, 0);
    pl->nsubmitted = 0;
    hipLaunchKernelGGL(k_clear_flags, dim3(grid_for(ns)), dim3(256), 0, st, pl->used_dev, (int)ns);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}

}  // namespace

extern "C" {

int exat_plan_create(exat_plan_t *plan, const exat_desc_t *desc)
{
    if (!plan) return EXAT_ERR_NULL;
    *plan = nullptr;
    int rc = validate_desc(desc);
    if (rc != EXAT_OK) return rc;
    exat_plan_s *pl = new (std::nothrow) exat_plan_s();
    if (!pl) return EXAT_ERR_ALLOC;
    pl->d = *desc;
    pl->PL = desc->P * desc->L;
    pl->MT = (desc->M + 31) / 32;
    pl->Mpad = 32 * pl->MT;
    pl->Npad = 32 * ((desc->N + 31) / 32);
    pl->Ipad = ceil_to(desc->I, 32);
    pl->Jpad = ceil_to(desc->J, 256);
    // every kernel variant the plan may pick must find its row groups inside the padding
    int64_t plpad = 0;
    const int rts_f32[] = {1, 2, 3, 4}, rts_bf16[] = {2, 3, 4, 5};
    if (desc->in_dtype == EXAT_BF16) { for (int rt : rts_bf16) { int64_t v = ceil_to(pl->PL, 128 * rt); if (v > plpad) plpad = v; } }
    else { for (int rt : rts_f32) { int64_t v = ceil_to(pl->PL, 128 * rt); if (v > plpad) plpad = v; } }
    pl->PLpad = (int)plpad;
    const size_t es = esize(desc->in_dtype);
    const size_t ub = (size_t)pl->PLpad * pl->Ipad * es;
    const size_t vb = (size_t)desc->P * pl->Mpad * pl->Jpad * 4;
    const size_t wb = (size_t)desc->P * desc->K * pl->Npad * 4;
    const size_t qb = (size_t)desc->K * pl->PLpad * pl->Mpad * 4;
    // one allocation, cut into the plan's arrays
    const bool bf = desc->in_dtype == EXAT_BF16, split = desc->in_dtype == EXAT_F32_SPLIT;
    const size_t un = (size_t)pl->PLpad * pl->Ipad, vn = (size_t)desc->P * pl->Mpad * pl->Jpad, vf = (size_t)desc->P * pl->Jpad * 64 * 2;
    const struct { void **ptr; size_t bytes; } cut[] = {
        {(void **)&pl->ranges, MPF_WORDS * sizeof(uint32_t)}, {(void **)&pl->Asplit, (size_t)3 * pl->Ipad * 64 * 2}, {&pl->Upack, ub},
        {&pl->Ufrag, bf ? ub : 0}, {&pl->Vfrag, bf ? vf : 0}, {&pl->Vfragz, bf ? vf : 0}, {&pl->Ump, bf ? 0 : un * 6 + MP_UPAD},
        {&pl->Vmp, bf ? 0 : vn * 6}, {&pl->Usp, split ? un * 4 + MP_UPAD : 0}, {&pl->Vsp, split ? vn * 4 : 0}, {(void **)&pl->Vpack, vb},
        {(void **)&pl->Wpack, wb}, {(void **)&pl->Q, qb}};
    size_t total = 0;
    for (const auto &c : cut) total += (c.bytes + 255) & ~(size_t)255;
    if (hipMalloc(&pl->arena, total) != hipSuccess) {
        (void)hipGetLastError();
        pl->arena = nullptr;
        exat_plan_destroy(pl);
        return EXAT_ERR_ALLOC;
    }
    char *at = (char *)pl->arena;
    for (const auto &c : cut)
        if (c.bytes) { *c.ptr = at; at += (c.bytes + 255) & ~(size_t)255; }
    pl->nblocks = cdiv(desc->I, desc->dI) * cdiv(desc->J, desc->dJ) * cdiv(desc->K, desc->dK);
    pl->ysize = (int64_t)desc->P * desc->L * desc->M * desc->N;
    *plan = pl;
    return EXAT_OK;
}

int exat_plan_destroy(exat_plan_t pl)
{
    if (pl) {
        for (int b = 0; b < exat_plan_s::kRing; b++) {
            if (pl->ring[b]) (void)hipFree(pl->ring[b]);
            if (pl->ev_copied[b]) (void)hipEventDestroy(pl->ev_copied[b]);
            if (pl->ev_free[b]) (void)hipEventDestroy(pl->ev_free[b]);
        }
        if (pl->copy_stream) (void)hipStreamDestroy(pl->copy_stream);
    }
    if (!pl) return EXAT_OK;
    (void)hipFree(pl->arena); (void)hipFree(pl->slots); (void)hipFree(pl->used_dev); (void)hipFree((void *)pl->xtab);
    for (auto &tr : pl->evr)
        for (hipEvent_t e : tr) if (e) (void)hipEventDestroy(e);
    delete pl;
    return EXAT_OK;
}

int exat_set_factors(exat_plan_t pl, const float *U, int64_t ldU, const float *V, int64_t ldV,
                     const float *W, int64_t ldW, void *stream)
{
    if (!pl || !U || !V || !W) return EXAT_ERR_NULL;
    const exat_desc_t &d = pl->d;
    if (ldU < d.I || ldV < d.J || ldW < d.K) return EXAT_ERR_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    const int64_t nu = (int64_t)pl->PLpad * pl->Ipad, nv = (int64_t)d.P * pl->Mpad * pl->Jpad, nw = (int64_t)d.P * d.K * pl->Npad;
    hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(64), 0, st, pl->ranges, (int)MPF_WORDS);
    if (d.in_dtype == EXAT_BF16) {
        hipLaunchKernelGGL(k_pack_u<__bf16>, dim3(grid_for(nu)), dim3(256), 0, st, U, ldU, pl->PL, d.I, (__bf16 *)pl->Upack, pl->PLpad, pl->Ipad);
        hipLaunchKernelGGL(k_pack_u_frag<__bf16>, dim3(grid_for(nu)), dim3(256), 0, st, U, ldU, pl->PL, d.I, (__bf16 *)pl->Ufrag, pl->PLpad / 32, pl->Ipad / 16);
        hipLaunchKernelGGL(k_pack_v_frag, dim3(grid_for((int64_t)d.P * pl->Jpad * 64)), dim3(256), 0, st, V, ldV, d.P, d.M, d.J, (__bf16 *)pl->Vfrag, pl->Jpad, 0, (uint32_t *)nullptr);
        hipLaunchKernelGGL(k_pack_v_frag, dim3(grid_for((int64_t)d.P * pl->Jpad * 64)), dim3(256), 0, st, V, ldV, d.P, d.M, d.J, (__bf16 *)pl->Vfragz, pl->Jpad, 1, pl->ranges);
        hipLaunchKernelGGL(k_pack_v<__bf16>, dim3(grid_for(nv)), dim3(256), 0, st, V, ldV, d.P, d.M, d.J, pl->Vpack, pl->Mpad, pl->Jpad);
        hipLaunchKernelGGL(k_pack_w<__bf16>, dim3(grid_for(nw)), dim3(256), 0, st, W, ldW, d.P, d.N, d.K, pl->Wpack, pl->Npad);
    } else {
        const int64_t nig = pl->Ipad / 16, nj16 = pl->Jpad / 16, nu8 = (int64_t)(pl->PLpad / 32) * nig * 64, nv8 = (int64_t)d.P * nj16 * pl->MT * 64;
        const PackF32 pk = {U, V, W, ldU, ldV, ldW, d.I, d.J, d.K, pl->Ipad, pl->Jpad, d.P, d.M, d.N, pl->PL, pl->PLpad, pl->MT, pl->Npad, (u32x4 *)pl->Ump,
                            (u32x4 *)pl->Vmp, (float *)pl->Upack, pl->Vpack, pl->Wpack, pl->ranges, {grid_for(nu8), grid_for(nv8), grid_for(nu), grid_for(nv), grid_for(nw)}};
        hipLaunchKernelGGL(k_pack_f32, dim3(pk.nb[0] + pk.nb[1] + pk.nb[2] + pk.nb[3] + pk.nb[4]), dim3(256), 0, st, pk);
        if (d.in_dtype == EXAT_F32_SPLIT) {
            hipLaunchKernelGGL(k_pack_u_mp<2>, dim3(grid_for(nu8)), dim3(256), 0, st, U, ldU, pl->PL, d.I, (u32x4 *)pl->Usp, pl->PLpad / 32, nig, (uint32_t *)nullptr);
            hipLaunchKernelGGL(k_pack_v_mp<2>, dim3(grid_for(nv8)), dim3(256), 0, st, V, ldV, d.P, d.M, d.J, (u32x4 *)pl->Vsp, pl->MT, nj16, (uint32_t *)nullptr);
        }
    }
    if (hipGetLastError() != hipSuccess) return EXAT_ERR_HIP;
    pl->factors_set = true;
    return EXAT_OK;
}

int exat_compress(exat_plan_t pl, const void *X, float *Y, void *stream)
{
    if (!pl || !X || !Y) return EXAT_ERR_NULL;
    if (!pl->factors_set) return EXAT_ERR_STATE;
    const exat_desc_t &d = pl->d;
    Mode12Params mp;
    memset(&mp, 0, sizeof(mp));
    mp.X = X; mp.x_sj = d.I; mp.x_sk = d.I * d.J;
    const int e16 = 16 / (int)esize(d.in_dtype);
    mp.x_vec = (d.I % e16 == 0) && (((uintptr_t)X & 15) == 0);
    mp.i0 = 0; mp.i1 = d.I; mp.j0 = 0; mp.j1 = d.J; mp.k0 = 0; mp.k1 = d.K;
    return run_chain(pl, mp, false, Y, 0, (hipStream_t)stream);
}

int exat_compress_gen(exat_plan_t pl, const exat_gen_t *gen, const exat_box_t *box, float *Y, void *stream)
{
    if (!pl || !Y) return EXAT_ERR_NULL;
    int rc = validate_gen(gen);
    if (rc != EXAT_OK) return rc;
    if (!pl->factors_set) return EXAT_ERR_STATE;
    const exat_desc_t &d = pl->d;
    exat_box_t b = {0, d.I, 0, d.J, 0, d.K};
    if (box) b = *box;
    if (b.i0 < 0 || b.j0 < 0 || b.k0 < 0 || b.i1 > d.I || b.j1 > d.J || b.k1 > d.K || b.i0 >= b.i1 || b.j0 >= b.j1 || b.k0 >= b.k1)
        return EXAT_ERR_SHAPE;
    Mode12Params mp;
    memset(&mp, 0, sizeof(mp));
    mp.A = gen->A; mp.B = gen->B; mp.C = gen->C; mp.ldA = d.I; mp.ldB = d.J; mp.ldC = d.K; mp.R = gen->R;
    mp.a_vec = (d.I % 4 == 0) && (((uintptr_t)gen->A & 15) == 0);
    mp.skey = seed_key(gen->seed);
    mp.amp2_ln2 = amp2_ln2_of(gen->sigma);
    mp.i0 = b.i0; mp.i1 = b.i1; mp.j0 = b.j0; mp.j1 = b.j1; mp.k0 = b.k0; mp.k1 = b.k1;
    return run_chain(pl, mp, true, Y, 0, (hipStream_t)stream);
}

int exat_compress_block(exat_plan_t pl, const void *Xblk, int32_t bi, int32_t bj, int32_t bk, void *stream)
{
    if (!pl || !Xblk) return EXAT_ERR_NULL;
    if (!pl->factors_set) return EXAT_ERR_STATE;
    const exat_desc_t &d = pl->d;
    const int64_t nbi = cdiv(d.I, d.dI), nbj = cdiv(d.J, d.dJ), nbk = cdiv(d.K, d.dK);
    if (bi < 0 || bj < 0 || bk < 0 || bi >= nbi || bj >= nbj || bk >= nbk) return EXAT_ERR_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    const int rcs = ensure_slots(pl, st);
    if (rcs != EXAT_OK) return rcs;
    const int64_t blk = bi + nbi * (bj + nbj * (int64_t)bk);
    if (pl->submitted[(size_t)blk]) return EXAT_ERR_STATE;
    const int slot = (int)(blk % pl->nslots);
    Mode12Params mp;
    memset(&mp, 0, sizeof(mp));
    const int64_t di = blk_ext(d.I, d.dI, bi), dj = blk_ext(d.J, d.dJ, bj), dk = blk_ext(d.K, d.dK, bk);
    mp.X = Xblk; mp.x_sj = di; mp.x_sk = di * dj;
    mp.xo_i = (int64_t)bi * d.dI; mp.xo_j = (int64_t)bj * d.dJ; mp.xo_k = (int64_t)bk * d.dK;
    const int e16 = 16 / (int)esize(d.in_dtype);
    mp.x_vec = (di % e16 == 0) && (mp.xo_i % e16 == 0) && (((uintptr_t)Xblk & 15) == 0);
    mp.i0 = mp.xo_i; mp.i1 = mp.xo_i + di; mp.j0 = mp.xo_j; mp.j1 = mp.xo_j + dj; mp.k0 = mp.xo_k; mp.k1 = mp.xo_k + dk;
    // the mode-3 launch of the block marks its slot as holding a partial result (the merge adds marked slots only)
    int rc = run_chain(pl, mp, false, pl->slots + (int64_t)slot * pl->ysize, pl->slot_used[(size_t)slot] ? 1 : 0, st,
                       pl->slot_used[(size_t)slot] ? nullptr : pl->used_dev + slot);
    if (rc != EXAT_OK) return rc;
    pl->slot_used[(size_t)slot] = 1;
    pl->submitted[(size_t)blk] = 1;
    pl->nsubmitted++;
    return EXAT_OK;
}

int exat_compress_blocks(exat_plan_t pl, const void *const *Xblk, int32_t bj0, int32_t bj1, int32_t bk0, int32_t bk1, void *stream)
{
    if (!pl || !Xblk) return EXAT_ERR_NULL;
    if (!pl->factors_set) return EXAT_ERR_STATE;
    const exat_desc_t &d = pl->d;
    const int64_t nbi = cdiv(d.I, d.dI), nbj = cdiv(d.J, d.dJ), nbk = cdiv(d.K, d.dK);
    if (bj0 < 0 || bk0 < 0 || bj0 >= bj1 || bk0 >= bk1 || bj1 > nbj || bk1 > nbk) return EXAT_ERR_SHAPE;
    const int64_t n = nbi * (bj1 - bj0) * (int64_t)(bk1 - bk0);
    for (int64_t q = 0; q < n; q++)
        if (!Xblk[q]) return EXAT_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    const int rcs = ensure_slots(pl, st);
    if (rcs != EXAT_OK) return rcs;
    for (int64_t bk = bk0; bk < bk1; bk++)
        for (int64_t bj = bj0; bj < bj1; bj++)
            for (int64_t bi = 0; bi < nbi; bi++)
                if (pl->submitted[(size_t)(bi + nbi * (bj + nbj * bk))]) return EXAT_ERR_STATE;
    // One launch over the slab reads X through a table of block pointers: whole stages of i
    // (16 values for fp32 plans, 32 for bf16 and split-fp16 plans) and whole 128-fibre chunks inside every block,
    // 16-byte aligned blocks.  Any other slab is compressed block by block.
    const int ei = d.in_dtype == EXAT_F32 ? 16 : 32;
    bool one_launch = d.I % d.dI == 0 && d.dI % ei == 0 && d.dJ % 128 == 0 && env_int("EXAT_PIPELINED", 1) != 0 && env_int("EXAT_SLAB", 1) != 0;
    for (int64_t q = 0; q < n && one_launch; q++)
        if ((uintptr_t)Xblk[q] & 15) one_launch = false;
    if (!one_launch) {
        int64_t q = 0;
        for (int64_t bk = bk0; bk < bk1; bk++)
            for (int64_t bj = bj0; bj < bj1; bj++)
                for (int64_t bi = 0; bi < nbi; bi++, q++) {
                    const int rc = exat_compress_block(pl, Xblk[q], (int32_t)bi, (int32_t)bj, (int32_t)bk, stream);
                    if (rc != EXAT_OK) return rc;
                }
        return EXAT_OK;
    }
    if (!pl->xtab) {
        if (pl->nblocks > (1LL << 24)) return EXAT_ERR_SHAPE;
        if (hipMalloc((void **)&pl->xtab, (size_t)pl->nblocks * sizeof(void *)) != hipSuccess) { (void)hipGetLastError(); pl->xtab = nullptr; return EXAT_ERR_ALLOC; }
    }
    // the slab's entries of the table (the kernel indexes it by global block coordinates)
    {
        PtrChunk c;
        int m = 0;
        int64_t q = 0;
        for (int64_t bk = bk0; bk < bk1; bk++)
            for (int64_t bj = bj0; bj < bj1; bj++)
                for (int64_t bi = 0; bi < nbi; bi++, q++) {
                    c.p[m] = Xblk[q]; c.idx[m] = bi + nbi * (bj + nbj * bk);
                    if (++m == 32 || q == n - 1) {
                        hipLaunchKernelGGL(k_set_ptrs, dim3(1), dim3(64), 0, st, pl->xtab, c, m);
                        m = 0;
                    }
                }
        if (hipGetLastError() != hipSuccess) return EXAT_ERR_HIP;
    }
    Mode12Params mp;
    memset(&mp, 0, sizeof(mp));
    mp.xtab = pl->xtab; mp.x_dI = d.dI; mp.x_dJ = d.dJ; mp.x_dK = d.dK; mp.tab_nbi = (int)nbi; mp.tab_nbj = (int)nbj;
    mp.x_vec = 1;
    mp.i0 = 0; mp.i1 = d.I;
    mp.j0 = (int64_t)bj0 * d.dJ; mp.j1 = std::min<int64_t>(d.J, (int64_t)bj1 * d.dJ);
    mp.k0 = (int64_t)bk0 * d.dK; mp.k1 = std::min<int64_t>(d.K, (int64_t)bk1 * d.dK);
    // the slab's partial result goes to the slot of its first block
    const int64_t first = nbi * (bj0 + nbj * (int64_t)bk0);
    const int slot = (int)(first % pl->nslots);
    const int rc = run_chain(pl, mp, false, pl->slots + (int64_t)slot * pl->ysize, pl->slot_used[(size_t)slot] ? 1 : 0, st,
                             pl->slot_used[(size_t)slot] ? nullptr : pl->used_dev + slot);
    if (rc != EXAT_OK) return rc;
    pl->slot_used[(size_t)slot] = 1;
    for (int64_t bk = bk0; bk < bk1; bk++)
        for (int64_t bj = bj0; bj < bj1; bj++)
            for (int64_t bi = 0; bi < nbi; bi++) pl->submitted[(size_t)(bi + nbi * (bj + nbj * bk))] = 1;
    pl->nsubmitted += n;
    return EXAT_OK;
}

int exat_finalize(exat_plan_t pl, float *Y, void *stream)
{
    if (!pl || !Y) return EXAT_ERR_NULL;
    if (!pl->slots || pl->nsubmitted == 0) return EXAT_ERR_STATE;
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_merge, dim3(grid_for(pl->ysize)), dim3(256), 0, st, pl->slots, pl->used_dev, pl->nslots, pl->ysize, Y);
    hipLaunchKernelGGL(k_clear_flags, dim3(grid_for(pl->nslots)), dim3(256), 0, st, pl->used_dev, pl->nslots);
    if (hipGetLastError() != hipSuccess) return EXAT_ERR_HIP;
    std::fill(pl->submitted.begin(), pl->submitted.end(), 0);
    std::fill(pl->slot_used.begin(), pl->slot_used.end(), 0);
    pl->nsubmitted = 0;
    return EXAT_OK;
}

int exat_compress_host(exat_plan_t pl, const void *Xhost, float *Y, void *stream)
{
    if (!pl || !Xhost || !Y) return EXAT_ERR_NULL;
    if (!pl->factors_set) return EXAT_ERR_STATE;
    if (pl->nsubmitted != 0) return EXAT_ERR_STATE;   // a block sequence of the caller's is open
    const exat_desc_t &d = pl->d;
    const size_t es = esize(d.in_dtype);
    const size_t blk_bytes = (size_t)d.dI * d.dJ * d.dK * es;
    hipStream_t st = (hipStream_t)stream;
    if (!pl->copy_stream) {
        // default priority: streams of different priorities are never mixed in this library
        if (hipStreamCreateWithFlags(&pl->copy_stream, hipStreamNonBlocking) != hipSuccess) { pl->copy_stream = nullptr; return EXAT_ERR_HIP; }
        for (int b = 0; b < exat_plan_s::kRing; b++) {
            if (hipMalloc(&pl->ring[b], blk_bytes) != hipSuccess) { pl->ring[b] = nullptr; (void)hipGetLastError(); return EXAT_ERR_ALLOC; }
            if (hipEventCreateWithFlags(&pl->ev_copied[b], hipEventDisableTiming) != hipSuccess ||
                hipEventCreateWithFlags(&pl->ev_free[b], hipEventDisableTiming) != hipSuccess) return EXAT_ERR_HIP;
        }
    }
    for (int b = 0; b < exat_plan_s::kRing; b++)
        if (!pl->ring[b] || !pl->ev_copied[b] || !pl->ev_free[b]) return EXAT_ERR_ALLOC;   // an earlier set-up failed half way
    const int nbi = (int)cdiv(d.I, d.dI), nbj = (int)cdiv(d.J, d.dJ), nbk = (int)cdiv(d.K, d.dK);
    int64_t n = 0;
    for (int bk = 0; bk < nbk; bk++)
        for (int bj = 0; bj < nbj; bj++)
            for (int bi = 0; bi < nbi; bi++, n++) {
                const int b = (int)(n % exat_plan_s::kRing);
                // the copy into buffer b may start once the block that used it last has been consumed
                if (pl->ring_used[b] && hipStreamWaitEvent(pl->copy_stream, pl->ev_free[b], 0) != hipSuccess) return EXAT_ERR_HIP;
                hipMemcpy3DParms cp;
                memset(&cp, 0, sizeof(cp));
                cp.srcPtr = make_hipPitchedPtr(const_cast<void *>(Xhost), (size_t)d.I * es, (size_t)d.I * es, (size_t)d.J);
                cp.srcPos = make_hipPos((size_t)bi * d.dI * es, (size_t)bj * d.dJ, (size_t)bk * d.dK);
                const size_t di = (size_t)blk_ext(d.I, d.dI, bi), dj = (size_t)blk_ext(d.J, d.dJ, bj), dk = (size_t)blk_ext(d.K, d.dK, bk);
                cp.dstPtr = make_hipPitchedPtr(pl->ring[b], di * es, di * es, dj);
                cp.dstPos = make_hipPos(0, 0, 0);
                cp.extent = make_hipExtent(di * es, dj, dk);
                cp.kind = hipMemcpyHostToDevice;
                if (hipMemcpy3DAsync(&cp, pl->copy_stream) != hipSuccess) return EXAT_ERR_HIP;
                if (hipEventRecord(pl->ev_copied[b], pl->copy_stream) != hipSuccess) return EXAT_ERR_HIP;
                if (hipStreamWaitEvent(st, pl->ev_copied[b], 0) != hipSuccess) return EXAT_ERR_HIP;
                const int rc = exat_compress_block(pl, pl->ring[b], bi, bj, bk, stream);
                if (rc != EXAT_OK) {
                    // leave no half-finished block sequence behind
                    hipLaunchKernelGGL(k_clear_flags, dim3(grid_for(pl->nslots)), dim3(256), 0, st, pl->used_dev, pl->nslots);
                    std::fill(pl->submitted.begin(), pl->submitted.end(), 0);
                    std::fill(pl->slot_used.begin(), pl->slot_used.end(), 0);
                    pl->nsubmitted = 0;
                    return rc;
                }
                if (hipEventRecord(pl->ev_free[b], st) != hipSuccess) return EXAT_ERR_HIP;
                pl->ring_used[b] = true;
            }
    return exat_finalize(pl, Y, stream);
}

int exat_gen_block(const exat_desc_t *desc, const exat_gen_t *gen, int32_t bi, int32_t bj, int32_t bk, void *out, void *stream)
{
    int rc = validate_desc(desc);
    if (rc != EXAT_OK) return rc;
    rc = validate_gen(gen);
    if (rc != EXAT_OK) return rc;
    if (!out) return EXAT_ERR_NULL;
    const exat_desc_t &d = *desc;
    if (bi < 0 || bj < 0 || bk < 0 || bi >= cdiv(d.I, d.dI) || bj >= cdiv(d.J, d.dJ) || bk >= cdiv(d.K, d.dK)) return EXAT_ERR_SHAPE;
    GenParams gp;
    gp.A = gen->A; gp.B = gen->B; gp.C = gen->C; gp.ldA = d.I; gp.ldB = d.J; gp.ldC = d.K; gp.R = gen->R;
    gp.skey = seed_key(gen->seed);
    gp.amp2_ln2 = amp2_ln2_of(gen->sigma);
    gp.i0 = (int64_t)bi * d.dI; gp.i1 = gp.i0 + blk_ext(d.I, d.dI, bi);
    gp.j0 = (int64_t)bj * d.dJ; gp.j1 = gp.j0 + blk_ext(d.J, d.dJ, bj);
    gp.k0 = (int64_t)bk * d.dK; gp.k1 = gp.k0 + blk_ext(d.K, d.dK, bk);
    const int64_t nq = ((gp.i1 - 1) >> 2) - (gp.i0 >> 2) + 1;
    hipStream_t st = (hipStream_t)stream;
    const int64_t dj = gp.j1 - gp.j0, dk = gp.k1 - gp.k0, nqb = cdiv(nq, GB_Q), njb = cdiv(dj, GB_J * GB_W), nb = nqb * njb * dk;
    if (4 * nq * dj <= GB_Q * nqb * GB_J * GB_W * njb) {   // at most a quarter of k_gen_box's lanes would be busy
        int lq = 0;
        while (lq < 6 && (1 << lq) < nq) lq++;
        const int64_t nt = cdiv(cdiv(dj * dk, GB_J * (64 >> lq)) * cdiv(nq, 1 << lq), 4);
        const dim3 grid((unsigned)(nt > (1 << 22) ? (1 << 22) : nt));
        if (d.in_dtype == EXAT_BF16) hipLaunchKernelGGL(k_gen_thin<__bf16>, grid, dim3(256), 0, st, gp, lq, (__bf16 *)out);
        else hipLaunchKernelGGL(k_gen_thin<float>, grid, dim3(256), 0, st, gp, lq, (float *)out);
        return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
    }
    const dim3 grid((unsigned)(nb > (1 << 22) ? (1 << 22) : nb));
    const size_t lds = (size_t)GB_W * gp.R * GB_J * sizeof(float);   // at most 32 KiB (R <= 256)
    if (d.in_dtype == EXAT_BF16) hipLaunchKernelGGL(k_gen_box<__bf16>, grid, dim3(64 * GB_W), lds, st, gp, (__bf16 *)out);
    else hipLaunchKernelGGL(k_gen_box<float>, grid, dim3(64 * GB_W), lds, st, gp, (float *)out);
    return hipGetLastError() == hipSuccess ? EXAT_OK : EXAT_ERR_HIP;
}

int exat_plan_set_timing(exat_plan_t pl, int enable)
{
    if (!pl) return EXAT_ERR_NULL;
    if (enable && !pl->evr[0][0]) {
        for (auto &tr : pl->evr)
            for (hipEvent_t &e : tr)
                if (hipEventCreate(&e) != hipSuccess) return EXAT_ERR_HIP;
    }
    pl->timing = enable != 0;
    pl->timed_calls = 0;
    return EXAT_OK;
}

int exat_plan_timing_of(exat_plan_t pl, int32_t age, float *ms_mode12, float *ms_mode3)
{
    if (!pl || !ms_mode12 || !ms_mode3) return EXAT_ERR_NULL;
    if (!pl->timing || age < 0 || age >= exat_plan_s::kTimeRing || age >= pl->timed_calls) return EXAT_ERR_STATE;
    hipEvent_t *ev = pl->evr[(pl->timed_calls - 1 - age) % exat_plan_s::kTimeRing];
    if (hipEventSynchronize(ev[2]) != hipSuccess) return EXAT_ERR_HIP;
    if (hipEventElapsedTime(ms_mode12, ev[0], ev[1]) != hipSuccess) return EXAT_ERR_HIP;
    if (hipEventElapsedTime(ms_mode3, ev[1], ev[2]) != hipSuccess) return EXAT_ERR_HIP;
    return EXAT_OK;
}

int exat_plan_last_timing(exat_plan_t pl, float *ms_mode12, float *ms_mode3)
{
    return exat_plan_timing_of(pl, 0, ms_mode12, ms_mode3);
}

const char *exat_strerror(int status)
{
    switch (status) {
    case EXAT_OK: return "success";
    case EXAT_ERR_NULL: return "a required pointer is NULL";
    case EXAT_ERR_SHAPE: return "invalid shape, block, box or leading dimension";
    case EXAT_ERR_DTYPE: return "unknown element type";
    case EXAT_ERR_STATE: return "call not valid in the plan's current state";
    case EXAT_ERR_ALLOC: return "allocation failed";
    case EXAT_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
    }
}

}  // extern "C"
