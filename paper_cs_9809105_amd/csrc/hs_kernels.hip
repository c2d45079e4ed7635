// hs_kernels.hip -- HIP kernels for gfx950 (CDNA4) implementing the
// hyper-systolic matrix product (Sec. 5.2.2, Algorithm HYPER-SYSTOLIC) on one
// GPU, with p virtual processors realised as groups of workgroups.
//
// Kernels
//   mm_kernel        the hot loop: one workgroup holds an output tile of
//                    G stripes of one residue class mod K and is the
//                    collector of the back-shift (base C = (0,1,..,1)): it
//                    visits the partials c^{K-1}, .., c^0 (the auxiliary
//                    arrays C^l of Sec. 5.2.2) and forms each on the spot as
//                    the virtual processor that owns it: K~ steps over the
//                    travelling blocks kb = (v + jK) mod p (base
//                    A = (0,K,..,K)), fetched through registers and a
//                    double-buffered LDS ring, times the pre-shifted static
//                    block (base B = (0,-1,..,-1)), on MFMA, into one
//                    accumulator that never leaves the registers.
//   backshift_kernel the collector of the all-pairs interaction (hs_nbody):
//                    sums K partial planes in FP64, fixed order.
//   gemv_kernel      y = A x, collector form: one wave (or two, four) owns a
//                    row and sums its K partial dot products in FP64.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "hs_mfma.h"

namespace hs {

// ---------------------------------------------------------------------------
// the hyper-systolic main loop on MFMA
// ---------------------------------------------------------------------------
template <int FAM, int FORM, int BM, int BN, int CPS, int WAVES>
struct MmCfg {
    static const int NP = Pieces<FAM, FORM>::NP;
    static const int NT = 64 * WAVES;                   // threads per workgroup
    static const int CB = FAM == FAM_FP8 ? 64 : 32;     // bytes per chunk row
    static const int NPL = CB / 16;                     // 16-byte planes per chunk row
    static const int A_STAGE = NP * CPS * BM * CB;      // LDS bytes per stage
    static const int B_STAGE = NP * CPS * BN * CB;
    static const int UA = NP * CPS * BM * NPL / NT;     // 16-byte loads per thread
    static const int UB = NP * CPS * BN * NPL / NT;
    static_assert(UA * NT == NP * CPS * BM * NPL && UB * NT == NP * CPS * BN * NPL, "tile/threads");
    static const int WM = BM / 2, WN = BN / (WAVES / 2); // waves: 2 along rows, WAVES/2 along columns
    static const int MT = Mfma<FAM>::T;
    static const int TM = WM / MT, TN = WN / MT;
    static const int STAGE = A_STAGE + B_STAGE;         // one slot of the LDS ring
    static const int LPS = UA + UB;                     // DMA loads per thread per stage
    // One wave per SIMD (4 waves of 128 x 128 on the 256 x 256 tile): both
    // operands through LDS, two slots of static LDS, the stage interleaved
    // by hand (FP32, plain BF16 and FP16)
    static const bool W1 = WAVES == 4 && BM == 256;
    // B fragments straight from memory into registers (32x32 families)
    static const bool BD = FAM != FAM_FP8 && !W1;
    static const int LDS_BYTES = W1 ? 0 : 2 * (BD ? A_STAGE : STAGE);   // dynamic LDS: two slots
};

// One FP8 pipeline stage from LDS: for every chunk of the stage, the wave's
// MFMA tiles accumulate A_rows x B_cols.  sa[c][P][mi] / sb[c][P][ni] are the
// E8M0 block-scale bytes of chunk c, piece P, row / column tile (uniform
// across the wave).
template <int FAM, int FORM, int BM, int BN, int CPS, int WAVES, typename AccArr, typename SA, typename SB>
DEVI void mm_compute(AccArr &acc, const uint8_t *Ab, const uint8_t *Bb, int lane, int wm, int wn,
                const SA &sa, const SB &sb) {
    typedef MmCfg<FAM, FORM, BM, BN, CPS, WAVES> C;
#pragma unroll
    for (int c = 0; c < CPS; ++c) {
        // lane group g holds contraction elements 32g..32g+31 of the
        // 64-element chunk: planes 2g and 2g+1 of the row
        const int r32 = lane & 31, g = lane >> 5;
        i32x8 bv[C::NP][C::TN];
#pragma unroll
        for (int P = 0; P < C::NP; ++P)
#pragma unroll
            for (int ni = 0; ni < C::TN; ++ni) {
                const uint8_t *q = Bb + (P * CPS + c) * BN * C::CB + (2 * g) * BN * 16 + (wn * C::WN + ni * 32 + r32) * 16;
                const u32x4 lo = *(const u32x4 *)q, hi = *(const u32x4 *)(q + BN * 16);
                bv[P][ni] = i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            }
#pragma unroll
        for (int mi = 0; mi < C::TM; ++mi) {
            i32x8 av[C::NP];
#pragma unroll
            for (int P = 0; P < C::NP; ++P) {
                const uint8_t *q = Ab + (P * CPS + c) * BM * C::CB + (2 * g) * BM * 16 + (wm * C::WM + mi * 32 + r32) * 16;
                const u32x4 lo = *(const u32x4 *)q, hi = *(const u32x4 *)(q + BM * 16);
                av[P] = i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            }
#pragma unroll
            for (int ni = 0; ni < C::TN; ++ni) {
                if constexpr (C::NP == 2) {
                    // q1 q0', q0 q1', q0 q0': smallest first
                    acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        av[1], bv[0][ni], acc[mi][ni], 0, 0, 0, sa[c][1][mi], 0, sb[c][0][ni]);
                    acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        av[0], bv[1][ni], acc[mi][ni], 0, 0, 0, sa[c][0][mi], 0, sb[c][1][ni]);
                }
                acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                    av[0], bv[0][ni], acc[mi][ni], 0, 0, 0, sa[c][0][mi], 0, sb[c][0][ni]);
            }
        }
    }
}

// Fragment reads and MFMA tile products of the 32x32 families (FP32,
// BF16, FP16, split-BF16) for the B-direct stage below.  Lane group g
// = lane / 32 holds plane g of a chunk row (16 bytes); lane & 31 the row.
template <int FAM, int FORM, int BM, int BN, int CPS, int WAVES, typename AV>
DEVI void read_a_frags(AV &av, const uint8_t *Ab, int c, int mi, int lane, int wm) {
    typedef MmCfg<FAM, FORM, BM, BN, CPS, WAVES> C;
    const int r32 = lane & 31, g = lane >> 5;
#pragma unroll
    for (int P = 0; P < C::NP; ++P)
        av[P] = *(const u32x4 *)(Ab + (P * CPS + c) * BM * C::CB + g * BM * 16 + (wm * C::WM + mi * 32 + r32) * 16);
}

// One stage of a 32x32 family whose B fragments are already in registers
// (bq[chunk][piece][column tile]); A fragments come from the LDS slot.
template <int FAM, int FORM, int BM, int BN, int CPS, int WAVES, typename AccArr, typename BQ>
DEVI void mm_compute_bd(AccArr &acc, const uint8_t *Ab, const BQ &bq, int lane, int wm) {
    typedef MmCfg<FAM, FORM, BM, BN, CPS, WAVES> C;
#pragma unroll
    for (int c = 0; c < CPS; ++c)
#pragma unroll
        for (int mi = 0; mi < C::TM; ++mi) {
            u32x4 av[C::NP];
            read_a_frags<FAM, FORM, BM, BN, CPS, WAVES>(av, Ab, c, mi, lane, wm);
            mfma_row<FAM, FORM, C::TN>(acc[mi], av, bq[c]);
        }
}

// Global -> registers for one stage: 16-byte buffer loads of the K static
// blocks and of the travelling block.  The per-thread part of each address
// is a constant 32-bit offset; the stage part is wave-uniform (SGPR).
template <int UA, int UB>
DEVI void stage_load(u32x4 (&r)[UA + UB], __amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb,
                     const uint32_t (&a_off)[UA], const uint32_t (&b_off)[UB], uint32_t ach, uint32_t bch) {
#pragma unroll
    for (int q = 0; q < UA; ++q)
        r[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_off[q], (int)ach, 0));
#pragma unroll
    for (int q = 0; q < UB; ++q)
        r[UA + q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rb, (int)b_off[q], (int)bch, 0));
}

// Registers -> LDS slot.  The LDS image of a stage is
// [slab = (piece, chunk)][plane][row][16 bytes]: unit ui = tid + NT q lands
// at ui * 16, so consecutive lanes write consecutive 16 bytes, and the 32
// lanes of an MFMA lane group later read 512 contiguous bytes of one plane.
template <int UA, int UB, int A_STAGE, int NT>
DEVI void stage_store(const u32x4 (&r)[UA + UB], uint8_t *slot, int tid) {
#pragma unroll
    for (int q = 0; q < UA; ++q) *(u32x4 *)(slot + (tid + NT * q) * 16) = r[q];
#pragma unroll
    for (int q = 0; q < UB; ++q) *(u32x4 *)(slot + A_STAGE + (tid + NT * q) * 16) = r[UA + q];
}

template <int UA>
DEVI void stage_load_a(u32x4 (&r)[UA], __amdgpu_buffer_rsrc_t ra, const uint32_t (&a_off)[UA], uint32_t ach) {
#pragma unroll
    for (int q = 0; q < UA; ++q)
        r[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_off[q], (int)ach, 0));
}

template <int UA, int NT>
DEVI void stage_store_a(const u32x4 (&r)[UA], uint8_t *slot, int tid) {
#pragma unroll
    for (int q = 0; q < UA; ++q) *(u32x4 *)(slot + (tid + NT * q) * 16) = r[q];
}

template <int FAM, int FORM, int BM, int BN, int CPS, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES / 4, WAVES / 4)))
void mm_kernel(MainArgs a) {
    typedef MmCfg<FAM, FORM, BM, BN, CPS, WAVES> C;
    typedef typename Mfma<FAM>::Acc Acc;
    extern __shared__ __attribute__((aligned(16))) uint8_t ring[];   // C::LDS_BYTES

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;

    // workgroup -> (class c, stripe group sg, stripe sub-group msub, column
    // tile).  The tile's rows are sub-group msub of the G stripes
    // r0 + i K (i < ng), r0 = c + sg G K: all of residue class c mod K, so
    // they need the same travelling block at every step (see the step order
    // below).  Workgroups are dealt to the 8 XCDs round robin; renumber them
    // so each XCD runs a contiguous range.  Inside it, 32 consecutive
    // workgroups (one per CU of the XCD) take G_V members of one class times
    // G_T column tiles, so the XCD's L2 serves each travelling tile to G_V
    // workgroups and each static tile to G_T of them.
    // With a.nsplit > 1 (launches with fewer output tiles than CUs) the grid
    // holds nsplit copies of the tile grid; copy q walks only stages
    // [q per, (q + 1) per) of the step order and leaves its sums in plane q
    // of a.part (a fixed-order FP64 sum of the planes follows).
    int64_t bid = blockIdx.x;
    {
        const int64_t nwg = gridDim.x, xcd = bid % 8, per = nwg / 8, rem = nwg % 8;
        bid = xcd * per + (xcd < rem ? xcd : rem) + bid / 8;
    }
    const int split = (int)(bid / (gridDim.x / a.nsplit));
    bid %= gridDim.x / a.nsplit;
    const int p = a.p, K = a.K, Kt = a.Kt, MS = a.MS, G = a.G;
    int64_t ntile, msub;
    int c_class, r0, ng;
    {
        const int64_t t_lo = bid % a.grp_t;  bid /= a.grp_t;
        const int64_t u_lo = bid % a.grp_v;  bid /= a.grp_v;
        const int64_t tg = bid % a.n_tg;     bid /= a.n_tg;
        const int64_t ug = bid % a.n_ug;
        c_class = (int)(bid / a.n_ug);
        ntile = tg * a.grp_t + t_lo;
        const int64_t u = ug * a.grp_v + u_lo;        // member of the class: (sg, msub)
        const int nsg = (Kt + G - 1) / G;              // stripe groups per class
        if (ntile >= a.n_ntiles || u >= (int64_t)nsg * a.GS) return;   // grid padding
        msub = u % a.GS;
        const int sg = (int)(u / a.GS);
        r0 = c_class + sg * G * K;
        ng = Kt - sg * G < G ? Kt - sg * G : G;        // stripes of this tile
    }

    const int64_t nch = a.nch;
    const int spb = (int)(nch / CPS);                   // stages per contraction block
    // this workgroup's stages of the p spb (< 2^31, host) of the step order
    const int s_begin = split * a.split_stages;
    const int nstages = p * spb - s_begin < a.split_stages ? p * spb - s_begin : a.split_stages;

    // Each workgroup addresses its own region of the packed operands with
    // 32-bit offsets: for the static operand the G groups msub of stripes
    // r0, r0 + K, .., which sit K GS groups apart; for the travelling operand
    // its group of BN columns.  The host keeps each region below 4 GiB,
    // whatever the size of the operands.  Per-thread load descriptors are
    // offsets that do not depend on the step (group, row, half-row, piece,
    // chunk); units past the tile's ng groups re-read offset 0: their tile
    // rows are never stored.
    uint32_t a_off[C::UA];
#pragma unroll
    for (int q = 0; q < C::UA; ++q) {
        const int ui = tid + C::NT * q;              // unit: [slab][plane][row]
        const int slab = ui / (BM * C::NPL);
        const int within = ui % (BM * C::NPL);
        const int plane = within / BM, rho = within % BM;
        const int P = slab / CPS, c = slab % CPS;
        const int i = rho / MS, ir = rho % MS;
        a_off[q] = i < ng ? (uint32_t)((int64_t)i * K * a.GS * a.a_group + (int64_t)P * a.a_piece +
                                       (int64_t)c * MS * C::CB + (int64_t)(plane * MS + ir) * 16)
                          : 0u;
    }
    uint32_t b_off[C::UB];
#pragma unroll
    for (int q = 0; q < C::UB; ++q) {
        const int ui = tid + C::NT * q;
        const int slab = ui / (BN * C::NPL);
        const int within = ui % (BN * C::NPL);
        const int P = slab / CPS, c = slab % CPS;
        b_off[q] = (uint32_t)((int64_t)P * a.b_piece + (int64_t)c * BN * C::CB + (int64_t)within * 16);
    }
    const __amdgpu_buffer_rsrc_t rsA = packed_rsrc(a.A + ((int64_t)r0 * a.GS + msub) * a.a_group, (uint32_t)a.a_span);
    const __amdgpu_buffer_rsrc_t rsB = packed_rsrc(a.B + ntile * a.b_group, (uint32_t)a.b_group);

    // The step order.  The collector visits the partials l = K-1, .., 0
    // (t = K-1-l).  Partial l of stripe s is virtual processor v = s + l's
    // work: its steps visit the travelling blocks kb = (v + jK) mod p,
    // j = 0..K~-1 (base A = (0, K, .., K)), a cycle of stride K through the
    // residue class (c + l) mod K, which is the same for every stripe of the
    // tile; the cycle is entered at its smallest block (c + l) mod K, so all
    // workgroups of class c hold the same block at the same time.  cs counts
    // the stages inside a block.  Past the last stage the position stays put,
    // so the surplus fetches re-read the last stage (never used).
    struct Pos { int kb, cs, j, t, n; };
    auto advance = [&](Pos &q) {
        if (++q.n >= nstages) return;
        if (++q.cs < spb) return;
        q.cs = 0;
        if (++q.j < Kt) {                               // next step: shift by K along the ring
            q.kb += K;
            return;
        }
        q.j = 0;                                        // next partial of the collector
        ++q.t;
        q.kb = (c_class + K - 1 - q.t) % K;
    };
    // position of stage s_begin: partial t, step j, stage cs of the block
    Pos start;
    {
        const int per_t = Kt * spb;
        start.t = s_begin / per_t;
        start.j = (s_begin % per_t) / spb;
        start.cs = s_begin % spb;
        start.kb = (c_class + K - 1 - start.t) % K + start.j * K;
        start.n = 0;
    }
    const uint32_t a_stage = (uint32_t)(MS * C::CB), b_stage = (uint32_t)(BN * C::CB);
    // first chunk of the stage at q, then advance q by one stage
    auto next_chunk = [&](Pos &q) -> uint32_t {
        // wave-uniform by construction; readfirstlane keeps the stage
        // offsets in SGPRs whatever the compiler's uniformity analysis finds
        const uint32_t ch = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)q.kb * (uint32_t)nch + (uint32_t)(q.cs * CPS)));
        advance(q);
        return ch;
    };
    Pos pa = start;
    auto fetch_offsets = [&](uint32_t &ach, uint32_t &bch) {
        const uint32_t ch = next_chunk(pa);
        ach = ch * a_stage;
        bch = ch * b_stage;
    };

    // FP8: block-scale bytes of the stage being multiplied.  Every 32-row
    // (32-column) MFMA tile and every 64-deep chunk lies inside one 128 x 128
    // scale tile (the host checks the alignment), so each scale is uniform
    // across the wave: 127 - e for q0, 127 - e - e1 for q1.
    int sa[CPS][C::NP][C::TM], sb[CPS][C::NP][C::TN];
    Pos pc = start;                                     // stage being multiplied
    int tra[C::TM], trb[C::TN];
    if constexpr (FAM == FAM_FP8) {
#pragma unroll
        for (int mi = 0; mi < C::TM; ++mi) {
            const int rho0 = wm * C::WM + mi * 32;
            const int i = rho0 / MS, i0 = rho0 % MS;
            // rows of the groups past ng are never stored: any valid scale
            int64_t row0 = (int64_t)(r0 + (i < ng ? i : 0) * K) * a.S_r + msub * MS + i0;
            row0 = row0 < a.M ? row0 : a.M - 1;
            tra[mi] = (int)(row0 / FP8_TILE);
        }
#pragma unroll
        for (int ni = 0; ni < C::TN; ++ni) {
            int64_t col0 = ntile * BN + wn * C::WN + ni * 32;
            col0 = col0 < a.N ? col0 : a.N - 1;
            trb[ni] = (int)(col0 / FP8_TILE);
        }
    }
    auto stage_scales = [&]() {
        if constexpr (FAM == FAM_FP8) {
            typedef const __attribute__((address_space(4))) int32_t cint;
            cint *ea = (cint *)a.a_exps;
            cint *eb = (cint *)a.b_exps;
#pragma unroll
            for (int c = 0; c < CPS; ++c) {
                int64_t kk = (int64_t)pc.kb * a.S_k + (int64_t)(pc.cs * CPS + c) * 64;
                kk = kk < a.Kd ? kk : a.Kd - 1;         // padding chunks hold zeros
                const int tc = __builtin_amdgcn_readfirstlane((int)(kk / FP8_TILE));
#pragma unroll
                for (int mi = 0; mi < C::TM; ++mi) {
                    const int t = __builtin_amdgcn_readfirstlane((int)((tra[mi] * a.a_tiles_k + tc) * 2));
                    const int e = ea[t], e1 = ea[t + 1];
                    sa[c][0][mi] = 127 - e;
                    if constexpr (C::NP == 2) sa[c][1][mi] = 127 - e - e1;
                }
#pragma unroll
                for (int ni = 0; ni < C::TN; ++ni) {
                    const int t = __builtin_amdgcn_readfirstlane((int)((trb[ni] * a.b_tiles_k + tc) * 2));
                    const int e = eb[t], e1 = eb[t + 1];
                    sb[c][0][ni] = 127 - e;
                    if constexpr (C::NP == 2) sb[c][1][ni] = 127 - e - e1;
                }
            }
            advance(pc);
        }
    };

    Acc acc[C::TM][C::TN];
#pragma unroll
    for (int mi = 0; mi < C::TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < C::TN; ++ni) acc[mi][ni] = Acc{};

    uint32_t ach, bch;
    if constexpr (C::BD) {
        // The travelling operand skips LDS: each wave loads its own MFMA
        // fragments of B (the packed layout already is the fragment layout:
        // 32 lanes read 512 contiguous bytes of one plane) one stage ahead,
        // into one of two register sets.  Only the static blocks go
        // through LDS (two slots, loaded two stages ahead, written one
        // stage ahead, one barrier per stage), which halves the LDS writes
        // and cuts the LDS reads by a third.
        const int r32 = lane & 31, g = lane >> 5;
        const uint32_t b_lane = (uint32_t)((int64_t)g * BN * 16 + (int64_t)(wn * C::WN + r32) * 16);
        const uint32_t b_piece = (uint32_t)a.b_piece;
        typedef u32x4 BQ[CPS][C::NP][C::TN];
        auto load_b = [&](BQ &bq, uint32_t ch) {
            const uint32_t bst = ch * b_stage;
#pragma unroll
            for (int c = 0; c < CPS; ++c)
#pragma unroll
                for (int P = 0; P < C::NP; ++P)
#pragma unroll
                    for (int ni = 0; ni < C::TN; ++ni)
                        bq[c][P][ni] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                            rsB, (int)(b_lane + ni * 32 * 16), (int)(bst + P * b_piece + c * BN * C::CB), 0));
        };
        u32x4 r0s[C::UA], r1s[C::UA];
        BQ q0, q1;
        Pos pb = start;
        fetch_offsets(ach, bch);
        stage_load_a<C::UA>(r0s, rsA, a_off, ach);
        fetch_offsets(ach, bch);
        stage_load_a<C::UA>(r1s, rsA, a_off, ach);
        load_b(q0, next_chunk(pb));
        stage_store_a<C::UA, C::NT>(r0s, ring, tid);
        __syncthreads();
#define HS_PIPE_STEP(RLOAD, RSTORE, QUSE, QLOAD)                                               \
    {                                                                                          \
        const int slot = (int)(s & 1);                                                         \
        fetch_offsets(ach, bch);                                                               \
        stage_load_a<C::UA>(RLOAD, rsA, a_off, ach);                                           \
        load_b(QLOAD, next_chunk(pb));                                                         \
        stage_store_a<C::UA, C::NT>(RSTORE, ring + (slot ^ 1) * C::A_STAGE, tid);              \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        mm_compute_bd<FAM, FORM, BM, BN, CPS, WAVES>(acc, ring + slot * C::A_STAGE, QUSE, lane, wm); \
        __syncthreads();                                                                       \
        if (++s >= nstages) break;                                                             \
    }
        for (int s = 0; s < nstages;) {
            HS_PIPE_STEP(r0s, r1s, q0, q1)
            HS_PIPE_STEP(r1s, r0s, q1, q0)
        }
#undef HS_PIPE_STEP
    } else if constexpr (C::W1) {
        // One wave per SIMD, so nothing else on the SIMD hides a wait: the
        // stage is laid out by hand.  Each LDS slot is a static array of
        // its own, which lets the compiler place the reads of one slot
        // between the writes to the other.  The one barrier per stage sits
        // before its last chunk: until then the wave multiplies chunk c
        // (fragments already in registers) while it reads chunk c + 1,
        // issues the loads of stage s + 2 and writes stage s + 1 (loaded a
        // stage earlier) into the other slot; after it the wave multiplies
        // the last chunk while it reads chunk 0 of stage s + 1 from the other
        // slot.  A slot is rewritten only after the barrier that follows its
        // last read.
        static_assert(CPS >= 2, "at least two chunks per stage");
        __shared__ __attribute__((aligned(16))) uint8_t slot0[C::STAGE];
        __shared__ __attribute__((aligned(16))) uint8_t slot1[C::STAGE];
        u32x4 r0s[C::LPS], r1s[C::LPS];
        const int r32 = lane & 31, g = lane >> 5;
        const int a_rd = g * BM * 16 + (wm * C::WM + r32) * 16;
        const int b_rd = C::A_STAGE + g * BN * 16 + (wn * C::WN + r32) * 16;
        u32x4 fa0[C::TM], fb0[C::TN], fa1[C::TM], fb1[C::TN];
        auto read_chunk = [&](const uint8_t *sl, int c, u32x4 (&fa)[C::TM], u32x4 (&fb)[C::TN]) {
#pragma unroll
            for (int ni = 0; ni < C::TN; ++ni) fb[ni] = *(const u32x4 *)(sl + b_rd + c * BN * C::CB + ni * 32 * 16);
#pragma unroll
            for (int mi = 0; mi < C::TM; ++mi) fa[mi] = *(const u32x4 *)(sl + a_rd + c * BM * C::CB + mi * 32 * 16);
        };
        auto mfma_chunk = [&](const u32x4 (&fa)[C::TM], const u32x4 (&fb)[C::TN]) {
#pragma unroll
            for (int mi = 0; mi < C::TM; ++mi) {
                u32x4 av[1] = {fa[mi]};
                u32x4 bv[1][C::TN];
#pragma unroll
                for (int ni = 0; ni < C::TN; ++ni) bv[0][ni] = fb[ni];
                mfma_row<FAM, FORM, C::TN>(acc[mi], av, bv);
            }
        };
        fetch_offsets(ach, bch);
        stage_load<C::UA, C::UB>(r0s, rsA, rsB, a_off, b_off, ach, bch);
        fetch_offsets(ach, bch);
        stage_load<C::UA, C::UB>(r1s, rsA, rsB, a_off, b_off, ach, bch);
        stage_store<C::UA, C::UB, C::A_STAGE, C::NT>(r0s, slot0, tid);
        __syncthreads();
        read_chunk(slot0, 0, fa0, fb0);
        // sched_group_barrier masks: 0x008 MFMA, 0x020 global load, 0x100
        // LDS read, 0x200 LDS write.  A chunk has W1_RD fragment reads and
        // W1_PER MFMAs per read (2 for BF16/FP16, 8 for FP32's 32x32x2).
        // Before the barrier, W1_SLOTS times: MFMA, read, (write), W1_PER - 1
        // MFMAs, (load), the LPS loads and writes on the first slots; after
        // it, W1_RD times: MFMA, read, W1_PER - 1 MFMAs.
        constexpr int W1_RD = C::TM + C::TN;
        constexpr int W1_PER = C::TM * C::TN * (FAM == FAM_F32 ? 4 : 1) / W1_RD;
        constexpr int W1_SLOTS = (CPS - 1) * W1_RD;          // reads before the barrier
        static_assert(C::LPS <= W1_SLOTS && W1_PER >= 2, "interleave pattern");
        // Before the barrier: chunks 0 .. CPS-2 (each while reading the next
        // chunk of this slot), the loads of stage s + 2 and the LDS writes of
        // stage s + 1 into the other slot.  After it: the last chunk, while
        // reading chunk 0 of stage s + 1 from the other slot.  Every read of
        // this slot precedes the barrier, so the next stage may rewrite it.
        auto first_part = [&](const uint8_t *X, uint8_t *Y, u32x4 (&RLOAD)[C::LPS], const u32x4 (&RSTORE)[C::LPS]) {
#pragma unroll
            for (int c = 0; c + 1 < CPS; ++c) {
                if (c % 2 == 0) { mfma_chunk(fa0, fb0); read_chunk(X, c + 1, fa1, fb1); }
                else { mfma_chunk(fa1, fb1); read_chunk(X, c + 1, fa0, fb0); }
            }
            stage_load<C::UA, C::UB>(RLOAD, rsA, rsB, a_off, b_off, ach, bch);
            stage_store<C::UA, C::UB, C::A_STAGE, C::NT>(RSTORE, Y, tid);
#pragma unroll
            for (int i = 0; i < W1_SLOTS; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                if (i < C::LPS) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, W1_PER - 1, 0);
                if (i < C::LPS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        };
        auto last_part = [&](const uint8_t *Y) {
            if constexpr ((CPS - 1) % 2 == 0) { mfma_chunk(fa0, fb0); read_chunk(Y, 0, fa0, fb0); }
            else { mfma_chunk(fa1, fb1); read_chunk(Y, 0, fa0, fb0); }
#pragma unroll
            for (int i = 0; i < W1_RD; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, W1_PER - 1, 0);
            }
        };
#define HS_W1_STEP(X, Y, RLOAD, RSTORE)                                                        \
    {                                                                                          \
        fetch_offsets(ach, bch);                                                               \
        first_part(X, Y, RLOAD, RSTORE);                                                       \
        __syncthreads();                                                                       \
        last_part(Y);                                                                          \
        if (++s >= nstages) break;                                                             \
    }
        for (int s = 0; s < nstages;) {
            HS_W1_STEP(slot0, slot1, r0s, r1s)
            HS_W1_STEP(slot1, slot0, r1s, r0s)
        }
#undef HS_W1_STEP
    } else {
        // Both operands through LDS, two slots: the global loads for stage
        // s + 2 are issued at the top of stage s into one of two register
        // sets; the LDS image of stage s + 1 is written into the other slot
        // at the top of stage s, and one barrier closes each stage.
        u32x4 r0s[C::LPS], r1s[C::LPS];
        fetch_offsets(ach, bch);
        stage_load<C::UA, C::UB>(r0s, rsA, rsB, a_off, b_off, ach, bch);
        fetch_offsets(ach, bch);
        stage_load<C::UA, C::UB>(r1s, rsA, rsB, a_off, b_off, ach, bch);
        stage_store<C::UA, C::UB, C::A_STAGE, C::NT>(r0s, ring, tid);
        __syncthreads();
#define HS_PIPE_STEP(RLOAD, RSTORE)                                                            \
    {                                                                                          \
        const int slot = (int)(s & 1);                                                         \
        fetch_offsets(ach, bch);                                                               \
        stage_load<C::UA, C::UB>(RLOAD, rsA, rsB, a_off, b_off, ach, bch);                     \
        stage_store<C::UA, C::UB, C::A_STAGE, C::NT>(RSTORE, ring + (slot ^ 1) * C::STAGE, tid); \
        stage_scales();                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        mm_compute<FAM, FORM, BM, BN, CPS, WAVES>(acc, ring + slot * C::STAGE,                 \
                                           ring + slot * C::STAGE + C::A_STAGE, lane, wm, wn,  \
                                           sa, sb);                                            \
        __syncthreads();                                                                       \
        if (++s >= nstages) break;                                                             \
    }
        for (int s = 0; s < nstages;) {
            HS_PIPE_STEP(r0s, r1s)
            HS_PIPE_STEP(r1s, r0s)
        }
#undef HS_PIPE_STEP
    }

    // epilogue: the collector has absorbed every partial; tile row rho is
    // row msub MS + (rho mod MS) of stripe r0 + (rho / MS) K.  One tile row
    // at a time (row index computed once, then its columns).
    const int64_t S_r = a.S_r;
    constexpr int NE = (int)(sizeof(Acc) / sizeof(acc[0][0][0]));
    // two-piece FP16: the tile holds C' = sum a' b' of the scaled operands;
    // C = C' 2^-(e_row + e_col) (exact unless the result is subnormal)
    constexpr bool ROWSCALE = FAM == FAM_F16 && FORM == 2;
    int ecol[C::TN];
#pragma unroll
    for (int ni = 0; ni < C::TN; ++ni) {
        ecol[ni] = 0;
        if constexpr (ROWSCALE) {
            const int64_t col = ntile * BN + wn * C::WN + ni * C::MT + (lane & 31);
            if (col < a.N) ecol[ni] = row_scale_exp(((const uint32_t *)a.b_exps)[col]);
        }
    }
#pragma unroll
    for (int mi = 0; mi < C::TM; ++mi) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int rho = wm * C::WM + mi * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
            const int i = rho / MS, ir = rho % MS;
            const int64_t within = msub * MS + ir;
            const int64_t row = (int64_t)(r0 + i * K) * S_r + within;
            const bool rok = i < ng && within < S_r && row < a.M;
            const int64_t cbase = ntile * BN + wn * C::WN + (lane & 31);
            int erow = 0;
            if constexpr (ROWSCALE) erow = rok ? row_scale_exp(((const uint32_t *)a.a_exps)[row]) : 0;
            // the element's destination: C, or plane `split` of a.part (rows of N)
            const bool to_part = a.nsplit > 1;
            const int64_t obase = to_part ? ((int64_t)split * a.M + row) * a.N + cbase : row * a.ldo + cbase;
            float *dst = (float *)(to_part ? a.part : a.out);
#pragma unroll
            for (int ni = 0; ni < C::TN; ++ni) {
                const bool ok = rok && cbase + ni * C::MT < a.N;
                if (ok) {
                    if constexpr (ROWSCALE) dst[obase + ni * C::MT] = ldexpf(acc[mi][ni][e], -(erow + ecol[ni]));
                    else dst[obase + ni * C::MT] = acc[mi][ni][e];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// back-shift and accumulation (fixed order, FP64)
// ---------------------------------------------------------------------------
// Each thread sums 4 consecutive columns of one row over the K partial
// planes, c^{K-1} first: S = c^l + S for l = K-2 .. 0 (back-shift order).
// VEC: N % 4 == 0 (16-byte partial loads); VST: 16-byte stores into C legal.
template <typename PT, typename OT, int VEC, int VST>
__global__ __launch_bounds__(256) void backshift_kernel(const PT *W, int64_t plane, int K,
                                                        int64_t M, int64_t N, OT *Cout, int64_t ldc) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t n4 = (N + 3) / 4;
    if (idx >= M * n4) return;
    const int64_t row = idx / n4, c0 = (idx % n4) * 4;
    const int cnt = (int)((N - c0) < 4 ? (N - c0) : 4);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int l = K - 1; l >= 0; --l) {
        const PT *wl = W + (int64_t)l * plane + row * N + c0;
        PT x[4];
        if constexpr (VEC && sizeof(PT) == 4) {
            const float4 v = *(const float4 *)wl;
            x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
        } else if constexpr (VEC) {
            const double2 v0 = *(const double2 *)wl, v1 = *(const double2 *)(wl + 2);
            x[0] = v0.x; x[1] = v0.y; x[2] = v1.x; x[3] = v1.y;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = e < cnt ? wl[e] : (PT)0;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = (l == K - 1) ? (double)x[e] : (double)x[e] + s[e];
    }
    OT *c = Cout + row * ldc + c0;
    if constexpr (VST && sizeof(OT) == 4) {
        *(float4 *)c = make_float4((float)s[0], (float)s[1], (float)s[2], (float)s[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < cnt) c[e] = (OT)s[e];
    }
}

template <typename OT>
__global__ __launch_bounds__(256) void fill_zero_kernel(OT *Cout, int64_t M, int64_t N, int64_t ldc) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= M * N) return;
    Cout[(idx / N) * ldc + idx % N] = (OT)0;
}

// ---------------------------------------------------------------------------
// matrix-vector product
// ---------------------------------------------------------------------------
// y = A x.  Every block product of the schedule belongs to one row, and the
// collector adds all K partials of a row in the wave (or the W = 2, 4 waves) that
// owns it, so the blocks are visited in storage order: one contiguous sweep over
// the row, VE elements per lane and load (16 bytes, at any element alignment), U
// loads in flight while the U before them are multiplied.  Each group's FP32 sum
// (16 products) goes into an FP64 sum, and the lanes' FP64 sums are added at the
// end.  Bound by reading A once: FP32 8192 x 8192 42.5 us (6.3 TB/s), 3001 x 2999
// (rows at any alignment) 7.0, 500 x 500 3.9.  Walking the blocks partial by
// partial in the order of base A, with a cross-lane sum after each, took 46.0, 11.0
// and (p = 64, K = 8) 45 us; the same walk as one pipelined sequence 42.5, 10.7
// and 4.4, but 5000 x 10000 44.5 against 35.5 here, for its index arithmetic.
// CX: complex64 (VE complex elements per load).  NT: A is read past the caches
// (it is larger than they are, see launch_gemv_t).
template <typename T, int CX, int NT>
__global__ __launch_bounds__(256) void gemv_kernel(GemvArgs a) {
    constexpr int VE = 16 / (int)(sizeof(T) * (1 + CX)), U = 4, NT4 = VE * (1 + CX);
    typedef T V __attribute__((ext_vector_type(VE * (1 + CX))));
    typedef V VU __attribute__((aligned(sizeof(T) * (1 + CX))));
    __shared__ double red[4][2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int W = a.waves, part = wave & (W - 1);   // W a power of two: 4 / W rows per workgroup
    const int64_t row = ((int64_t)blockIdx.x * 4 + wave) / W;
    const int64_t n = row < a.m ? a.n : 0;
    const int start = (part * 64 + lane) * VE, stride = 64 * W * VE;
    const T *Ar = (const T *)a.A + row * a.lda * (1 + CX);
    const T *x = (const T *)a.x;
    double Sr = 0.0, Si = 0.0;
    auto multiply = [&](const V (&av)[U], const V (&xv)[U]) {
        T re = 0, im = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (CX) {
#pragma unroll
                for (int c = 0; c < VE; ++c) {
                    const T ar = av[u][2 * c], ai = av[u][2 * c + 1], xr = xv[u][2 * c], xi = xv[u][2 * c + 1];
                    re = __builtin_fmaf(ar, xr, re);
                    re = __builtin_fmaf(-ai, xi, re);
                    im = __builtin_fmaf(ar, xi, im);
                    im = __builtin_fmaf(ai, xr, im);
                }
            } else {
#pragma unroll
                for (int c = 0; c < VE; ++c) re += av[u][c] * xv[u][c];
            }
        }
        Sr += (double)re;
        if constexpr (CX) Si += (double)im;
    };
    // whole groups: every lane's U loads lie inside the row
    const int groups = (int)(n / ((int64_t)stride * U));
    auto load = [&](V (&av)[U], V (&xv)[U], int g) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = ((int64_t)(g * U + u) * stride + start) * (1 + CX);
            if constexpr (NT) av[u] = __builtin_nontemporal_load((const VU *)(Ar + at));
            else av[u] = *(const VU *)(Ar + at);
            xv[u] = *(const VU *)(x + at);
        }
    };
    V a0[U], x0[U], a1[U], x1[U];
    if (groups > 0) {
        load(a0, x0, 0);
        for (int g = 1;; g += 2) {
            if (g >= groups) {
                multiply(a0, x0);
                break;
            }
            load(a1, x1, g);
            multiply(a0, x0);
            if (g + 1 >= groups) {
                multiply(a1, x1);
                break;
            }
            load(a0, x0, g + 1);
            multiply(a1, x1);
        }
    }
    // the rest of the row: a load may end inside it
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t col = (int64_t)(groups * U + u) * stride + start;
        a0[u] = V{};
        x0[u] = V{};
        if (col + VE <= n) {
            a0[u] = *(const VU *)(Ar + col * (1 + CX));
            x0[u] = *(const VU *)(x + col * (1 + CX));
        } else {
#pragma unroll
            for (int c = 0; c < NT4 - (1 + CX); ++c)
                if (col + c / (1 + CX) < n) {
                    a0[u][c] = Ar[col * (1 + CX) + c];
                    x0[u][c] = x[col * (1 + CX) + c];
                }
        }
    }
    multiply(a0, x0);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        Sr += __shfl_xor(Sr, m, 64);
        if constexpr (CX) Si += __shfl_xor(Si, m, 64);
    }
    if (W > 1) {                               // the row's waves
        if (lane == 0) {
            red[wave][0] = Sr;
            red[wave][1] = Si;
        }
        __syncthreads();
        if (part != 0) return;
        for (int w = 1; w < W; ++w) {
            Sr += red[wave + w][0];
            Si += red[wave + w][1];
        }
    }
    if (lane != 0 || row >= a.m) return;
    T *y = (T *)a.y + row * (1 + CX);
    y[0] = (T)Sr;
    if constexpr (CX) y[1] = (T)Si;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned nblocks(int64_t work) { return (unsigned)((work + 255) / 256); }

// Events of the next timed launch (hs_profile_begin / hs_profile_end): the
// dispatch itself records them (hipExtLaunchKernel), so they bracket the
// kernel's execution alone, without the gaps that separate event records
// add around a short kernel.
static hipEvent_t g_timed_start = nullptr, g_timed_stop = nullptr;
static bool g_timed_used = false;
void set_timed_launch(hipEvent_t start, hipEvent_t stop) {
    g_timed_start = start;
    g_timed_stop = stop;
    g_timed_used = false;
}
bool take_timed_launch(hipEvent_t *start, hipEvent_t *stop) {
    if (!g_timed_start) return false;
    *start = g_timed_start;
    *stop = g_timed_stop;
    g_timed_start = g_timed_stop = nullptr;
    g_timed_used = true;
    return true;
}
// true if the events set last were taken by a launch; clears them
bool timed_launch_done() {
    const bool used = g_timed_used;
    g_timed_start = g_timed_stop = nullptr;
    g_timed_used = false;
    return used;
}
#define HS_LAUNCH_TIMED(KERNEL, GRID, BLOCK, SHM, ST, ...)                                    \
    do {                                                                                     \
        hipEvent_t ts_, te_;                                                                 \
        if (take_timed_launch(&ts_, &te_))                                                   \
            hipExtLaunchKernelGGL(KERNEL, GRID, BLOCK, SHM, ST, ts_, te_, 0, __VA_ARGS__);   \
        else                                                                                 \
            hipLaunchKernelGGL(KERNEL, GRID, BLOCK, SHM, ST, __VA_ARGS__);                   \
    } while (0)

template <int FAM, int FORM, int BM, int BN, int CPS, int WAVES>
static hipError_t launch_mm_t(const MainArgs &a, hipStream_t st) {
    typedef MmCfg<FAM, FORM, BM, BN, CPS, WAVES> C;
    // the dynamic LDS limit is a per-device function attribute: set it once
    // on each device the kernel runs on (setting it twice is harmless)
    static bool attr_set[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    if (dev < 0 || dev >= 64 || !attr_set[dev]) {
        hipError_t e = hipFuncSetAttribute((const void *)mm_kernel<FAM, FORM, BM, BN, CPS, WAVES>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) attr_set[dev] = true;
    }
    const int64_t nwg = (int64_t)a.K * a.n_ug * a.n_tg * a.grp_v * a.grp_t * a.nsplit;
    HS_LAUNCH_TIMED((mm_kernel<FAM, FORM, BM, BN, CPS, WAVES>), dim3((unsigned)nwg), dim3(C::NT), C::LDS_BYTES, st, a);
    return hipGetLastError();
}

// Tile shapes per family: rows of the workgroup tile (K groups of MS rows),
// columns, and chunks per pipeline stage.  FP64 runs on the wave kernel
// alone; its entries are the geometry in which a call's limits are stated.
int mm_tile_rows(int fam) { return fam == FAM_F64 ? 64 : 256; }
int mm_tile_cols(int fam) { return fam == FAM_F64 ? 64 : 256; }
int mm_chunks_per_stage(int fam, int form) {
    if (fam == FAM_F64) return 4;
    if (fam == FAM_FP8) return form == 1 ? 1 : 2;
    if (fam == FAM_F32) return 2;
    // split forms one 16-deep chunk per stage (split-BF16: 48 MFMAs per wave;
    // two-piece FP16: 24, measured 2.45 ms against 2.60 with two chunks at
    // n = 8192), BF16 and FP16 four (64 per wave; 0.915 against 0.934 ms for
    // BF16 with two at n = 8192)
    return form == 1 || form == 2 ? 1 : 4;
}

// 8 waves (2 per SIMD) for the split forms' and FP8's 256 x 256 tiles, 4
// (one per SIMD) for FP32, plain BF16 and FP16 (measured at n = 8192 on
// one box against 8 waves: FP32 7.33 against 7.61 ms, BF16 0.930 against
// 0.970 ms, FP16 0.970 against 1.008 ms, with two chunks per stage).
hipError_t launch_mm(int fam, int form, const MainArgs &a, hipStream_t st) {
    if (fam == FAM_F32) return launch_mm_t<FAM_F32, 0, 256, 256, 2, 4>(a, st);
    if (fam == FAM_F16 && form == 0) return launch_mm_t<FAM_F16, 0, 256, 256, 4, 4>(a, st);
    if (fam == FAM_F16 && form == 2) return launch_mm_t<FAM_F16, 2, 256, 256, 1, 8>(a, st);
    if (fam == FAM_BF16 && form == 0) return launch_mm_t<FAM_BF16, 0, 256, 256, 4, 4>(a, st);
    if (fam == FAM_BF16 && form == 1) return launch_mm_t<FAM_BF16, 1, 256, 256, 1, 8>(a, st);
    if (fam == FAM_FP8 && form == 0) return launch_mm_t<FAM_FP8, 0, 256, 256, 2, 8>(a, st);
    if (fam == FAM_FP8 && form == 1) return launch_mm_t<FAM_FP8, 1, 256, 256, 1, 8>(a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_backshift(int f64, const void *W, int64_t plane, int K, int64_t M, int64_t N,
                            void *Cout, int64_t ldc, hipStream_t st) {
    const int64_t work = M * ((N + 3) / 4);
    if (work == 0) return hipSuccess;
    const bool vec = N % 4 == 0;
    const bool vst = vec && ldc % 4 == 0 && ((uintptr_t)Cout % 16) == 0;
    const dim3 grid(nblocks(work)), block(256);
    if (f64) {
        if (vec) hipLaunchKernelGGL((backshift_kernel<double, double, 1, 0>), grid, block, 0, st,
                                    (const double *)W, plane, K, M, N, (double *)Cout, ldc);
        else hipLaunchKernelGGL((backshift_kernel<double, double, 0, 0>), grid, block, 0, st,
                                (const double *)W, plane, K, M, N, (double *)Cout, ldc);
    } else {
        if (vst) hipLaunchKernelGGL((backshift_kernel<float, float, 1, 1>), grid, block, 0, st,
                                    (const float *)W, plane, K, M, N, (float *)Cout, ldc);
        else if (vec) hipLaunchKernelGGL((backshift_kernel<float, float, 1, 0>), grid, block, 0, st,
                                         (const float *)W, plane, K, M, N, (float *)Cout, ldc);
        else hipLaunchKernelGGL((backshift_kernel<float, float, 0, 0>), grid, block, 0, st,
                                (const float *)W, plane, K, M, N, (float *)Cout, ldc);
    }
    return hipGetLastError();
}

hipError_t launch_fill_zero(int f64, void *Cout, int64_t M, int64_t N, int64_t ldc, hipStream_t st) {
    if (M * N == 0) return hipSuccess;
    if (f64)
        hipLaunchKernelGGL((fill_zero_kernel<double>), dim3(nblocks(M * N)), dim3(256), 0, st, (double *)Cout, M, N, ldc);
    else
        hipLaunchKernelGGL((fill_zero_kernel<float>), dim3(nblocks(M * N)), dim3(256), 0, st, (float *)Cout, M, N, ldc);
    return hipGetLastError();
}

template <typename T, int CX>
static hipError_t launch_gemv_t(const GemvArgs &a, hipStream_t st) {
    const dim3 grid((unsigned)((a.m * a.waves + 3) / 4));
    // A of 256 MiB or more does not stay in the memory-side cache between
    // calls; reading it past the caches is then faster (FP32 8192 x 8192, the
    // kernel before this one: 44.9 us against 48.2; 8192 x 2048, which stays in
    // that cache: 13.8 against 12.6)
    if (a.m * a.n * (int64_t)(sizeof(T) * (1 + CX)) >= (int64_t)256 << 20)
        HS_LAUNCH_TIMED((gemv_kernel<T, CX, 1>), grid, dim3(256), 0, st, a);
    else
        HS_LAUNCH_TIMED((gemv_kernel<T, CX, 0>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_gemv(int f64, const GemvArgs &a, hipStream_t st) {
    if (a.m == 0) return hipSuccess;
    if (a.cplx) return launch_gemv_t<float, 1>(a, st);
    return f64 ? launch_gemv_t<double, 0>(a, st) : launch_gemv_t<float, 0>(a, st);
}

}  // namespace hs
