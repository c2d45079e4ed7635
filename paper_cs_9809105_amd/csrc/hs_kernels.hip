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
//                    A = (0,K,..,K)), loaded straight into a ring of LDS
//                    stages, times the pre-shifted static
//                    block (base B = (0,-1,..,-1)), on MFMA, into one
//                    accumulator that never leaves the registers.
//   backshift_kernel the collector of the all-pairs interaction (hs_nbody):
//                    sums K partial planes in FP64, fixed order.
//   gemv_kernel      y = A x: one wave (or two, four, or a quarter of one)
//                    sweeps a row once, its FP32 sums of 16 products added
//                    in FP64.
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
    // One wave per SIMD (4 waves of 128 x 128): SLOTS stages in LDS; otherwise
    // (refined FP8) two waves per SIMD and two slots
    static const bool W1 = WAVES == 4;
    static const int SLOTS = W1 ? 3 : 2;
    static const int LDS_BYTES = SLOTS * STAGE;         // dynamic LDS
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

typedef int i32x4 __attribute__((ext_vector_type(4)));

// A packed operand's buffer resource as four scalar registers.
DEVI i32x4 packed_rsrc_s(const uint8_t *base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    return i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)p), __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)),
                 __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
}

// 64 lanes x 16 bytes from memory straight to LDS bytes lds .. lds + 1023 (one
// 16-byte unit per lane, in lane order).  As an asm statement, so that the
// compiler's wait counts do not include it: with the builtin every LDS read
// that follows waits for all such loads in flight.  The caller waits (vmcnt)
// before the barrier that publishes the stage, and before the wave ends.  The
// statement has no register outputs.
DEVI void load_to_lds(uint32_t lds, int voff, i32x4 rsrc, uint32_t soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory");
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
    // below).
    // With a.nsplit > 1 (launches with fewer output tiles than CUs) the grid
    // holds nsplit copies of the tile grid; copy q walks only stages
    // [q per, (q + 1) per) of the step order and leaves its sums in plane q
    // of a.part (a fixed-order FP64 sum of the planes follows).
    const int p = a.p, K = a.K, Kt = a.Kt, MS = a.MS, G = a.G;
    const uint32_t GS = (uint32_t)a.GS;
    const TileAt at = tile_at(blockIdx.x, gridDim.x, (uint32_t)a.nsplit, (uint32_t)((Kt + G - 1) / G) * GS,
                              (uint32_t)a.n_ntiles, (uint32_t)a.grp_v, (uint32_t)a.grp_t);
    const int split = at.split, c_class = at.cls, sg = (int)(at.member / GS);
    const int64_t ntile = at.col, msub = at.member % GS;
    const int r0 = c_class + sg * G * K;
    const int ng = Kt - sg * G < G ? Kt - sg * G : G;      // stripes of this tile

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
    const i32x4 rA = packed_rsrc_s(a.A + ((int64_t)r0 * a.GS + msub) * a.a_group, (uint32_t)a.a_span);
    const i32x4 rB = packed_rsrc_s(a.B + ntile * a.b_group, (uint32_t)a.b_group);
    // LDS address of this wave's first unit of a stage: unit ui lands at ui * 16
    const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)ring + wave * 1024);

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
    uint32_t tra[C::TM], trb[C::TN];                    // index of each tile's scale at contraction tile 0
    if constexpr (FAM == FAM_FP8) {
#pragma unroll
        for (int mi = 0; mi < C::TM; ++mi) {
            const int rho0 = wm * C::WM + mi * 32;
            const int i = rho0 / MS, i0 = rho0 % MS;
            // rows of the groups past ng are never stored: any valid scale
            int64_t row0 = (int64_t)(r0 + (i < ng ? i : 0) * K) * a.S_r + msub * MS + i0;
            row0 = row0 < a.M ? row0 : a.M - 1;
            tra[mi] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(row0 / FP8_TILE * a.a_tiles_k * 2));
        }
#pragma unroll
        for (int ni = 0; ni < C::TN; ++ni) {
            int64_t col0 = ntile * BN + wn * C::WN + ni * 32;
            col0 = col0 < a.N ? col0 : a.N - 1;
            trb[ni] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(col0 / FP8_TILE * a.b_tiles_k * 2));
        }
    }
    // a wave's columns lie in one scale tile (128-column waves, or 64 of a 128);
    // its rows do too where stripes are whole scale tiles
    static_assert(FAM != FAM_FP8 || (FP8_TILE % C::WN == 0 && BN % FP8_TILE == 0), "one column scale tile per wave");
    bool one_row_tile = true;
    if constexpr (FAM == FAM_FP8) {
#pragma unroll
        for (int mi = 1; mi < C::TM; ++mi) one_row_tile = one_row_tile && tra[mi] == tra[0];
    }
    // index of the stage's scale tile along the contraction, then to the next stage
    auto scale_col = [&]() -> uint32_t {
        // positions below p S_k < 2^31 (host); padding chunks hold zeros
        uint32_t kk = (uint32_t)pc.kb * (uint32_t)a.S_k + (uint32_t)pc.cs * 64u;
        kk = kk < (uint32_t)a.Kd ? kk : (uint32_t)a.Kd - 1;
        advance(pc);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(kk / FP8_TILE * 2));
    };
    auto stage_scales = [&]() {
        if constexpr (FAM == FAM_FP8) {
            static_assert(CPS == 1, "one 64-deep chunk per stage");
            typedef const __attribute__((address_space(4))) int32_t cint;
            cint *ea = (cint *)a.a_exps;
            cint *eb = (cint *)a.b_exps;
            const uint32_t tc = scale_col();
            auto scale = [&](cint *e, int (&s0), int &s1) {
                s0 = 127 - e[0];
                if constexpr (C::NP == 2) s1 = s0 - e[1];
            };
            int s0 = 0, s1 = 0;
            scale(eb + trb[0] + tc, s0, s1);
#pragma unroll
            for (int ni = 0; ni < C::TN; ++ni) {
                sb[0][0][ni] = s0;
                if constexpr (C::NP == 2) sb[0][1][ni] = s1;
            }
            scale(ea + tra[0] + tc, s0, s1);
#pragma unroll
            for (int mi = 0; mi < C::TM; ++mi) {
                sa[0][0][mi] = s0;
                if constexpr (C::NP == 2) sa[0][1][mi] = s1;
            }
            if (!one_row_tile) {
#pragma unroll
                for (int mi = 1; mi < C::TM; ++mi) {
                    scale(ea + tra[mi] + tc, s0, s1);
                    sa[0][0][mi] = s0;
                    if constexpr (C::NP == 2) sa[0][1][mi] = s1;
                }
            }
        }
    };

    Acc acc[C::TM][C::TN];
#pragma unroll
    for (int mi = 0; mi < C::TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < C::TN; ++ni) acc[mi][ni] = Acc{};

    uint32_t ach, bch;
    if constexpr (C::W1) {
        // One wave per SIMD; the loads of a stage write LDS themselves, so
        // neither staging registers nor LDS write instructions exist, and
        // SLOTS stages fit.  A stage's one barrier sits before its last chunk:
        // there every wave has read the whole stage s (its slot is free for
        // stage s + SLOTS) and has waited for its own loads of stage s + 1;
        // stages s + 2 .. s + SLOTS - 1 stay in flight.  Between MFMA tiles the
        // wave reads the next chunk's fragments into the other register set and
        // issues the loads, in an order pinned by sched_barrier.
        constexpr int NP = C::NP, S = C::SLOTS, LD = C::NPL / 2;   // LD: 16-byte reads per fragment
        constexpr int RD = (C::TM + C::TN) * NP * LD, TILES = C::TM * C::TN;
        constexpr int UNR = (S * CPS) % 2 ? 2 * S : S;      // stages per turn of the loop
        const int r32 = lane & 31, g = lane >> 5;
        const int a_rd = g * LD * BM * 16 + (wm * C::WM + r32) * 16;
        const int b_rd = C::A_STAGE + g * LD * BN * 16 + (wn * C::WN + r32) * 16;
        u32x4 fa[2][C::TM][NP][LD], fb[2][C::TN][NP][LD];
        // read i of a chunk: A tile 0, the B tiles, the other A tiles
        auto rd = [&](int set, const uint8_t *sl, int c, int i) {
            const int h = i % LD, P = i / LD % NP, k = i / LD / NP;
            if (k >= 1 && k <= C::TN)
                fb[set][k - 1][P][h] =
                    *(const u32x4 *)(sl + b_rd + (P * CPS + c) * BN * C::CB + h * BN * 16 + (k - 1) * 32 * 16);
            else {
                const int mi = k == 0 ? 0 : k - C::TN;
                fa[set][mi][P][h] = *(const u32x4 *)(sl + a_rd + (P * CPS + c) * BM * C::CB + h * BM * 16 + mi * 32 * 16);
            }
        };
        // FP8: exponents of the next stage's scale tiles (na, nb) and block scales
        // of the stage being multiplied (ca, cb).  The scalar loads are issued
        // among one stage's MFMAs and first used right after the next barrier,
        // where no LDS read is in flight that would have to be waited for too.
        int na[C::TM], nb = 0, ca[C::TM] = {}, cb = 0;
        auto next_scales = [&]() {
            if constexpr (FAM == FAM_FP8) {
                typedef const __attribute__((address_space(4))) int32_t cint;
                const uint32_t tc = scale_col();
                nb = ((cint *)a.b_exps)[trb[0] + tc];
                na[0] = ((cint *)a.a_exps)[tra[0] + tc];
                if (!one_row_tile) {
#pragma unroll
                    for (int i = 1; i < C::TM; ++i) na[i] = ((cint *)a.a_exps)[tra[i] + tc];
                }
            }
        };
        auto use_scales = [&]() {
            if constexpr (FAM == FAM_FP8) {
                static_assert(FORM == 0 && CPS == 1, "one scale per tile and stage");
                cb = 127 - nb;
#pragma unroll
                for (int i = 0; i < C::TM; ++i) ca[i] = 127 - na[0];
                if (!one_row_tile) {
#pragma unroll
                    for (int i = 1; i < C::TM; ++i) ca[i] = 127 - na[i];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto ld = [&](int slot, int i) {                    // load i of a stage: LPS of 4 KiB, 1 KiB per wave
            const uint32_t at = lds0 + (uint32_t)(slot * C::STAGE + (i < C::UA ? i : i - C::UA) * C::NT * 16 +
                                                  (i < C::UA ? 0 : C::A_STAGE));
            if (i < C::UA) load_to_lds(at, (int)a_off[i < C::UA ? i : 0], rA, ach);
            else load_to_lds(at, (int)b_off[i < C::UA ? 0 : i - C::UA], rB, bch);
        };
        constexpr int FIRST = 2;                            // MFMA tile after which a chunk's loads start
        // one chunk from register set `set`; meanwhile read chunk c of slot sl
        // into the other set and issue loads [l0, l1) of a stage into `slot`
        auto chunk = [&](int set, const uint8_t *sl, int c, int slot, int l0, int l1, bool last) {
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                const int mi = t / C::TN, ni = t % C::TN;
                if constexpr (FAM == FAM_FP8) {
                    auto frag = [](const u32x4 (&w)[LD]) {
                        const u32x4 lo = w[0], hi = w[LD - 1];
                        return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3],
                                     (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
                    };
                    acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        frag(fa[set][mi][0]), frag(fb[set][ni][0]), acc[mi][ni], 0, 0, 0, ca[mi], 0, cb);
                } else {
                    u32x4 av[NP], bv[NP][1];
#pragma unroll
                    for (int P = 0; P < NP; ++P) {
                        av[P] = fa[set][mi][P][0];
                        bv[P][0] = fb[set][ni][P][0];
                    }
                    Acc row[1] = {acc[mi][ni]};
                    mfma_row<FAM, FORM, 1>(row, av, bv);
                    acc[mi][ni] = row[0];
                }
#pragma unroll
                for (int i = 0; i < RD; ++i)
                    if (i * TILES / RD == t) rd(set ^ 1, sl, c, i);
#pragma unroll
                for (int i = 0; i < C::LPS; ++i)
                    if (i >= l0 && i < l1 && FIRST + (i - l0) * (TILES - FIRST) / (l1 - l0) == t) ld(slot, i);
                __builtin_amdgcn_sched_barrier(0);
                // scalar work of the next stage, while MFMAs run
                if (last && t == 0) fetch_offsets(ach, bch);
                if (last && t == 2) next_scales();
            }
        };
        // a stage's loads: an equal share in its predecessor's last chunk (right
        // after the slot is free) and in each chunk before the next barrier
        constexpr int SH = C::LPS / CPS;
        static_assert(SH * CPS == C::LPS && (S - 2) * C::LPS < 64, "load shares, vmcnt range");
#pragma unroll
        for (int q = 0; q < S; ++q) {
            fetch_offsets(ach, bch);
#pragma unroll
            for (int i = 0; i < (q + 1 < S ? C::LPS : SH); ++i) ld(q, i);
        }
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"((S - 2) * C::LPS + SH) : "memory");
#pragma unroll
        for (int i = 0; i < RD; ++i) rd(0, ring, 0, i);
        next_scales();
        for (int s = 0;;) {
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const uint8_t *cur = ring + (u % S) * C::STAGE, *nxt = ring + ((u + 1) % S) * C::STAGE;
#pragma unroll
                for (int c = 0; c + 1 < CPS; ++c)
                    chunk((u * CPS + c) & 1, cur, c + 1, (u + S - 1) % S, (c + 1) * SH, (c + 2) * SH, false);
                // this wave has read all of stage s and its share of stage s + 1 has landed
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((S - 2) * C::LPS) : "memory");
                use_scales();
                chunk((u * CPS + CPS - 1) & 1, nxt, 0, u % S, 0, SH, true);
                if (++s >= nstages) goto dma_done;
            }
        }
    dma_done:
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");   // no load may outlive the workgroup's LDS
    } else {
        // FP8: two waves per SIMD, two slots.  The loads of stage s + 1 write
        // the other slot themselves while stage s is multiplied; the barrier
        // that ends a stage follows each wave's wait for them.
        auto ld_stage = [&](int slot) {
            fetch_offsets(ach, bch);
#pragma unroll
            for (int i = 0; i < C::UA; ++i)
                load_to_lds(lds0 + (uint32_t)(slot * C::STAGE + i * C::NT * 16), (int)a_off[i], rA, ach);
#pragma unroll
            for (int i = 0; i < C::UB; ++i)
                load_to_lds(lds0 + (uint32_t)(slot * C::STAGE + C::A_STAGE + i * C::NT * 16), (int)b_off[i], rB, bch);
        };
        ld_stage(0);
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" : : : "memory");
        for (int s = 0; s < nstages; ++s) {
            const int slot = s & 1;
            ld_stage(slot ^ 1);
            stage_scales();
            __builtin_amdgcn_sched_barrier(0);
            mm_compute<FAM, FORM, BM, BN, CPS, WAVES>(acc, ring + slot * C::STAGE, ring + slot * C::STAGE + C::A_STAGE,
                                                      lane, wm, wn, sa, sb);
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");
        }
    }

    // epilogue: the collector has absorbed every partial; tile row rho is
    // row msub MS + (rho mod MS) of stripe r0 + (rho / MS) K.  A tile that lies
    // inside the matrix (all but the last ones of ragged sizes) stores without
    // checks: with them and a division per row, the 64 rows of each lane cost
    // 6 % of a BF16 4096^3 launch (110 us against 118) and 13 % of an FP8 one (66
    // against 75).
    constexpr int NE = (int)(sizeof(Acc) / sizeof(acc[0][0][0]));
    // two-piece FP16: the tile holds C' = sum a' b' of the scaled operands;
    // C = C' 2^-(e_row + e_col) (exact unless the result is subnormal)
    constexpr bool ROWSCALE = FAM == FAM_F16 && FORM == 2;
    const int64_t cbase = ntile * BN + wn * C::WN + (lane & 31);
    const uint32_t inv = (65536u + (uint32_t)MS - 1) / (uint32_t)MS;   // rho / MS = rho inv >> 16 for rho < 256
    const bool to_part = a.nsplit > 1;
    const int64_t ld = to_part ? a.N : a.ldo;
    float *dst = to_part ? (float *)a.part + (int64_t)split * a.M * a.N : (float *)a.out;
    auto store_tile = [&](auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        int ecol[C::TN];
#pragma unroll
        for (int ni = 0; ni < C::TN; ++ni) {
            ecol[ni] = 0;
            if constexpr (ROWSCALE)
                if (WHOLE || cbase + ni * C::MT < a.N)
                    ecol[ni] = row_scale_exp(((const uint32_t *)a.b_exps)[cbase + ni * C::MT]);
        }
#pragma unroll
        for (int mi = 0; mi < C::TM; ++mi) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const uint32_t rho = wm * C::WM + mi * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
                const uint32_t i = rho * inv >> 16, ir = rho - i * (uint32_t)MS;
                const uint32_t within = (uint32_t)msub * (uint32_t)MS + ir;
                const int64_t row = (int64_t)(r0 + i * (uint32_t)K) * a.S_r + within;
                if (!WHOLE && ((int)i >= ng || within >= a.S_r || row >= a.M)) continue;
                int erow = 0;
                if constexpr (ROWSCALE) erow = row_scale_exp(((const uint32_t *)a.a_exps)[row]);
                float *d = dst + row * ld + cbase;
#pragma unroll
                for (int ni = 0; ni < C::TN; ++ni) {
                    if (!WHOLE && cbase + ni * C::MT >= a.N) continue;
                    if constexpr (ROWSCALE) d[ni * C::MT] = ldexpf(acc[mi][ni][e], -(erow + ecol[ni]));
                    else d[ni * C::MT] = acc[mi][ni][e];
                }
            }
        }
    };
    const bool inside = ng * MS == BM && (msub + 1) * MS <= a.S_r && (ntile + 1) * BN <= a.N &&
                        (int64_t)(r0 + (ng - 1) * K) * a.S_r + (msub + 1) * MS <= a.M;
    if (inside) store_tile(std::true_type{});
    else store_tile(std::false_type{});
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
// A value moved within its row of 16 lanes (DPP).
template <int CTRL>
DEVI double dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// The sum over each L = 16 or 64 lanes, in every lane.
template <int L>
DEVI double lanes_sum(double v) {
    v += dpp<0xB1>(v);                         // quad_perm 1, 0, 3, 2
    v += dpp<0x4E>(v);                         // quad_perm 2, 3, 0, 1
    v += dpp<0x141>(v);                        // row_half_mirror
    v += dpp<0x140>(v);                        // row_mirror
    if constexpr (L == 64) {
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
    }
    return v;
}

// y = A x.  Every block product of the schedule belongs to one row, and the
// collector adds all K partials of a row in the wave (or the W = 2, 4 waves, or the
// 16 lanes) that owns it, so the blocks are visited in storage order: one contiguous
// sweep over the row, VE elements per lane and load (16 bytes, at any element
// alignment), U loads in flight while the U before them are multiplied.  Each
// group's FP32 sum (16 products) goes into an FP64 sum, and the lanes' FP64 sums are
// added at the end.  Bound by reading A once: FP32 8192 x 8192 39.0 us the same one
// over and over (6.9 TB/s), 46.2 others in turn (8192 x 9728, past the caches, 49.5
// and 50.9), 3001 x 2999 (rows at any alignment) 7.0, 500 x 500 3.9.  Walking the blocks partial by
// partial in the order of base A, with a cross-lane sum after each, took 39.9 and
// 47.1, 11.0 and (p = 64, K = 8) 45 us; the same walk as one pipelined sequence
// 10.7 and 4.4, but 5000 x 10000 44.5 against 35.5 here, for its index arithmetic.
// CX: complex64 (VE complex elements per load).  NT: A is read past the caches
// (it is larger than they are, by a fifth: launch_gemv_t).
// L: lanes of a row.  16 where rows are many and short (hs_gemv): a wave then takes
// four of them, whose sums across lanes cost what one row's do.
template <typename T, int CX, int NT, int L>
__global__ __launch_bounds__(256) void gemv_kernel(GemvArgs a) {
    constexpr int VE = 16 / (int)(sizeof(T) * (1 + CX)), U = 4, NT4 = VE * (1 + CX);
    typedef T V __attribute__((ext_vector_type(VE * (1 + CX))));
    typedef V VU __attribute__((aligned(sizeof(T) * (1 + CX))));
    __shared__ double red[4][2];
    const int lane = threadIdx.x & (L - 1), wave = threadIdx.x >> 6;
    const int W = L == 64 ? a.waves : 1, part = wave & (W - 1);   // W a power of two: 256 / (L W) rows per workgroup
    const int64_t row = ((int64_t)blockIdx.x * (256 / L) + threadIdx.x / L) / W;
    // past the last row: nothing to read, or (beside other rows of the wave) the last
    // row again; never stored
    const int64_t n = L < 64 || row < a.m ? a.n : 0;
    const int start = (part * L + lane) * VE, stride = L * W * VE;
    const T *Ar = (const T *)a.A + (L == 64 || row < a.m ? row : a.m - 1) * a.lda * (1 + CX);
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
    Sr = lanes_sum<L>(Sr);
    if constexpr (CX) Si = lanes_sum<L>(Si);
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
    const int64_t nwg = (int64_t)a.K * ((a.Kt + a.G - 1) / a.G) * a.GS * a.n_ntiles * a.nsplit;
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
    if (fam == FAM_FP8) return 1;
    if (fam == FAM_F32) return 2;
    // split forms one 16-deep chunk per stage (96 and 48 MFMAs per wave), BF16
    // and FP16 two (32; with four, and two slots, BF16 n = 8192 takes 0.888 ms
    // against 0.860)
    return form == 1 || form == 2 ? 1 : 2;
}

// 4 waves (one per SIMD) of 128 x 128, but 8 of 128 x 64 for refined FP8, whose
// fragments (two pieces of 32 bytes) do not fit in registers twice at 128 x 128.
// Same box, same run, against the layouts before (tiles through registers into
// two LDS slots; split forms and FP8 with 8 waves, the travelling operand of
// the split forms straight into registers), n = 8192, ms: BF16 0.806 / 0.883,
// FP16 0.863 / 0.951, two-piece FP16 2.35 / 2.50, split-BF16 4.11 / 4.23, FP32
// 7.20 / 7.28, FP8 0.427 / 0.551, refined FP8 1.09 / 1.21.
hipError_t launch_mm(int fam, int form, const MainArgs &a, hipStream_t st) {
    if (fam == FAM_F32) return launch_mm_t<FAM_F32, 0, 256, 256, 2, 4>(a, st);
    if (fam == FAM_F16 && form == 0) return launch_mm_t<FAM_F16, 0, 256, 256, 2, 4>(a, st);
    if (fam == FAM_F16 && form == 2) return launch_mm_t<FAM_F16, 2, 256, 256, 1, 4>(a, st);
    if (fam == FAM_BF16 && form == 0) return launch_mm_t<FAM_BF16, 0, 256, 256, 2, 4>(a, st);
    if (fam == FAM_BF16 && form == 1) return launch_mm_t<FAM_BF16, 1, 256, 256, 1, 4>(a, st);
    if (fam == FAM_FP8 && form == 0) return launch_mm_t<FAM_FP8, 0, 256, 256, 1, 4>(a, st);
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
    const int rows = 256 / (a.lanes * a.waves);           // per workgroup; at least one
    const dim3 grid((unsigned)((a.m + rows - 1) / rows));
    // Reads past the caches: matrices not read just before take less time (FP32,
    // two in turn, 8192 x 8192 42.9 us a call against 46.5, 8192 x 9728 50.9 against
    // 56.0), but the same one over and over, as in an iterative solver, takes more
    // while most of it stays in the 256 MiB memory-side cache: FP32 256 MiB 41.5
    // against 38.8, 280 MiB 46.5 against 44.0, 288 MiB 46.6 against 45.8 (FP64 48.8,
    // 47.5; complex 49.8, 48.2).  From 304 MiB on that is the faster one too: FP32
    // 49.5 against 51.9, FP64 50.9 against 52.9, FP32 12288 x 12288 94 against 101.
    const bool past = a.m * a.n * (int64_t)(sizeof(T) * (1 + CX)) >= (int64_t)304 << 20;
    if (a.lanes == 64 && past) HS_LAUNCH_TIMED((gemv_kernel<T, CX, 1, 64>), grid, dim3(256), 0, st, a);
    else if (a.lanes == 64) HS_LAUNCH_TIMED((gemv_kernel<T, CX, 0, 64>), grid, dim3(256), 0, st, a);
    else if (past) HS_LAUNCH_TIMED((gemv_kernel<T, CX, 1, 16>), grid, dim3(256), 0, st, a);
    else HS_LAUNCH_TIMED((gemv_kernel<T, CX, 0, 16>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_gemv(int f64, const GemvArgs &a, hipStream_t st) {
    if (a.m == 0) return hipSuccess;
    if (a.cplx) return launch_gemv_t<float, 1>(a, st);
    return f64 ? launch_gemv_t<double, 0>(a, st) : launch_gemv_t<float, 0>(a, st);
}

}  // namespace hs
