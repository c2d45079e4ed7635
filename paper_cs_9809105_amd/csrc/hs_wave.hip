// hs_wave.hip -- the hyper-systolic main loop for launches whose 256 x 256
// output tiles would leave most of the chip idle (small, narrow and
// medium-sized products).
//
// What bounds such a launch is not the MFMA rate but how many SIMDs have work
// and how long one wave's chain of chunks is.  So the output tile is small
// (64 x 64, or 32 x 32 where even those are fewer than the CUs; 96 x 64, 64 x 96 or
// 128 x 64 where these come out just under a round of the chip), and the
// workgroup's kg waves share one tile: each walks its own run of the
// tile's chunks in the step order of mm_kernel (partials l = K-1 .. 0, steps
// of stride K, chunks of a block) with its own accumulators, and the kg sums
// are added in LDS in a fixed order at the end.  A wave loads its MFMA
// fragments straight from the packed operands (their layout is the fragment
// layout: 32 lanes read 512 contiguous bytes) into D register sets, D - 1
// chunks ahead, so there is no LDS staging and no barrier in the loop.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "hs_internal.h"
#include "hs_mfma.h"

namespace hs {

bool take_timed_launch(hipEvent_t *start, hipEvent_t *stop);   // hs_kernels.hip

// TR x TC MFMA tiles per wave.  D: register sets of fragments (chunks in
// flight + 1); a set is (TR + TC) NP LD x 4 registers.  MAX_KG: eight waves
// share a tile, two to a SIMD, where sets and sums fit 256 registers (3 x 2
// tiles at 1100 x 900 x 1000: 22.4 us with 8 waves, 23.8 with 4).  One or two sets more changed
// nothing beyond noise (split-BF16 1024^3 19.1 against 18.9 us, FP32 2500^3 287
// against 289): the vector-memory path is the limit there, at about 28 bytes
// per clock and CU with it busy three quarters of the time.
template <int FAM, int FORM, int TR, int TC>
struct WvCfg {
    static const int NP = Pieces<FAM, FORM>::NP;
    static const int MT = Mfma<FAM>::T;
    static const int ROWS = TR * MT, COLS = TC * MT;
    static const int CB = FAM == FAM_FP8 || FAM == FAM_F64 ? 64 : 32;   // bytes per chunk row
    static const int LD = FAM == FAM_FP8 ? 2 : 1;                // 16-byte loads per fragment
    static const int SET = (TR + TC) * NP * LD * 4;                 // registers of one set
    static const int D = SET <= 8 ? 8 : SET <= 16 ? 4 : SET <= 24 ? 3 : 2;
    static const int MAX_KG = TR * TC <= 6 && SET * D + TR * TC * 16 <= 216 ? 8 : 4;
    static const bool EIGHT = MAX_KG == 8 && TR * TC != 4;          // 2 x 2 tiles have at most four waves
    typedef typename Mfma<FAM>::Acc Acc;
    static const int NE = (int)(sizeof(Acc) / (FAM == FAM_F64 ? 8 : 4));
};

template <int FAM, int FORM, int TR, int TC>
__global__ __launch_bounds__(64 * (WvCfg<FAM, FORM, TR, TC>::MAX_KG)) void wave_kernel(WaveArgs a) {
    typedef WvCfg<FAM, FORM, TR, TC> C;
    typedef typename C::Acc Acc;
    typedef typename std::conditional<FAM == FAM_F64, double, float>::type E;
    extern __shared__ __attribute__((aligned(32))) uint8_t red[];   // kg > 1: min(kg, 4) accumulator sets
    constexpr int NP = C::NP, MT = C::MT, LD = C::LD;
    const int lane = threadIdx.x & 63;
    const int kgi = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));

    const int p = a.p, K = a.K, Kt = a.Kt;
    const TileAt wg = tile_at(blockIdx.x, gridDim.x, (uint32_t)a.nsplit, (uint32_t)a.GS, (uint32_t)a.n_ntiles,
                              (uint32_t)a.grp_v, (uint32_t)a.grp_t);
    const int split = wg.split, cls = wg.cls;
    const uint32_t ntile = wg.col, gi = wg.member;        // column tile, group of the class
    const int rows = gi + 1 == a.GS ? a.a_last : a.a_rows;        // rows of this group
    const uint32_t nch = (uint32_t)a.nch;
    const uint32_t a_chunk = (uint32_t)(rows * C::CB), b_chunk = (uint32_t)(C::COLS * C::CB);
    const uint32_t a_piece = (uint32_t)p * nch * a_chunk, b_piece = (uint32_t)p * nch * b_chunk;
    const __amdgpu_buffer_rsrc_t rsA = packed_rsrc(a.A + cls * a.a_class + (int64_t)gi * a.a_group, a_piece * NP);
    const __amdgpu_buffer_rsrc_t rsB = packed_rsrc(a.B + (int64_t)ntile * a.b_group, b_piece * NP);

    // Fragment addresses: lane group g = lane / MT holds plane g (FP8: planes
    // 2g, 2g + 1) of row lane % MT.  Tile rows past the group's own re-read
    // row 0; they are never stored.
    const int r = lane & (MT - 1), g = lane / MT;
    int a_off[TR], a_pl;
#pragma unroll
    for (int mi = 0; mi < TR; ++mi) {
        const int row = mi * MT + r < rows ? mi * MT + r : 0;
        a_off[mi] = (g * LD * rows + row) * 16;
    }
    a_pl = rows * 16;
    const int b_off = (g * LD * C::COLS + r) * 16;

    // this wave's chunks of the workgroup's [split per, (split + 1) per)
    const int total = p * (int)nch;
    const int w0 = split * a.split_chunks;
    const int wn = total - w0 < a.split_chunks ? total - w0 : a.split_chunks;
    const int each = (wn + a.kg - 1) / a.kg;
    const int s0 = kgi * each < wn ? kgi * each : wn;
    const int n = wn - s0 < each ? wn - s0 : each;
    struct Pos { int kb, cs, j, t, n; };
    Pos q;
    {
        const uint32_t s = n > 0 ? w0 + s0 : 0, blk = s / nch;
        q.cs = (int)(s - blk * nch);
        q.t = (int)(blk / (uint32_t)Kt);
        q.j = (int)(blk - (uint32_t)q.t * Kt);
        q.kb = (int)((uint32_t)(cls + K - 1 - q.t) % (uint32_t)K) + q.j * K;
        q.n = 0;
    }
    Pos qc = q;                                          // FP8: the chunk being multiplied
    auto advance = [&](Pos &x) {                         // past the last chunk the position stays put
        if (++x.n >= n) return;
        if (++x.cs < (int)nch) return;
        x.cs = 0;
        if (++x.j < Kt) { x.kb += K; return; }
        x.j = 0;
        ++x.t;
        x.kb = (int)((uint32_t)(cls + K - 1 - x.t) % (uint32_t)K);
    };

    struct Set { u32x4 a[NP][TR][LD], b[NP][TC][LD]; };
    Set f[C::D];
    auto load = [&](Set &x) {
        const uint32_t ch = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)q.kb * nch + (uint32_t)q.cs));
        advance(q);
        const uint32_t sa = ch * a_chunk, sb = ch * b_chunk;
#pragma unroll
        for (int P = 0; P < NP; ++P)
#pragma unroll
            for (int h = 0; h < LD; ++h) {
#pragma unroll
                for (int i = 0; i < TR; ++i)
                    x.a[P][i][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                        rsA, a_off[i] + h * a_pl, (int)(sa + P * a_piece), 0));
#pragma unroll
                for (int i = 0; i < TC; ++i)
                    x.b[P][i][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                        rsB, b_off + (i * MT + h * C::COLS) * 16, (int)(sb + P * b_piece), 0));
            }
    };

    // FP8: scale tile of each row / column tile (uniform across the wave)
    int tra[TR], trb[TC];
    if constexpr (FAM == FAM_FP8) {
#pragma unroll
        for (int i = 0; i < TR; ++i) {
            const int64_t at = (int64_t)gi * a.a_rows + i * MT;
            int64_t row = (cls + at / a.S_r * K) * a.S_r + at % a.S_r;
            row = row < a.M ? row : a.M - 1;             // rows past M are never stored
            tra[i] = (int)(row / FP8_TILE);
        }
#pragma unroll
        for (int i = 0; i < TC; ++i) {
            int64_t col = (int64_t)ntile * C::COLS + i * MT;
            col = col < a.N ? col : a.N - 1;
            trb[i] = (int)(col / FP8_TILE);
        }
    }

    Acc acc[TR][TC];
#pragma unroll
    for (int mi = 0; mi < TR; ++mi)
#pragma unroll
        for (int ni = 0; ni < TC; ++ni) acc[mi][ni] = Acc{};

    auto multiply = [&](const Set &x) {
        if constexpr (FAM == FAM_FP8) {
            typedef const __attribute__((address_space(4))) int32_t cint;
            cint *ea = (cint *)a.a_exps;
            cint *eb = (cint *)a.b_exps;
            int64_t kk = (int64_t)qc.kb * a.S_k + (int64_t)qc.cs * 64;
            kk = kk < a.Kd ? kk : a.Kd - 1;              // padding chunks hold zeros
            advance(qc);
            const int tc = __builtin_amdgcn_readfirstlane((int)(kk / FP8_TILE));
            int sa[NP][TR], sb[NP][TC];
#pragma unroll
            for (int i = 0; i < TR; ++i) {
                const int ta = __builtin_amdgcn_readfirstlane((int)((tra[i] * a.a_tiles_k + tc) * 2));
                sa[0][i] = 127 - ea[ta];
                if constexpr (NP == 2) sa[1][i] = sa[0][i] - ea[ta + 1];
            }
#pragma unroll
            for (int i = 0; i < TC; ++i) {
                const int tb = __builtin_amdgcn_readfirstlane((int)((trb[i] * a.b_tiles_k + tc) * 2));
                sb[0][i] = 127 - eb[tb];
                if constexpr (NP == 2) sb[1][i] = sb[0][i] - eb[tb + 1];
            }
            auto frag = [](const u32x4 (&w)[LD]) {
                const u32x4 lo = w[0], hi = w[LD - 1];
                return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            };
#pragma unroll
            for (int mi = 0; mi < TR; ++mi)
#pragma unroll
                for (int ni = 0; ni < TC; ++ni) {
                    if constexpr (NP == 2) {             // q1 q0', q0 q1', q0 q0': smallest first
                        acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            frag(x.a[1][mi]), frag(x.b[0][ni]), acc[mi][ni], 0, 0, 0, sa[1][mi], 0, sb[0][ni]);
                        acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            frag(x.a[0][mi]), frag(x.b[1][ni]), acc[mi][ni], 0, 0, 0, sa[0][mi], 0, sb[1][ni]);
                    }
                    acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        frag(x.a[0][mi]), frag(x.b[0][ni]), acc[mi][ni], 0, 0, 0, sa[0][mi], 0, sb[0][ni]);
                }
        } else if constexpr (FAM == FAM_F64) {
            // a lane's 16 bytes are contraction elements 2g, 2g + 1 of the
            // 8-deep chunk; MFMA t takes element t of A and B alike
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int mi = 0; mi < TR; ++mi)
#pragma unroll
                    for (int ni = 0; ni < TC; ++ni) {
                        const u32x4 av = x.a[0][mi][0], bv = x.b[0][ni][0];
                        acc[mi][ni] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            __hiloint2double((int)av[2 * t + 1], (int)av[2 * t]),
                            __hiloint2double((int)bv[2 * t + 1], (int)bv[2 * t]), acc[mi][ni], 0, 0, 0);
                    }
        } else {
            u32x4 bv[NP][TC];
#pragma unroll
            for (int P = 0; P < NP; ++P)
#pragma unroll
                for (int ni = 0; ni < TC; ++ni) bv[P][ni] = x.b[P][ni][0];
#pragma unroll
            for (int mi = 0; mi < TR; ++mi) {
                u32x4 av[NP];
#pragma unroll
                for (int P = 0; P < NP; ++P) av[P] = x.a[P][mi][0];
                mfma_row<FAM, FORM, TC>(acc[mi], av, bv);
            }
        }
    };

    if (n > 0) {
#pragma unroll
        for (int d = 0; d < C::D; ++d) load(f[d]);
        for (int s = 0;;) {
#pragma unroll
            for (int d = 0; d < C::D; ++d) {
                multiply(f[d]);
                load(f[d]);
                if (++s >= n) goto done;
            }
        }
    }
done:

    // epilogue: tile row rho is position gi a_rows + rho of the class's list
    constexpr bool ROWSCALE = FAM == FAM_F16 && FORM == 2;
    const bool to_part = a.nsplit > 1;
    const uint32_t S = (uint32_t)a.S_r, base = (uint32_t)gi * (uint32_t)a.a_rows;
    const uint32_t *eca = (const uint32_t *)a.a_exps, *ecb = (const uint32_t *)a.b_exps;
    auto store = [&](int mi, int ni, int e, E v) {
        const int rho = mi * MT + (FAM == FAM_F64 ? 4 * e + g : (e >> 2) * 8 + g * 4 + (e & 3));
        const uint32_t at = base + rho, i = at / S;
        const int64_t row = (int64_t)(cls + i * K) * S + (at - i * S);
        const int64_t col = (int64_t)ntile * C::COLS + ni * MT + r;
        if (rho >= rows || row >= a.M || col >= a.N) return;
        if constexpr (ROWSCALE) v = ldexpf(v, -(row_scale_exp(eca[row]) + row_scale_exp(ecb[col])));
        if (to_part) ((E *)a.part)[((int64_t)split * a.M + row) * a.N + col] = v;
        else ((E *)a.out)[row * a.ldo + col] = v;
    };
    if (a.kg == 1) {
#pragma unroll
        for (int mi = 0; mi < TR; ++mi)
#pragma unroll
            for (int e = 0; e < C::NE; ++e)
#pragma unroll
                for (int ni = 0; ni < TC; ++ni) store(mi, ni, e, acc[mi][ni][e]);
        return;
    }
    // Every wave leaves its sums in LDS (of eight, the upper four first, so that
    // LDS holds four sets); then wave w adds and stores quads w, w + kg, .. of
    // accumulator elements, the sets in a fixed order: in FP64, rounded once,
    // where there are eight or they stand for the parts of a split step order (as
    // its planes are added), else in FP32 (there FP64 takes longer for nothing
    // that one chain had: BF16 1024^3 16.9 us against 16.4, 256^3 7.5 against 7.3).
    // (A pairwise tree after which one wave stored the tile took longer:
    // split-BF16 256^3 7.9 us against 5.8, 1024^3 22 against 19.)
    typedef E E4 __attribute__((ext_vector_type(4)));
    typedef double D4 __attribute__((ext_vector_type(4)));
    constexpr int NQ = TR * TC * C::NE / 4;                // quads per lane: (mi, ni, e / 4)
    E4 *buf = (E4 *)red;
    auto leave = [&](int w) {
#pragma unroll
        for (int mi = 0; mi < TR; ++mi)
#pragma unroll
            for (int ni = 0; ni < TC; ++ni)
#pragma unroll
                for (int h = 0; h < C::NE / 4; ++h)
                    buf[(w * NQ + (mi * TC + ni) * (C::NE / 4) + h) * 64 + lane] =
                        E4{acc[mi][ni][4 * h], acc[mi][ni][4 * h + 1], acc[mi][ni][4 * h + 2], acc[mi][ni][4 * h + 3]};
    };
    auto sum64 = [&](D4 v, int q4, int sets) {             // v + a quad of the sets
        for (int w = 0; w < sets; ++w) v += __builtin_convertvector(buf[(w * NQ + q4) * 64 + lane], D4);
        return v;
    };
    auto store_quad = [&](int q4, const E4 &v) {
        const int h = q4 % (C::NE / 4), tile = q4 / (C::NE / 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) store(tile / TC, tile % TC, 4 * h + e, v[e]);
    };
    if constexpr (C::EIGHT)
        if (a.kg == 8) {
            constexpr int QW = (NQ + 7) / 8;               // quads per wave
            D4 v[QW];
            if (kgi >= 4) leave(kgi - 4);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < QW; ++i)
                if (kgi + 8 * i < NQ) v[i] = sum64(D4{}, kgi + 8 * i, 4);
            __syncthreads();                               // the upper sets are read
            if (kgi < 4) leave(kgi);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < QW; ++i)
                if (kgi + 8 * i < NQ) store_quad(kgi + 8 * i, __builtin_convertvector(sum64(v[i], kgi + 8 * i, 4), E4));
            return;
        }
    leave(kgi);
    __syncthreads();
    for (int q4 = kgi; q4 < NQ; q4 += a.kg) {
        E4 v;
        if (a.sums64) {
            v = __builtin_convertvector(sum64(D4{}, q4, a.kg), E4);
        } else {
            v = buf[q4 * 64 + lane];
            for (int w = 1; w < a.kg; ++w) v += buf[(w * NQ + q4) * 64 + lane];
        }
        store_quad(q4, v);
    }
}

template <int FAM, int FORM, int TR, int TC>
static hipError_t launch_wave_t(const WaveArgs &a, hipStream_t st) {
    typedef WvCfg<FAM, FORM, TR, TC> C;
    if (a.kg > (C::EIGHT ? 8 : 4)) return hipErrorInvalidValue;     // the kernel has no place for more sums
    const int64_t nwg = (int64_t)a.K * a.GS * a.n_ntiles * a.nsplit;
    const unsigned lds = a.kg == 1 ? 0 : (unsigned)(a.kg < 4 ? a.kg : 4) * TR * TC * sizeof(typename C::Acc) * 64;   // <= 128 KiB
    // LDS beyond 64 KiB has to be allowed per kernel and device, once
    static std::atomic<uint64_t> allowed{0};
    int dev = 0;
    if (lds > 65536) {
        if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
        if (dev >= 64 || !(allowed.load() >> dev & 1)) {
            hipError_t e = hipFuncSetAttribute((const void *)wave_kernel<FAM, FORM, TR, TC>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 131072);
            if (e != hipSuccess) return e;
            if (dev < 64) allowed.fetch_or((uint64_t)1 << dev);
        }
    }
    hipEvent_t ts, te;
    if (take_timed_launch(&ts, &te))
        hipExtLaunchKernelGGL((wave_kernel<FAM, FORM, TR, TC>), dim3((unsigned)nwg), dim3(64 * a.kg), lds, st, ts, te, 0, a);
    else
        hipLaunchKernelGGL((wave_kernel<FAM, FORM, TR, TC>), dim3((unsigned)nwg), dim3(64 * a.kg), lds, st, a);
    return hipGetLastError();
}

// Bytes per chunk row of the packed operands of this kernel.
int wave_chunk_bytes(int fam) { return fam == FAM_FP8 || fam == FAM_F64 ? 64 : 32; }
// Tile rows (or columns) of t MFMA tiles.
int wave_tile(int fam, int t) { return t * (fam == FAM_F64 ? 16 : 32); }

hipError_t launch_wave(int fam, int form, int tr, int tc, const WaveArgs &a, hipStream_t st) {
#define HS_WV(F, O, R, C) \
    if (fam == F && form == O && tr == R && tc == C) return launch_wave_t<F, O, R, C>(a, st)
#define HS_WALL(R, C)          \
    HS_WV(FAM_F64, 0, R, C);   \
    HS_WV(FAM_F32, 0, R, C);   \
    HS_WV(FAM_F16, 0, R, C);   \
    HS_WV(FAM_F16, 2, R, C);   \
    HS_WV(FAM_BF16, 0, R, C);  \
    HS_WV(FAM_BF16, 1, R, C);  \
    HS_WV(FAM_FP8, 0, R, C);   \
    HS_WV(FAM_FP8, 1, R, C)
    HS_WALL(1, 1);
    HS_WALL(2, 2);
    HS_WV(FAM_F16, 0, 3, 2);
    HS_WV(FAM_F16, 2, 3, 2);
    HS_WV(FAM_BF16, 0, 3, 2);
    HS_WV(FAM_BF16, 1, 3, 2);
    HS_WV(FAM_F16, 0, 2, 3);
    HS_WV(FAM_F16, 2, 2, 3);
    HS_WV(FAM_BF16, 0, 2, 3);
    HS_WV(FAM_BF16, 1, 2, 3);
    HS_WV(FAM_F16, 2, 4, 2);
    HS_WV(FAM_BF16, 1, 4, 2);
#undef HS_WALL
#undef HS_WV
    return hipErrorInvalidValue;
}

}  // namespace hs
