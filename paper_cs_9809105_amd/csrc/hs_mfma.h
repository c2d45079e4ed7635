// hs_mfma.h -- device helpers shared by the two main-loop kernels
// (hs_kernels.hip, hs_wave.hip): vector types, the MFMA of each family and
// form, and the buffer resource of a packed operand.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hs_internal.h"

namespace hs {

#define DEVI __device__ __forceinline__

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // 16 bytes, a native vector
typedef int i32x8 __attribute__((ext_vector_type(8)));             // 32 fp8 values

// Scale exponent of an operand row from its amax bits: the largest e with
// amax 2^e < 2^15 is 15 - frexp_exp(amax) (frexp_exp(0) = 0: any e suits
// a row of zeros).
DEVI int row_scale_exp(uint32_t amax_bits) { return 15 - __builtin_amdgcn_frexp_expf(__uint_as_float(amax_bits)); }

// FORM 0: one piece per operand, one product.  FORM 1: three bf16 pieces,
// the six products a_i b_j with i + j <= 2, smallest first.  FORM 2: two
// f16 pieces of the row-scaled operands, the three products a_i b_j with
// i + j <= 1, smallest first; the epilogue removes the row scales.
template <int FORM> struct Form;
template <> struct Form<0> { static const int NP = 1; };
template <> struct Form<1> { static const int NP = 3; };
template <> struct Form<2> { static const int NP = 2; };

template <int FAM> struct Mfma;
template <> struct Mfma<FAM_F64> { static const int T = 16; typedef f64x4 Acc; };
template <> struct Mfma<FAM_F32> { static const int T = 32; typedef f32x16 Acc; };
template <> struct Mfma<FAM_BF16> { static const int T = 32; typedef f32x16 Acc; };
template <> struct Mfma<FAM_F16> { static const int T = 32; typedef f32x16 Acc; };
template <> struct Mfma<FAM_FP8> { static const int T = 32; typedef f32x16 Acc; };

// Pieces per operand: split-BF16 3, two-piece FP16 2, refined FP8 2 (q0,
// q1), otherwise 1.
template <int FAM, int FORM>
struct Pieces { static const int NP = FAM == FAM_FP8 ? (FORM ? 2 : 1) : Form<FORM>::NP; };

template <int FAM, int FORM, int TN, typename AccRow, typename AV, typename BV>
DEVI void mfma_row(AccRow &accr, const AV &av, const BV &bv) {
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
        if constexpr (FAM == FAM_F32) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                accr[ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av[0][t]), __uint_as_float(bv[0][ni][t]),
                                                               accr[ni], 0, 0, 0);
        } else if constexpr (FAM == FAM_F16 && FORM == 2) {
            // a1 b0, a0 b1, a0 b0: smallest first
            accr[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, av[1]),
                                                              __builtin_bit_cast(f16x8, bv[0][ni]), accr[ni], 0, 0, 0);
            accr[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, av[0]),
                                                              __builtin_bit_cast(f16x8, bv[1][ni]), accr[ni], 0, 0, 0);
            accr[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, av[0]),
                                                              __builtin_bit_cast(f16x8, bv[0][ni]), accr[ni], 0, 0, 0);
        } else if constexpr (FAM == FAM_F16) {
            accr[ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, av[0]),
                                                              __builtin_bit_cast(f16x8, bv[0][ni]), accr[ni], 0, 0, 0);
        } else if constexpr (FORM == 0) {
            accr[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[0]),
                                                               __builtin_bit_cast(bf16x8, bv[0][ni]), accr[ni], 0, 0, 0);
        } else {
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const int pa = q < 3 ? 2 - q : (q == 3 ? 1 : 0);
                const int pb = q < 3 ? q : (q == 4 ? 1 : 0);
                accr[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[pa]),
                                                                   __builtin_bit_cast(bf16x8, bv[pb][ni]), accr[ni], 0, 0, 0);
            }
        }
    }
}

// Workgroup -> (split, class, member of the class, column tile).  Workgroups are
// dealt to the 8 XCDs round robin; they are renumbered so that each XCD runs a
// contiguous range, in batches of gv members x gt column tiles, which share
// fetches in the XCD's L2.  The last batches are as small as the remainders, so
// that every number is a tile: with whole batches padded by empty ones an XCD
// could hold twice the tiles of another (split-BF16 2304^3, p = 2: 240 us
// against 122; BF16 2304^3, p = 64, K = 8: 81 against 49).
struct TileAt {
    int split, cls;
    uint32_t member, col;
};
DEVI TileAt tile_at(uint32_t id, uint32_t nwg, uint32_t nsplit, uint32_t members, uint32_t cols, uint32_t gv,
                    uint32_t gt) {
    const uint32_t xcd = id % 8, per = nwg / 8, rem = nwg % 8;
    uint32_t n = xcd * per + (xcd < rem ? xcd : rem) + id / 8;
    const uint32_t per_split = nwg / nsplit, per_cls = members * cols;
    TileAt t;
    t.split = (int)(n / per_split);
    n -= t.split * per_split;
    t.cls = (int)(n / per_cls);
    n -= t.cls * per_cls;
    const uint32_t band = gv * cols, b = n / band;       // gv members (fewer in the last band) x all columns
    n -= b * band;
    const uint32_t h = members - b * gv < gv ? members - b * gv : gv;
    const uint32_t q = n / (h * gt);                     // gt columns (fewer in the last group) of the band
    n -= q * h * gt;
    const uint32_t w = cols - q * gt < gt ? cols - q * gt : gt;
    t.member = b * gv + n / w;
    t.col = q * gt + n % w;
    return t;
}

// Buffer resource over a packed operand (raw buffer, byte addressed; the
// third dword is the gfx9 default format word).
DEVI __amdgpu_buffer_rsrc_t packed_rsrc(const uint8_t *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, (int)bytes, 0x00020000);
}

}  // namespace hs
