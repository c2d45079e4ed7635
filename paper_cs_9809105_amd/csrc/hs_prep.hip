// hs_prep.hip -- operand preparation: copies, splits or quantises the two
// row-major operands of a product into the packed tile layout described in
// hs_internal.h (pack_kernel, one launch for both), after the scans that some
// forms need first (row amaxes, FP8 tile exponents).  All of it is bound by
// memory: each operand read once per kernel, the packed image written once.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hs_internal.h"
#include "hs_mfma.h"

namespace hs {

// ---------------------------------------------------------------------------
// number formats
// ---------------------------------------------------------------------------
// Eight floats -> the 16-byte units of their three BF16 pieces,
// x = a0 + a1 + a2 with a0 = bf16(x), a1 = bf16(x - a0), a2 = bf16(x - a0 - a1):
// round to nearest even, two values per conversion instruction
// (v_cvt_pk_bf16_f32), residuals exact in FP32.  Word j of a unit holds
// elements 2j (low half) and 2j + 1.  The instruction was compared with a
// software round-to-nearest-even on 24 million values (random bit patterns,
// every exponent, exact ties, denormals): no difference.
DEVI void split3_units(const float (&x)[8], u32x4 &p0, u32x4 &p1, u32x4 &p2) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const f32x2 v = {x[2 * j], x[2 * j + 1]};
        const uint32_t w0 = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
        const f32x2 r1 = v - f32x2{__uint_as_float(w0 << 16), __uint_as_float(w0 & 0xffff0000u)};
        const uint32_t w1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(r1, bf16x2));
        const f32x2 r2 = r1 - f32x2{__uint_as_float(w1 << 16), __uint_as_float(w1 & 0xffff0000u)};
        p0[j] = w0;
        p1[j] = w1;
        p2[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r2, bf16x2));
    }
}

// float -> e4m3 (OCP FP8: 1 sign, 4 exponent bits with bias 7, 3 mantissa
// bits; largest finite 448, no infinities), round to nearest, ties to even,
// saturating at 448 (subnormals m * 2^-9, m = 1..7), four values at a time:
// gfx950's conversion instruction on values clamped to [-448, 448].  The
// instruction's rounding was compared with a software round-to-nearest-even
// encoder on every e4m3 value, every midpoint between neighbours and the
// floats next to each midpoint, both signs, values below the smallest
// subnormal and 8 million random ones: no difference.  The tests compare
// the quantisation bit for bit with the oracle's encoder.
DEVI uint32_t e4m3x4(float x0, float x1, float x2, float x3) {
    auto c = [](float x) { return fminf(fmaxf(x, -448.0f), 448.0f); };
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(c(x0), c(x1), 0, false);     // bytes 0, 1
    w = __builtin_amdgcn_cvt_pk_fp8_f32(c(x2), c(x3), w, true);          // bytes 2, 3
    return (uint32_t)w;
}
// byte B of a word of four e4m3 codes -> float (exact)
template <int B> DEVI float e4m3_byte_to_f32(uint32_t w) { return __builtin_amdgcn_cvt_f32_fp8((int)w, B); }

// Largest e with amax * 2^e <= 448 (0 for an all-zero tile), clamped so that
// the block-scale byte 127 - e stays a finite E8M0 value.
DEVI int fp8_exponent(float amax) {
    if (!(amax > 0.0f) || !(amax < 3.0e38f)) return 0;
    int E;
    const float m = frexpf(amax, &E);                      // amax = m 2^E, m in [0.5, 1)
    int e = (m <= 0.875f ? 9 : 8) - E;                     // 448 = 0.875 * 2^9
    return e < -126 ? -126 : (e > 126 ? 126 : e);
}

// ---------------------------------------------------------------------------
// FP8 tile exponents
// ---------------------------------------------------------------------------
// One workgroup per 128 x 128 scale tile: amax of the tile, then (with
// refinement) amax of the residuals a 2^e - q0, both turned into exponents.
// The tile is 128 lines of 128 contiguous floats in memory (rows of a
// K-major source, contraction rows of an MN-major one); each of the 512
// threads holds 8 float4 of it in registers (one read of the tile), line
// t * 16 + tid / 32, float4 tid % 32, so a wave reads two 512-byte lines per
// load.  vec: rows are 16-byte aligned (ld % 4 == 0, 16-byte aligned base).
// One launch takes both operands (workgroups below nb0 the first).
DEVI float wave_max(float m) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) m = fmaxf(m, __shfl_xor(m, s, 64));
    return m;
}

struct ExpPair {
    Fp8ExpArgs x[2];
    uint32_t nb0;
};

DEVI void fp8_tile_exp(const Fp8ExpArgs &a, uint32_t blk, float (&red)[2][8]) {
    const int64_t tr = blk / a.tiles_k, tc = blk % a.tiles_k;
    const int tid = threadIdx.x, wave = tid >> 6;
    // memory lines (outer index) and contiguous positions (inner index)
    const int64_t o0 = (a.kmajor ? tr : tc) * FP8_TILE, i0 = (a.kmajor ? tc : tr) * FP8_TILE;
    const int64_t olim = a.kmajor ? a.R : a.Kd, ilim = a.kmajor ? a.Kd : a.R;
    const int64_t ib = i0 + (tid & 31) * 4;
    float4 v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int64_t o = o0 + t * 16 + (tid >> 5);
        const float *q = a.src + o * a.ld + ib;
        if (a.vec && o < olim && ib + 3 < ilim) {
            v[t] = *(const float4 *)q;
        } else {
            const bool ol = o < olim;
            v[t].x = ol && ib < ilim ? q[0] : 0.f;
            v[t].y = ol && ib + 1 < ilim ? q[1] : 0.f;
            v[t].z = ol && ib + 2 < ilim ? q[2] : 0.f;
            v[t].w = ol && ib + 3 < ilim ? q[3] : 0.f;
        }
    }
    auto block_max = [&](float m, float (&r)[8]) {
        m = wave_max(m);
        if ((tid & 63) == 0) r[wave] = m;
        __syncthreads();
        float x = r[0];
#pragma unroll
        for (int w = 1; w < 8; ++w) x = fmaxf(x, r[w]);
        return x;
    };
    float m = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t)
        m = fmaxf(m, fmaxf(fmaxf(fabsf(v[t].x), fabsf(v[t].y)), fmaxf(fabsf(v[t].z), fabsf(v[t].w))));
    const float amax = block_max(m, red[0]);
    const int e = fp8_exponent(amax);
    int e1 = 0;
    if (a.refine) {
        float mr = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            // a 2^e is exact; its residual after rounding to e4m3 is exact too
            const float x0 = ldexpf(v[t].x, e), x1 = ldexpf(v[t].y, e), x2 = ldexpf(v[t].z, e),
                        x3 = ldexpf(v[t].w, e);
            const uint32_t q = e4m3x4(x0, x1, x2, x3);
            mr = fmaxf(mr, fmaxf(fmaxf(fabsf(x0 - e4m3_byte_to_f32<0>(q)), fabsf(x1 - e4m3_byte_to_f32<1>(q))),
                                 fmaxf(fabsf(x2 - e4m3_byte_to_f32<2>(q)), fabsf(x3 - e4m3_byte_to_f32<3>(q)))));
        }
        const float rmax = block_max(mr, red[1]);
        e1 = rmax > 0.0f ? fp8_exponent(rmax) : 0;
        if (e1 > 127 - e) e1 = 127 - e;                    // keep 127 - e - e1 >= 0
        if (e1 < -127 - e) e1 = -127 - e;
    }
    if (tid == 0) {
        a.exps[blk * 2] = e;
        a.exps[blk * 2 + 1] = e1;
    }
}

__global__ __launch_bounds__(512) void fp8_tile_exp_kernel(ExpPair p) {
    __shared__ float red[2][8];
    if (blockIdx.x < p.nb0) fp8_tile_exp(p.x[0], blockIdx.x, red);
    else fp8_tile_exp(p.x[1], blockIdx.x - p.nb0, red);
}

// ---------------------------------------------------------------------------
// pack: one unit
// ---------------------------------------------------------------------------
// Eight floats of one row -> the 16-byte units of their two FP16 pieces,
// x' = x 2^e, a0 = f16(x'), a1 = f16(x' - a0): round to nearest even, the
// residual exact in FP32 (a0 is within a factor 2 of x', or both lie below
// 2^-14 on the 2^-24 grid).  Word j holds elements 2j (low half), 2j + 1.
DEVI void split2_f16_units(const float (&x)[8], int e, u32x4 &p0, u32x4 &p1) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const f32x2 v = {ldexpf(x[2 * j], e), ldexpf(x[2 * j + 1], e)};   // exact
        const f16x2 h0 = __builtin_convertvector(v, f16x2);
        const f32x2 r = v - __builtin_convertvector(h0, f32x2);
        p0[j] = __builtin_bit_cast(uint32_t, h0);
        p1[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
    }
}

template <int KIND> struct PackTraits;
template <> struct PackTraits<PK_F64> { typedef double S; static const int UE = 2; static const int ESZ = 8; static const int NP = 1; };
template <> struct PackTraits<PK_F32> { typedef float S; static const int UE = 4; static const int ESZ = 4; static const int NP = 1; };
template <> struct PackTraits<PK_B16> { typedef uint16_t S; static const int UE = 8; static const int ESZ = 2; static const int NP = 1; };
template <> struct PackTraits<PK_SPLIT3> { typedef float S; static const int UE = 8; static const int ESZ = 2; static const int NP = 3; };
template <> struct PackTraits<PK_FP8> { typedef float S; static const int UE = 16; static const int ESZ = 1; static const int NP = 2; };
template <> struct PackTraits<PK_SPLIT2F16> { typedef float S; static const int UE = 8; static const int ESZ = 2; static const int NP = 2; };

// Position rr of group grp: the operand row it holds, if any (rows past a
// list or the operand are padding), and where the group lies.
struct GroupAt {
    int64_t row;
    bool valid;
    uint32_t rows;            // rows of the group: rr >= rows is outside it
    int64_t base;             // byte offset of the group
};

DEVI GroupAt group_at(const PackArgs &a, uint32_t grp, uint32_t rr) {
    const OperandGeom &g = a.g;
    const uint32_t GS = (uint32_t)g.GS, c = fast_div(grp, a.by_GS), gi = grp - c * GS;
    const uint32_t at = gi * (uint32_t)g.grp_rows + rr;      // host: below 2^32
    const uint32_t i = fast_div(at, a.by_run);
    GroupAt r;
    r.row = (int64_t)(c + i * g.step) * g.run + (at - i * g.run);
    r.valid = i < g.runs && r.row < g.R;
    r.rows = (uint32_t)(gi + 1 == GS ? g.last_rows : g.grp_rows);
    r.base = c * g.list_bytes + gi * g.group_bytes;
    return r;
}

// Write one 16-byte unit (of each piece) of the packed image: row rr of
// group grp, block kb, chunk ch, plane half, from the unit's values.
template <int KIND>
DEVI void pack_emit(const PackArgs &a, const GroupAt &at, uint32_t kb, uint32_t ch, uint32_t half, uint32_t rr,
                    int64_t kk0, const float *vals_f, const double *vals_d, const uint16_t *vals_h) {
    if (rr >= at.rows) return;
    const OperandGeom &g = a.g;
    const int64_t row = at.row, piece = at.rows * g.row_bytes;
    const bool rvalid = at.valid;
    // chunk = UPR planes of 16 bytes per row: [plane][row][16 bytes]
    // [group][piece][block][chunk][plane][row][16 bytes]
    const int64_t inner = ((int64_t)kb * (uint32_t)g.nch + ch) * at.rows * g.chunk_bytes + ((int64_t)half * at.rows + rr) * 16;
    uint8_t *dst = (uint8_t *)a.dst + at.base + inner;
    auto put = [&](int64_t o, const u32x4 &w) { *(u32x4 *)(dst + o) = w; };
    if constexpr (KIND == PK_F64) {
        put(0, __builtin_bit_cast(u32x4, make_double2(vals_d[0], vals_d[1])));
    } else if constexpr (KIND == PK_F32) {
        put(0, u32x4{__float_as_uint(vals_f[0]), __float_as_uint(vals_f[1]), __float_as_uint(vals_f[2]),
                     __float_as_uint(vals_f[3])});
    } else if constexpr (KIND == PK_B16) {
        u32x4 w;
        w[0] = vals_h[0] | ((uint32_t)vals_h[1] << 16);
        w[1] = vals_h[2] | ((uint32_t)vals_h[3] << 16);
        w[2] = vals_h[4] | ((uint32_t)vals_h[5] << 16);
        w[3] = vals_h[6] | ((uint32_t)vals_h[7] << 16);
        put(0, w);
    } else if constexpr (KIND == PK_FP8) {
        // all 16 elements of the unit lie in one 128 x 128 scale tile
        int e = 0, e1 = 0;
        if (rvalid && kk0 < g.Kd) {
            const int64_t t2 = ((row / FP8_TILE) * a.exp_tiles_k + kk0 / FP8_TILE) * 2;
            e = a.exps[t2];
            e1 = a.exps[t2 + 1];
        }
        u32x4 w0, w1 = {0, 0, 0, 0};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            float xs[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) xs[i] = ldexpf(vals_f[4 * d + i], e);   // exact
            w0[d] = e4m3x4(xs[0], xs[1], xs[2], xs[3]);
            if (a.refine) {
                // the residual a 2^e - q0 is exact; scaled by 2^e1, rounded again
                const uint32_t q = w0[d];
                w1[d] = e4m3x4(ldexpf(xs[0] - e4m3_byte_to_f32<0>(q), e1), ldexpf(xs[1] - e4m3_byte_to_f32<1>(q), e1),
                               ldexpf(xs[2] - e4m3_byte_to_f32<2>(q), e1), ldexpf(xs[3] - e4m3_byte_to_f32<3>(q), e1));
            }
        }
        put(0, w0);
        if (a.refine) put(piece, w1);
    } else if constexpr (KIND == PK_SPLIT2F16) {
        const int e = rvalid ? row_scale_exp(((const uint32_t *)a.exps)[row]) : 0;
        u32x4 w0, w1;
        split2_f16_units(*(const float(*)[8])vals_f, e, w0, w1);
        put(0, w0);
        put(piece, w1);
    } else {   // PK_SPLIT3: a0 = bf16(a), a1 = bf16(a - a0), a2 = bf16(a - a0 - a1)
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = vals_f[e];
        u32x4 w0, w1, w2;
        split3_units(x, w0, w1, w2);
        put(0, w0);
        put(piece, w1);
        put(2 * piece, w2);
    }
}

// ---------------------------------------------------------------------------
// row amax of the two-piece FP16 split
// ---------------------------------------------------------------------------
// One launch scans both operands (workgroups below nb0 take the first).  It is
// bound by reading each operand once.  NaNs are skipped (fmaxf); they reach the
// product through the values themselves.  Every source is read 16 bytes at a
// time at whatever alignment its elements have (one element a load where rows
// are not 16-byte aligned, whole calls of two-piece FP16: tn 4097 x 2049 x 8191 741
// us, 575 here; 64 x 513 x 4097 105 and 42), the last columns of a row by reading its
// last four again.
//   K-major source: one wave per row.
//   MN-major source (element (kk, c) of the float view at src[kk ld + c]): a
//   workgroup owns 32 float columns (one 128-byte line) over all contraction
//   rows, 64 rows per pass, 8 passes in flight, so the result needs neither
//   atomics nor a cleared buffer (columns of 4096 x 2048 and of 4096 x 8192
//   together 49 us; two fills and two slab scans with atomics 93).
struct AmaxPair {
    RowAmaxArgs x[2];
    uint32_t nb0;
};
const int AMAX_COLS = 32;

DEVI float4 load4(const float *q) {
    float4 v;
    __builtin_memcpy(&v, q, 16);
    return v;
}
DEVI int64_t amax_ncol(const RowAmaxArgs &a) { return (a.embed == EMB_TRANS || a.embed == EMB_CONJ) ? 2 * a.R : a.R; }
DEVI int64_t amax_nk(const RowAmaxArgs &a) { return a.embed == EMB_NONE ? a.Kd : a.Kd / 2; }

template <int KMAJOR>
DEVI void row_amax_one(const RowAmaxArgs &a, uint32_t blk, float (&red)[64][AMAX_COLS + 1]) {
    const int tid = threadIdx.x;
    if constexpr (KMAJOR) {
        const int64_t row = (int64_t)blk * 8 + (tid >> 6);
        const int lane = tid & 63;
        if (row >= a.R) return;
        const float *q = a.src + (a.embed == EMB_BLOCKS_H ? row >> 1 : row) * a.ld;
        float m = 0.f;
        const int64_t k4 = a.Kd / 4 * 4;
#pragma unroll 4
        for (int64_t k = lane * 4; k < k4; k += 256) {
            const float4 v = load4(q + k);
            m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
        }
        if (k4 + lane < a.Kd) m = fmaxf(m, fabsf(q[k4 + lane]));
        m = wave_max(m);
        if (lane == 0) a.amax[row] = __float_as_uint(m);
        return;
    }
    const int64_t ncol = amax_ncol(a), nk = amax_nk(a);
    const int64_t c0 = (int64_t)blk * AMAX_COLS;
    constexpr int LANES = AMAX_COLS / 4, ROWS = 512 / LANES;   // threads per row, 4 columns each
    int64_t c = c0 + (tid % LANES) * 4;
    if (c < ncol && c + 3 >= ncol && ncol - 4 >= c0) c = ncol - 4;     // the block's last columns again
    const int r0 = tid / LANES;
    float m0 = 0.f, m1 = 0.f, m2 = 0.f, m3 = 0.f;
    if (c + 3 < ncol) {
#pragma unroll 8
        for (int64_t kk = r0; kk < nk; kk += ROWS) {
            const float4 v = load4(a.src + kk * a.ld + c);
            m0 = fmaxf(m0, fabsf(v.x));
            m1 = fmaxf(m1, fabsf(v.y));
            m2 = fmaxf(m2, fabsf(v.z));
            m3 = fmaxf(m3, fabsf(v.w));
        }
    } else {
#pragma unroll 8
        for (int64_t kk = r0; kk < nk; kk += ROWS) {
            const float *q = a.src + kk * a.ld + c;
            if (c < ncol) m0 = fmaxf(m0, fabsf(q[0]));
            if (c + 1 < ncol) m1 = fmaxf(m1, fabsf(q[1]));
            if (c + 2 < ncol) m2 = fmaxf(m2, fabsf(q[2]));
        }
    }
    float *d = &red[r0][c - c0];
    d[0] = m0; d[1] = m1; d[2] = m2; d[3] = m3;
    __syncthreads();
    if (tid >= AMAX_COLS || c0 + tid >= ncol) return;
    float m = 0.f;
    for (int r = 0; r < ROWS; ++r) m = fmaxf(m, red[r][tid]);
    // complex sources: a pair of float columns (both in this workgroup, and in
    // neighbouring lanes) shares its rows of the embedding
    if (a.embed != EMB_NONE) {
        m = fmaxf(m, __shfl_xor(m, 1));
        if (a.embed != EMB_BLOCKS) {
            if (!(tid & 1)) a.amax[(c0 + tid) >> 1] = __float_as_uint(m);
            return;
        }
    }
    a.amax[c0 + tid] = __float_as_uint(m);
}

template <int KA, int KB>
__global__ __launch_bounds__(512) void row_amax_kernel(AmaxPair p) {
    __shared__ float red[64][AMAX_COLS + 1];
    if (blockIdx.x < p.nb0) row_amax_one<KA>(p.x[0], blockIdx.x, red);
    else row_amax_one<KB>(p.x[1], blockIdx.x - p.nb0, red);
}

// The same by slabs (where launch_row_amax says): a workgroup takes 1024 columns,
// 4 per thread, of 256 contraction rows, then one atomic max per column into its
// row (two for EMB_BLOCKS) of the zero-filled amax.  Workgroup b takes column
// block b % ncb of slab b / ncb.  (Fewer columns and the threads below one another
// multiply the atomics: 64 x 32 x 524288, the call, 1044 us; waves below one another
// 1315, quarter waves 2432.)
__global__ __launch_bounds__(256) void row_amax_slab_kernel(RowAmaxArgs a) {
    const int64_t ncol = amax_ncol(a), nk = amax_nk(a);
    const int64_t ncb = (ncol + 1023) / 1024;
    int64_t c = (int64_t)(blockIdx.x % ncb) * 1024 + threadIdx.x * 4;
    const int64_t k0 = (int64_t)(blockIdx.x / ncb) * 256, k1 = k0 + 256 < nk ? k0 + 256 : nk;
    float m[4] = {0.f, 0.f, 0.f, 0.f};
    if (ncol < 4) {                                        // fewer than 16 bytes: a thread per row
        const int64_t kk = k0 + threadIdx.x;
#pragma unroll
        for (int j = 0; j < 3; ++j) m[j] = wave_max(kk < k1 && j < ncol ? fabsf(a.src[kk * a.ld + j]) : 0.f);
        if (threadIdx.x & 63) return;
        c = 0;
    } else {
        if (c >= ncol) return;
        if (c + 3 >= ncol) c = ncol - 4;                   // the last columns again: a maximum does not mind
#pragma unroll 8
        for (int64_t kk = k0; kk < k1; ++kk) {
            const float4 v = load4(a.src + kk * a.ld + c);
            m[0] = fmaxf(m[0], fabsf(v.x));
            m[1] = fmaxf(m[1], fabsf(v.y));
            m[2] = fmaxf(m[2], fabsf(v.z));
            m[3] = fmaxf(m[3], fabsf(v.w));
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (c + j >= ncol) continue;
        const uint32_t bits = __float_as_uint(m[j]);
        if (a.embed == EMB_BLOCKS) {
            atomicMax(a.amax + ((c + j) & ~(int64_t)1), bits);
            atomicMax(a.amax + ((c + j) | 1), bits);
        } else {
            atomicMax(a.amax + (a.embed == EMB_NONE ? c + j : (c + j) >> 1), bits);
        }
    }
}

// ---------------------------------------------------------------------------
// pack: the kernel
// ---------------------------------------------------------------------------
// t mod v.d, and t divided by it
DEVI uint32_t pop(uint32_t &t, const FastDiv &v) {
    const uint32_t q = fast_div(t, v), r = t - q * v.d;
    t = q;
    return r;
}

// An MN-major unit of pack_kernel's numbering: row rr of group grp, block
// kb, chunk ch, plane half, and where its elements lie in the source.
struct MnUnit {
    uint32_t rr, half, ch, kb;
    GroupAt at;
    int64_t kin0, kk0;
};

template <int KIND>
DEVI MnUnit mn_decode(uint32_t u, const PackArgs &a) {
    typedef PackTraits<KIND> T;
    const OperandGeom &g = a.g;
    const int KC = g.chunk_bytes / T::ESZ;
    MnUnit d;
    uint32_t t = u;
    d.rr = pop(t, a.by_rows);
    d.half = t & ((1u << a.upr_log) - 1);
    t >>= a.upr_log;
    d.ch = pop(t, a.by_chunks);
    d.kb = pop(t, a.by_p);
    d.at = group_at(a, t, d.rr);
    d.kin0 = (int64_t)d.ch * KC + d.half * T::UE;
    d.kk0 = (int64_t)d.kb * g.S_k + d.kin0;
    return d;
}

// MN-major source, transposed through LDS: the workgroup's 256 units (rows
// fastest, see mn_decode) are read as 16-byte runs of RW = 4 (FP32) or 8
// (16-bit) rows per contraction index -- consecutive lanes read consecutive
// runs, one contiguous stretch per group -- into an [element][unit] tile, then
// each thread packs and writes its own unit, so consecutive threads write
// consecutive 16-byte rows.  Host: rows of the source 16-byte aligned, grp_rows
// and, for a striped operand, S_r multiples of RW; total_units is then one too.
// U: such blocks of 256 units per workgroup, their loads issued together.
template <int KIND, int U>
DEVI void pack_mn_block(const PackArgs &a, uint32_t blk, void *lds) {
    typedef PackTraits<KIND> T;
    typedef typename T::S S;
    constexpr int UE = T::UE, RW = 16 / (int)sizeof(S), RUNS = 256 / RW;
    S(*tile)[256] = (S(*)[256])lds;             // [U][UE][256]
    const OperandGeom &g = a.g;
    const S *src = (const S *)a.src;
    const uint32_t base = blk * (256u * U);
    constexpr int PER = UE * RUNS / 256;        // runs per thread and block of units
    union Run { u32x4 w; S s[RW]; } v[U * PER];
#pragma unroll
    for (int i = 0; i < U * PER; ++i) {
        const uint32_t q = threadIdx.x + 256u * (i % PER);
        const uint32_t run = q % RUNS, e = q / RUNS;
        const uint32_t u = base + i / PER * 256u + run * RW;     // units u .. u + RW - 1: rows rr .. of one group
        v[i].w = u32x4{0, 0, 0, 0};
        if (u < (uint32_t)a.total_units) {
            const MnUnit d = mn_decode<KIND>(u, a);
            const int64_t kk = d.kk0 + e;
            if (d.at.valid && d.kin0 + e < g.S_k && kk < g.Kd) {
                const S *q4 = src + kk * a.ld + d.at.row;
                if (d.at.row + RW <= g.R) {     // one stripe: S_r % RW == 0
                    v[i].w = *(const u32x4 *)q4;
                } else {
#pragma unroll
                    for (int r = 0; r < RW; ++r)
                        if (d.at.row + r < g.R) v[i].s[r] = q4[r];
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < U * PER; ++i) {
        const uint32_t q = threadIdx.x + 256u * (i % PER);
        *(u32x4 *)&tile[i / PER * UE + q / RUNS][q % RUNS * RW] = v[i].w;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < U; ++b) {
        const uint32_t u = base + b * 256u + threadIdx.x;
        if (u >= (uint32_t)a.total_units) return;
        const MnUnit d = mn_decode<KIND>(u, a);
        float vals_f[UE];
        double vals_d[1] = {0.0};
        uint16_t vals_h[UE];
#pragma unroll
        for (int e = 0; e < UE; ++e) {
            if constexpr (KIND == PK_B16) vals_h[e] = tile[b * UE + e][threadIdx.x];
            else vals_f[e] = tile[b * UE + e][threadIdx.x];
        }
        pack_emit<KIND>(a, d.at, d.kb, d.ch, d.half, d.rr, d.kk0, vals_f, vals_d, vals_h);
    }
}

// One thread makes one 16-byte unit of the packed image (for the split form,
// the same unit of each of the three pieces).  Consecutive threads take
// consecutive rows of one (group, block, chunk, plane), so the packed writes
// are contiguous; for a row-major (MN-major) source the reads are contiguous
// too, for a K-major source each thread reads its own 16-32 bytes of a row.
// A unit: where it goes, and its 16-byte loads if its elements lie side by side.
template <int KIND>
struct PackUnit {
    typedef PackTraits<KIND> T;
    static const int NV = T::UE * (int)sizeof(typename T::S) / 16;
    GroupAt at;
    uint32_t rr, half, ch, kb;
    int64_t kin0, kk0;
    bool live, run;
    u32x4 w[NV];
};

template <int KIND, int KMAJOR>
DEVI void unit_load(const PackArgs &a, uint32_t u, PackUnit<KIND> &x) {
    typedef PackTraits<KIND> T;
    typedef typename T::S S;
    const OperandGeom &g = a.g;
    x.live = false;
    if (u >= (uint32_t)a.total_units) return;               // host: total_units < 2^32
    const int KC = g.chunk_bytes / T::ESZ;      // elements per chunk row
    uint32_t t = u, rr, half, ch, kb;
    if (KMAJOR) {
        // 8 x 8 blocks of (row, unit along the contraction): a wave reads 8
        // rows x 8 consecutive units (128-256 contiguous bytes per row) and
        // writes, per (chunk, plane), 8 consecutive rows (128 bytes).
        const uint32_t nu = (uint32_t)g.nch << a.upr_log;      // units along one block row
        const uint32_t uu = t % 8;  t /= 8;
        const uint32_t rlo = t % 8; t /= 8;
        const uint32_t ku = pop(t, a.by_chunks) * 8 + uu;
        rr = pop(t, a.by_rows) * 8 + rlo;
        if (ku >= nu || rr >= (uint32_t)g.grp_rows) return;
        ch = ku >> a.upr_log;
        half = ku & ((1u << a.upr_log) - 1);
    } else {
        rr = pop(t, a.by_rows);
        half = t & ((1u << a.upr_log) - 1);
        t >>= a.upr_log;
        ch = pop(t, a.by_chunks);
    }
    kb = pop(t, a.by_p);
    x.live = true;
    x.at = group_at(a, t, rr);
    x.rr = rr; x.half = half; x.ch = ch; x.kb = kb;
    x.kin0 = (int64_t)ch * KC + half * T::UE;
    x.kk0 = (int64_t)kb * g.S_k + x.kin0;
    x.run = KMAJOR && a.embed == EMB_NONE && x.kk0 + T::UE <= g.Kd;
    if (x.run) {
        // The unit's elements lie side by side in the row: 16-byte loads at the
        // elements' own alignment, what belongs to the next block cleared.
        // (One element a load wherever rows or blocks were not 16-byte aligned:
        // split-BF16 1100 x 900 x 1000 in 125-wide blocks, the call, 31.3 us, 30.0 here;
        // the complex step of 1000 x 700 x 900 149.2 and 147.8.)
        const bool ok = x.at.valid && x.kin0 < g.S_k;
        const S *q = (const S *)a.src + x.at.row * a.ld + x.kk0;
#pragma unroll
        for (int i = 0; i < x.NV; ++i) {
            x.w[i] = u32x4{0, 0, 0, 0};
            if (ok) __builtin_memcpy(&x.w[i], q + i * (16 / (int)sizeof(S)), 16);
        }
    }
}

template <int KIND, int KMAJOR>
DEVI void unit_store(const PackArgs &a, const PackUnit<KIND> &x) {
    typedef PackTraits<KIND> T;
    typedef typename T::S S;
    if (!x.live) return;
    const OperandGeom &g = a.g;
    const int64_t row = x.at.row, kin0 = x.kin0, kk0 = x.kk0;
    const bool rvalid = x.at.valid;
    const S *src = (const S *)a.src;
    float vals_f[T::UE];
    double vals_d[T::UE];
    uint16_t vals_h[T::UE];
    if (KMAJOR && x.run) {
        constexpr int SB = (int)sizeof(S);             // source element bytes
        const int have = g.S_k - kin0 < T::UE ? (int)(g.S_k - kin0) : T::UE;
#pragma unroll
        for (int e = 0; e < T::UE; ++e) {
            const int byte = e * SB;
            const uint32_t word = x.w[byte / 16][(byte % 16) / 4];
            if constexpr (KIND == PK_F64) {
                vals_d[e] = e < have ? __hiloint2double((int)x.w[byte / 16][(byte % 16) / 4 + 1], (int)word) : 0.0;
            } else if constexpr (KIND == PK_B16) {
                vals_h[e] = e < have ? (uint16_t)(word >> ((byte % 4) * 8)) : (uint16_t)0;
            } else {
                vals_f[e] = e < have ? __uint_as_float(word) : 0.0f;
            }
        }
    } else {
#pragma unroll
        for (int e = 0; e < T::UE; ++e) {
            const int64_t kin = kin0 + e;
            const int64_t kk = kk0 + e;
            const bool ok = rvalid && kin < g.S_k && kk < g.Kd;
            int64_t idx = KMAJOR ? row * a.ld + kk : kk * a.ld + row;
            bool neg = false;
            if constexpr (KIND == PK_F32 || KIND == PK_SPLIT3 || KIND == PK_SPLIT2F16) {
                // complex sources: sr = kk % 2 and c = row % 2 pick the entry
                // of the 2 x 2 block [[re, im], [-im, re]]
                const int64_t sr = kk & 1, c = row & 1;
                if (!KMAJOR && a.embed == EMB_BLOCKS) {
                    idx = (kk >> 1) * a.ld + (row - c) + (sr ^ c);
                    neg = sr == 1 && c == 0;
                } else if (KMAJOR && a.embed == EMB_BLOCKS_H) {
                    // conj(x): the im entries change sign
                    idx = (row >> 1) * a.ld + 2 * (kk >> 1) + (sr ^ c);
                    neg = sr == 0 && c == 1;
                } else if (!KMAJOR && (a.embed == EMB_CONJ || a.embed == EMB_TRANS)) {
                    idx = (kk >> 1) * a.ld + 2 * row + sr;
                    neg = a.embed == EMB_CONJ && sr == 1;
                }
            }
            if constexpr (KIND == PK_F64) vals_d[e] = ok ? (double)src[idx] : 0.0;
            else if constexpr (KIND == PK_B16) vals_h[e] = ok ? (uint16_t)src[idx] : (uint16_t)0;
            else vals_f[e] = ok ? (neg ? -(float)src[idx] : (float)src[idx]) : 0.0f;
        }
    }
    pack_emit<KIND>(a, x.at, x.kb, x.ch, x.half, x.rr, kk0, vals_f, vals_d, vals_h);
}

// U units a thread, 256 apart, their loads issued before the first is used.
template <int KIND, int KMAJOR, int U>
DEVI void pack_block(const PackArgs &a, uint32_t blk) {
    PackUnit<KIND> x[U];
#pragma unroll
    for (int i = 0; i < U; ++i) unit_load<KIND, KMAJOR>(a, (blk * U + i) * 256u + threadIdx.x, x[i]);
#pragma unroll
    for (int i = 0; i < U; ++i) unit_store<KIND, KMAJOR>(a, x[i]);
}

// Both operands of a product in one launch: workgroups below nb0 pack the
// first.  A product's preparation is one kernel instead of two (FP64 256^3, a
// whole call: 18.1 us against 21.4), and a small operand's workgroups run beside
// the other's.  How each source is read is a template argument.
struct PackPair {
    PackArgs x[2];
    uint32_t nb0;
};

template <int KIND, int MODE, int U>
DEVI void pack_one(const PackArgs &a, uint32_t blk, void *lds) {
    if constexpr (MODE == PACK_MN_LDS) pack_mn_block<KIND, U>(a, blk, lds);
    else pack_block<KIND, MODE == PACK_K, U>(a, blk);
}

template <int KIND, int MA, int MB, int U>
__global__ __launch_bounds__(256) void pack_kernel(PackPair p) {
    constexpr bool LDS = MA == PACK_MN_LDS || MB == PACK_MN_LDS;
    typedef PackTraits<KIND> T;
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS ? U * T::UE * 256 * sizeof(typename T::S) : 16];
    if (blockIdx.x < p.nb0) pack_one<KIND, MA, U>(p.x[0], blockIdx.x, lds);
    else pack_one<KIND, MB, U>(p.x[1], blockIdx.x - p.nb0, lds);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned nblocks(int64_t work) { return (unsigned)((work + 255) / 256); }

// Launches one grid of na + nb workgroups of `threads` for both operands, or,
// where those are 2^32 threads or more (the runtime's limit), a grid for each:
// launch(pair, workgroups) with pair.nb0 workgroups for the first operand.
template <class Pair, class Launch>
static hipError_t launch_pair(Pair p, unsigned na, unsigned nb, unsigned threads, Launch launch) {
    p.nb0 = na;
    if (na + nb == 0) return hipSuccess;
    if (((uint64_t)na + nb) * threads >> 32 == 0) {
        launch(p, na + nb);
        return hipGetLastError();
    }
    if (na) {
        launch(p, na);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (nb) {
        p.nb0 = 0;
        launch(p, nb);
    }
    return hipGetLastError();
}

// Units per thread.  A unit of the 16-bit and FP32 forms is one 16-byte load and
// one such store; with one a thread too few bytes are in flight.  Four where
// that leaves every CU 16 workgroups, and not for the element-wise MN reads:
// both operands of FP32 4096^3, transposed, 65 to 56 us (268 MB: 4.1 to 4.8 TB/s),
// of BF16 8192^3 143 to 138 (537 MB: 3.8 to 3.9 TB/s).  The forms with pieces have
// two loads and two or three stores a unit and reach 5 to 6 TB/s with one.
static int units_per_thread(int kind, const PackArgs &a, const PackArgs &b) {
    if ((kind != PK_B16 && kind != PK_F32) || a.mode == PACK_MN || b.mode == PACK_MN) return 1;
    const int64_t n = a.total_units + b.total_units;
    return n >= (int64_t)16 * 256 * 1024 && n < (int64_t)1 << 31 ? 4 : 1;
}

template <int KIND>
static hipError_t launch_pack_k(const PackArgs &a, const PackArgs &b, hipStream_t st) {
    const int ma = a.mode, mb = b.mode, U = units_per_thread(KIND, a, b);
    const unsigned na = nblocks((a.total_units + U - 1) / U), nb = nblocks((b.total_units + U - 1) / U);
#define HS_PACK_U(A_, B_, U_)                                                                                  \
    if (ma == A_ && mb == B_ && U == U_)                                                                       \
        return launch_pair(PackPair{{a, b}, 0}, na, nb, 256, [&](const PackPair &p, unsigned n) {               \
            hipLaunchKernelGGL((pack_kernel<KIND, A_, B_, U_>), dim3(n), dim3(256), 0, st, p);                  \
        });
#define HS_PACK(A_, B_)                                                                          \
    HS_PACK_U(A_, B_, 1)                                                                         \
    if constexpr ((KIND == PK_B16 || KIND == PK_F32) && A_ != PACK_MN && B_ != PACK_MN) {        \
        HS_PACK_U(A_, B_, 4)                                                                     \
    }
    // the static operand is read along the contraction (NN, NT) or across it (TN)
    HS_PACK(PACK_K, PACK_K)
    HS_PACK(PACK_K, PACK_MN)
    HS_PACK(PACK_MN, PACK_MN)
    if constexpr (KIND != PK_F64) {
        HS_PACK(PACK_K, PACK_MN_LDS)
        HS_PACK(PACK_MN, PACK_MN_LDS)
        HS_PACK(PACK_MN_LDS, PACK_MN)
        HS_PACK(PACK_MN_LDS, PACK_MN_LDS)
    }
#undef HS_PACK
#undef HS_PACK_U
    return hipErrorInvalidValue;
}

hipError_t launch_pack(int kind, const PackArgs &a, const PackArgs &b, hipStream_t st) {
    switch (kind) {
        case PK_F64: return launch_pack_k<PK_F64>(a, b, st);
        case PK_F32: return launch_pack_k<PK_F32>(a, b, st);
        case PK_B16: return launch_pack_k<PK_B16>(a, b, st);
        case PK_SPLIT3: return launch_pack_k<PK_SPLIT3>(a, b, st);
        case PK_FP8: return launch_pack_k<PK_FP8>(a, b, st);
        case PK_SPLIT2F16: return launch_pack_k<PK_SPLIT2F16>(a, b, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_fill_zero(int f64, void *Cout, int64_t M, int64_t N, int64_t ldc, hipStream_t st);

// Row amaxes of both operands.  An MN-major source goes through the slab kernel
// where a workgroup's walk over all rows would be the longer wait (over 8192 rows
// on fewer than 128 workgroups of 32 columns), and where it is larger than the
// memory-side cache: there long stretches of a row are read faster, and of rows
// that do not start on 128-byte lines each line between two workgroups' columns
// would be read twice.  Whole calls with m = 64, n x k (slabs / columns), us:
// 33 x 65537 111 / 401, 512 x 131072 420 / 724, 1000 x 16384 71 / 82, 32 x 16384 40.5 /
// 41.3, but 2048 x 8192 67 / 62; 10240 x 10240 379 / 402, 16384 x 16384 914 / 929, but
// 16384 x 2048 147 / 140; unaligned 8191 x 16385 586 / 630, 16383 x 4097 304 / 317.
// Of complex sources on whole lines the slabs' atomics, two per column, cost what
// they save: 4096 x 8192 558 / 548.
hipError_t launch_row_amax(const RowAmaxArgs &a, const RowAmaxArgs &b, hipStream_t st) {
    if (!a.kmajor && b.kmajor) return hipErrorInvalidValue;    // no product reads its operands so
    AmaxPair p{};
    unsigned nb[2] = {0, 0};
    const RowAmaxArgs *in[2] = {&a, &b};
    for (int i = 0; i < 2; ++i) {
        RowAmaxArgs &x = p.x[i];
        x = *in[i];
        if (x.R == 0) continue;
        if (x.kmajor) {
            nb[i] = (unsigned)((x.R + 7) / 8);
            continue;
        }
        const int64_t ncol = (x.embed == EMB_TRANS || x.embed == EMB_CONJ) ? 2 * x.R : x.R;
        const int64_t nk = x.embed == EMB_NONE ? x.Kd : x.Kd / 2;
        const int64_t wide = (ncol + AMAX_COLS - 1) / AMAX_COLS;
        const bool lines = x.ld % 32 == 0 && (uintptr_t)x.src % 128 == 0;
        const bool slabs = (nk > 8192 && wide < 128) ||
                           (ncol * nk * 4 >= (int64_t)256 << 20 && (x.embed == EMB_NONE || !lines));
        if (!slabs) {
            nb[i] = (unsigned)wide;
            continue;
        }
        hipError_t e = launch_fill_zero(0, x.amax, 1, x.R, x.R, st);   // zero bits = 0.0f
        if (e != hipSuccess) return e;
        const int64_t ncb = (ncol + 1023) / 1024;
        hipLaunchKernelGGL(row_amax_slab_kernel, dim3((unsigned)(ncb * ((nk + 255) / 256))), dim3(256), 0, st, x);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_pair(p, nb[0], nb[1], 512, [&](const AmaxPair &q, unsigned n) {
        if (!a.kmajor) hipLaunchKernelGGL((row_amax_kernel<0, 0>), dim3(n), dim3(512), 0, st, q);
        else if (b.kmajor) hipLaunchKernelGGL((row_amax_kernel<1, 1>), dim3(n), dim3(512), 0, st, q);
        else hipLaunchKernelGGL((row_amax_kernel<1, 0>), dim3(n), dim3(512), 0, st, q);
    });
}

hipError_t launch_fp8_exps(const Fp8ExpArgs &a, int64_t ta, const Fp8ExpArgs &b, int64_t tb, hipStream_t st) {
    ExpPair p{{a, b}, (uint32_t)ta};
    for (Fp8ExpArgs &x : p.x) x.vec = x.ld % 4 == 0 && ((uintptr_t)x.src % 16) == 0;
    if (ta + tb == 0) return hipSuccess;
    hipLaunchKernelGGL(fp8_tile_exp_kernel, dim3((unsigned)(ta + tb)), dim3(512), 0, st, p);
    return hipGetLastError();
}

}  // namespace hs
