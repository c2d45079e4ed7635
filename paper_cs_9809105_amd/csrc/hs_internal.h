// hs_internal.h -- structures shared by the host API and the HIP kernels.
//
// Packed operand layout ("pack").  A product C[M,N] = sum_k X[M,k] Y[k,N]
// sees two operands, each as a matrix of R "rows" (the non-contraction
// dimension) by Kd contraction elements:
//   * the static operand X (R = M) is cut into p row stripes of S_r rows
//     (virtual processor v owns stripe v, Sec. 5.2.2); each stripe into GS
//     groups of MS rows, zero padded; stripe s's groups sit at positions
//     s GS .. s GS + GS - 1;
//   * the travelling operand Y (R = N, one row per output column) is cut into
//     groups of BN rows (the workgroup column tile);
//   * the contraction is cut into p blocks of S_k elements (block kb is the
//     stripe of Y that a virtual processor holds after kb-v shifts), each
//     padded with zeros to nch chunks of KC elements (32 or 64 bytes).
// Packed bytes: [group][piece][kb][chunk][plane][row in group][16 bytes].
// One (group, kb, chunk) is therefore a contiguous run of rows x 32 bytes,
// which is exactly one HBM->LDS fetch of a pipeline stage.
#pragma once
#include <stdint.h>
#include <stddef.h>

namespace hs {

enum Family : int { FAM_F64 = 0, FAM_F32 = 1, FAM_BF16 = 2, FAM_F16 = 3, FAM_FP8 = 4 };

// What the pack kernel converts from/to.
enum PackKind : int {
    PK_F64 = 0,      // f64 -> f64
    PK_F32 = 1,      // f32 -> f32
    PK_B16 = 2,      // 16-bit -> same 16-bit (bf16 or f16 copy)
    PK_SPLIT3 = 3,   // f32 -> three bf16 pieces
    PK_FP8 = 4,      // f32 -> e4m3 q0 (+ q1) with per-tile power-of-two scales
    PK_SPLIT2F16 = 5 // f32 -> two f16 pieces of x 2^e, e per operand row
};

// Two-piece FP16 split: each operand row (non-contraction index) r gets the
// scale 2^e_r, e_r = the largest integer with amax_r 2^e_r < 2^15, found
// from the row's amax (kept as its float bits, which order like unsigned
// integers for amax >= 0): e_r = 15 - frexp_exp(amax_r) (15 for amax 0).
// Complex sources (embed, see PackEmbed) are scanned as their float view
// (ld in floats): EMB_NONE reads the operand itself; EMB_BLOCKS_H (K-major)
// takes row r from float row r / 2 of the Kd floats of a complex row;
// EMB_BLOCKS (MN-major, Kd / 2 rows of R floats) folds float column c into
// rows c & ~1 and c | 1; EMB_TRANS and EMB_CONJ (MN-major, Kd / 2 rows of
// 2R floats) fold float column c into row c / 2.
struct RowAmaxArgs {
    const float *src;
    int64_t ld;
    int kmajor;               // 1: row r is contiguous along the contraction
    int64_t R, Kd;
    uint32_t *amax;           // [R] float bits of max |x| over the row
    int embed;
};

// FP8 scale tiles: 128 x 128 blocks of the logical operand (rows x
// contraction); per tile two int32 exponents {e, e1}: q0 = e4m3(a 2^e) and,
// with refinement, q1 = e4m3((a 2^e - q0) 2^e1).
const int FP8_TILE = 128;

struct Fp8ExpArgs {
    const float *src;
    int64_t ld;
    int kmajor;
    int64_t R, Kd;
    int64_t tiles_k;          // tiles along the contraction
    int refine;
    int32_t *exps;            // [tile_r][tile_k][2]
    int vec;                  // 16-byte loads are legal (set by launch_fp8_exps)
};

// How an operand's rows are cut into groups.  Each kind is a number of lists
// (one; p stripes; K classes) of GS groups; position q of list c is row
// (c + (q / run) step) run + q mod run, while q / run < runs:
//   OPG_TILES    one list of all rows (run past the operand, runs 1)
//   OPG_STRIPES  stripe c: rows c S_r .. of one stripe (run S_r, runs 1)
//   OPG_CLASSES  residue class c mod K: its K~ stripes one after the other
//                (run S_r, runs K~, step K); its last group may be shorter,
//                nothing is padded
// Group gi of list c starts at c list_bytes + gi group_bytes, and its own row
// count is the stride of its planes.
enum OperandGroups : int { OPG_TILES = 0, OPG_STRIPES = 1, OPG_CLASSES = 2 };

struct OperandGeom {
    int64_t R;        // logical rows
    int64_t Kd;       // contraction length
    int striped;      // OperandGroups
    int64_t S_r;      // stripe height (striped) -- ceil(R / p)
    int grp_rows;     // rows per group
    int last_rows;    // rows of a list's last group
    int64_t GS;       // groups per list
    int64_t n_groups; // all groups
    uint32_t run, runs, step;   // the list formula above
    int64_t list_bytes;
    int p;
    int64_t S_k;      // contraction block length -- ceil(Kd / p)
    int64_t nch;      // chunks per block (padded)
    int chunk_bytes;  // 32 (f32, 16-bit) or 64 (fp8, f64)
    int pieces;       // planes written
    int64_t row_bytes;    // one piece of one row: p blocks x nch chunks x chunk_bytes
    int64_t piece_bytes;  // one piece of one group of grp_rows rows
    int64_t group_bytes;  // that group, all pieces
};

// Exact division of any 32-bit n by a constant d >= 1 that the host prepares
// (T. Granlund and P. Montgomery, Division by Invariant Integers using
// Multiplication, 1994): with 2^(l-1) < d <= 2^l, m = floor(2^32 (2^l - d) / d) + 1,
// t = high word of m n, s1 = min(l, 1), n / d = (t + ((n - t) >> s1)) >> (l - s1).
// A pack unit's place takes five such divisions, 5 instructions each against about
// 25 for a division by a kernel argument (the pack kernel of 16384 x 16384 FP32
// read across its rows: plain FP8 395 us to 253, two-piece FP16 502 to 401, refined
// FP8 378 to 297).
struct FastDiv {
    uint32_t d, m, l;
};
constexpr FastDiv fast_div_by(uint32_t d) {
    const uint32_t l = d > 1 ? 32 - (uint32_t)__builtin_clz(d - 1) : 0;
    if ((d & (d - 1)) == 0) return FastDiv{d, 1, l};
    const uint64_t m = (((((uint64_t)1 << l) - d) << 32) / d) + 1;
    return FastDiv{d, (uint32_t)m, l};
}
constexpr uint32_t fast_div(uint32_t n, const FastDiv &v) {
    const uint32_t t = (uint32_t)(((uint64_t)v.m * n) >> 32), s1 = v.l < 1 ? v.l : 1;
    return (t + ((n - t) >> s1)) >> (v.l - s1);
}

// How a source is read: along the contraction, across it element by element,
// or across it in 16-byte runs transposed through LDS.
enum PackMode : int { PACK_K = 0, PACK_MN = 1, PACK_MN_LDS = 2 };

struct PackArgs {
    const void *src;
    int64_t ld;
    OperandGeom g;
    void *dst;
    int64_t total_units;     // < 2^32
    int mode;                // PackMode
    const int32_t *exps;     // fp8: tile exponents (Fp8ExpArgs); two-piece FP16:
                             // the rows' amax bits (RowAmaxArgs), as uint32
    int64_t exp_tiles_k;
    int refine;              // fp8 only: write q1 as the second piece
    int embed;               // complex sources (interleaved re, im; ld in
                             // floats), see PackEmbed
    // divisors of the unit numbering: rows of a group (PACK_K: its 8-row blocks),
    // chunks of a contraction block (PACK_K: its 8-unit runs), blocks, groups of a
    // list, its run
    FastDiv by_rows, by_chunks, by_p, by_GS, by_run;
    uint32_t upr_log;        // log2 of the 16-byte units per chunk row
};

// How the pack kernel reads a complex source (element (kk, row) of the real
// operand; kk the contraction index, row the output row or column).
enum PackEmbed {
    EMB_NONE = 0,      // real source, or complex already laid out as reals
    EMB_BLOCKS = 1,    // MN-major source X[t][j] (t = kk/2, j = row/2): the real
                       // 2 x 2 block embedding [[re x, im x], [-im x, re x]]
    EMB_BLOCKS_H = 2,  // K-major source X[t][j] (t = row/2, j = kk/2): the block
                       // embedding of conj(X[t][j]), i.e. of X^H
    EMB_CONJ = 3,      // MN-major source X[i][t] (i = kk/2, t = row): conj(X)^T
                       // as reals, kk = 2i + (0 re, 1 im)
    EMB_TRANS = 4      // the same read without the conjugation: X^T as reals
};

// One workgroup computes an output tile of G stripe groups -- stripes
// r0, r0 + K, .., r0 + (G-1) K, all of one residue class mod K, sub-group
// msub of each -- by BN columns, and acts as the collector of the back-shift
// (base C = (0, 1, .., 1)): it visits the partials c^{K-1}, .., c^0 in that
// order, computing each on the spot (partial l of stripe s is the work of
// virtual processor s + l: travelling blocks (s + l + jK) mod p, static
// blocks of stripe s) and accumulating it into the same registers.
struct MainArgs {
    const uint8_t *A;        // packed static operand (layout [group][piece][block][chunk]...)
    int64_t a_piece;         // bytes between pieces inside a group
    int64_t a_group;         // bytes between groups
    const uint8_t *B;        // packed travelling operand
    int64_t b_piece;
    int64_t b_group;
    int64_t a_span;          // bytes one workgroup addresses from its first group, < 4 GiB
    const int32_t *a_exps;   // fp8: tile exponents of each operand; two-piece
    const int32_t *b_exps;   // FP16: each operand's row amax bits (uint32)
    int64_t a_tiles_k, b_tiles_k;
    int64_t S_k;             // contraction block length (fp8 scale lookup)
    int64_t Kd;              // contraction length
    void *out;               // the result C
    int64_t ldo;             // row stride of out (elements)
    int p, K, Kt;
    int MS;                  // static-operand rows per group
    int G;                   // stripes per workgroup tile (one residue class)
    int64_t GS;              // groups per stripe
    int64_t nch;             // chunks per contraction block
    int64_t S_r;             // stripe height
    int64_t M, N;
    int64_t n_ntiles;        // column tiles
    // workgroup groups: grp_v class members x grp_t column tiles run together
    int64_t grp_v, grp_t;
    // launches with fewer output tiles than CUs: nsplit workgroups per tile,
    // each over split_stages consecutive stages of the step order, their sums
    // in planes [nsplit][M][N] of part (element type as out), summed after
    int nsplit;
    int split_stages;
    void *part;
};

// The wave-tile kernel (launches that 256 x 256 tiles leave most of the chip
// idle): one workgroup of kg waves per output tile of one group of a residue
// class's rows (OPG_CLASSES) by bn columns; each wave walks its own run of
// the tile's chunks in the step order, and the kg sums are added in LDS.
struct WaveArgs {
    const uint8_t *A;
    const uint8_t *B;
    int64_t a_group, a_class;      // bytes between groups of a class, between classes
    int64_t b_group;
    int a_rows, a_last;            // rows of a group, of a class's last group
    int64_t GS;                    // groups per class
    const int32_t *a_exps;         // as in MainArgs
    const int32_t *b_exps;
    int64_t a_tiles_k, b_tiles_k;
    int64_t S_k, Kd;
    void *out;
    int64_t ldo;
    int p, K, Kt;
    int64_t nch;                   // chunks per contraction block
    int64_t S_r;
    int64_t M, N;
    int64_t n_ntiles;
    int64_t grp_v, grp_t;          // members x column tiles that run together
    int kg;                        // waves per workgroup, a power of two
    int sums64;                    // the sums of up to four are added in FP64 (of eight they always are)
    int nsplit;                    // workgroups per tile (planes of part if > 1)
    int split_chunks;              // chunks each of them walks
    void *part;
};

struct GemvArgs {
    const void *A;
    int64_t lda;
    const void *x;
    void *y;
    int64_t m, n;
    int cplx;                // 1: complex64 A, x, y (lda in complex elements)
    int waves;               // waves per row: 1, 2 or 4
    int lanes;               // lanes per row of one wave: 64, or 16 (waves 1)
};

// All-pairs n-body interaction on the two-array recipe (hs_nbody.hip).
struct NbodyArgs {
    int64_t n;               // bodies
    double eps2;             // softening, >= 0 (rounded to float for FP32)
    int p, K, Kt;            // ring of p virtual processors, K * Kt == p
    int S;                   // bodies per block, ceil(n / p)
    int sub;                 // workgroups along one block: ceil(S / 64)
    int ss;                  // waves per workgroup: runs of the travelling bodies
};

}  // namespace hs
