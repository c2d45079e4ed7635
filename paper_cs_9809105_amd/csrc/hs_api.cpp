// hs_api.cpp -- host side of the C ABI declared in include/hs.h: argument
// validation, the schedule (bases of Sec. 5.2.1), workspace planning and the
// launch sequence pack -> main loop (whose workgroups also collect the
// back-shift) on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>
#include <utility>
#include <vector>

#include "hs.h"
#include "hs_internal.h"

namespace hs {
hipError_t launch_pack(int kind, const PackArgs &a, const PackArgs &b, hipStream_t st);
hipError_t launch_mm(int fam, int form, const MainArgs &a, hipStream_t st);
hipError_t launch_wave(int fam, int form, int tr, int tc, const WaveArgs &a, hipStream_t st);
int wave_chunk_bytes(int fam);
int wave_tile(int fam, int t);
hipError_t launch_backshift(int f64, const void *W, int64_t plane, int K, int64_t M, int64_t N,
                            void *Cout, int64_t ldc, hipStream_t st);
hipError_t launch_fill_zero(int f64, void *Cout, int64_t M, int64_t N, int64_t ldc, hipStream_t st);
hipError_t launch_gemv(int f64, const GemvArgs &a, hipStream_t st);
hipError_t launch_fp8_exps(const Fp8ExpArgs &a, int64_t ta, const Fp8ExpArgs &b, int64_t tb, hipStream_t st);
hipError_t launch_row_amax(const RowAmaxArgs &a, const RowAmaxArgs &b, hipStream_t st);
void set_timed_launch(hipEvent_t start, hipEvent_t stop);
bool timed_launch_done();
hipError_t launch_nbody(int f64, const void *bodies, void *out, const NbodyArgs &a, hipStream_t st);
int mm_tile_rows(int fam);
int mm_tile_cols(int fam);
int mm_chunks_per_stage(int fam, int form);
}  // namespace hs

using namespace hs;

namespace {

const int kMaxP = 4096;
const size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct FormInfo {
    int fam, form, pack, in_esz, out_f64, packed_esz;
};

bool form_info(int dt, FormInfo *f) {
    switch (dt) {
        case HS_F64: *f = {FAM_F64, 0, PK_F64, 8, 1, 8}; return true;
        case HS_F32: *f = {FAM_F32, 0, PK_F32, 4, 0, 4}; return true;
        case HS_BF16: *f = {FAM_BF16, 0, PK_B16, 2, 0, 2}; return true;
        case HS_F16: *f = {FAM_F16, 0, PK_B16, 2, 0, 2}; return true;
        case HS_SPLIT3_BF16: *f = {FAM_BF16, 1, PK_SPLIT3, 4, 0, 2}; return true;
        case HS_FP8_E4M3: *f = {FAM_FP8, 0, PK_FP8, 4, 0, 1}; return true;
        case HS_FP8_E4M3_R1: *f = {FAM_FP8, 1, PK_FP8, 4, 0, 1}; return true;
        case HS_SPLIT2_F16: *f = {FAM_F16, 2, PK_SPLIT2F16, 4, 0, 2}; return true;
        default: return false;
    }
}

// The complex dtypes run as one real product of their base form.
bool complex_base(int dt, hs_dtype *base) {
    if (dt == HS_C32) { *base = HS_F32; return true; }
    if (dt == HS_C32_SPLIT3_BF16) { *base = HS_SPLIT3_BF16; return true; }
    if (dt == HS_C32_SPLIT2_F16) { *base = HS_SPLIT2_F16; return true; }
    return false;
}

// Default K: the divisor of p minimising the shift count K + p/K - 1
// (Thm. on minimal length, Sec. 4.4); ties go to the smaller K.
int default_K(int p) {
    int best = 1, cost = std::numeric_limits<int>::max();
    for (int K = 1; K <= p; ++K)
        if (p % K == 0 && K + p / K - 1 < cost) { cost = K + p / K - 1; best = K; }
    return best;
}

struct Plan {
    FormInfo f;
    int p, K, Kt;
    int64_t M, N, Kd;
    OperandGeom ga, gb;
    size_t off_a, off_b, total;
    int G;                            // stripes per workgroup tile (one residue class)
    int64_t a_span;                   // bytes of a workgroup's static-operand region
    size_t off_ea, off_eb;            // fp8: tile exponents of each operand
    int64_t tiles_k, tiles_ra, tiles_rb;
    int nsplit, split_stages;         // workgroups per output tile, stages each
    size_t off_part;                  // their partial planes (nsplit > 1)
    int tr, tc;                       // MFMA tiles down and across the wave kernel's tile; 0: mm_kernel
    int kg;                           // its waves per workgroup
    bool sums64;                      // their sums are added in FP64
};

// Compute units of the MI355X: a launch with fewer output tiles than this
// leaves CUs idle unless each tile's stage sequence is split.
const int64_t kCUs = 256;

// Bytes of a packed operand.
int64_t operand_bytes(const OperandGeom &g) { return g.n_groups / g.GS * g.list_bytes; }

// The group geometry that follows from striped, S_r, grp_rows, GS and the
// contraction: `lists` lists of `rows` rows each.
void finish_geom(OperandGeom *g, int p, int K, int64_t lists, int64_t rows) {
    g->n_groups = lists * g->GS;
    g->row_bytes = (int64_t)p * g->nch * g->chunk_bytes;
    g->piece_bytes = g->grp_rows * g->row_bytes;
    g->group_bytes = g->pieces * g->piece_bytes;
    g->last_rows = g->grp_rows;
    g->list_bytes = g->GS * g->group_bytes;
    g->run = g->striped == OPG_TILES ? 0x7fffffffu : (uint32_t)g->S_r;
    g->runs = 1;
    g->step = 0;
    if (g->striped == OPG_CLASSES) {
        g->last_rows = (int)(rows - (g->GS - 1) * g->grp_rows);
        g->list_bytes = rows * g->pieces * g->row_bytes;
        g->runs = (uint32_t)(p / K);
        g->step = (uint32_t)K;
    }
}

// Threads of the pack kernel: one per 16-byte unit; a K-major source is
// walked in 8 x 8 (row, unit) blocks, so both counts round up to 8.
int64_t pack_units(const OperandGeom &g, int kmajor) {
    const int64_t nu = g.nch * (g.chunk_bytes / 16);
    if (kmajor) return g.n_groups * g.p * ((nu + 7) / 8 * 8) * ((g.grp_rows + 7) / 8 * 8);
    return g.n_groups * g.p * nu * g.grp_rows;
}

// Workspace layout: the two packed operands (no partial planes: the collector
// keeps every partial in registers), the FP8 tile exponents or the two-piece
// FP16 row amaxes, and the split planes.
void layout_workspace(Plan *P) {
    size_t off = 0;
    P->off_a = off; off = align_up(off + (size_t)operand_bytes(P->ga));
    P->off_b = off; off = align_up(off + (size_t)operand_bytes(P->gb));
    P->tiles_k = ceil_div(P->Kd, FP8_TILE);
    P->tiles_ra = ceil_div(P->M, FP8_TILE);
    P->tiles_rb = ceil_div(P->N, FP8_TILE);
    P->off_ea = P->off_eb = off;
    if (P->f.fam == FAM_FP8) {
        P->off_ea = off; off = align_up(off + (size_t)P->tiles_ra * P->tiles_k * 2 * sizeof(int32_t));
        P->off_eb = off; off = align_up(off + (size_t)P->tiles_rb * P->tiles_k * 2 * sizeof(int32_t));
    }
    if (P->f.pack == PK_SPLIT2F16) {
        P->off_ea = off; off = align_up(off + (size_t)P->M * sizeof(uint32_t));
        P->off_eb = off; off = align_up(off + (size_t)P->N * sizeof(uint32_t));
    }
    P->off_part = off;
    if (P->nsplit > 1) off = align_up(off + (size_t)P->nsplit * P->M * P->N * (P->f.out_f64 ? 8 : 4));
    P->total = (P->M == 0 || P->N == 0 || P->Kd == 0) ? 0 : off;
}

// Whether the wave kernel takes the product that *P plans for mm_kernel, and
// with which tile.  mm_kernel needs its 256 x 256 tiles to fill the chip: a
// launch of `tiles` of them keeps u = tiles / (256 rounds) of the CUs busy.
// The wave kernel's small tiles fill it sooner, but every wave reads its own
// fragments; below u = r it is the faster one.  Whole calls, n x n x k, us
// (wave / mm): u = 0.39 (n = 2560, k = 1024): BF16 36 / 43, two-piece FP16
// 75 / 88, split-BF16 93 / 120, FP8 34 / 43, refined FP8 46 / 57; u = 0.56
// (n = 3072, k = 1024): 44 / 40, 95 / 90, 125 / 116, 39 / 38, 61 / 54, so r is
// one half; for FP32, whose fragments are cheap, u = 0.77 (n = 3584): 837 / 955
// at k = 4096, u = 0.88 (n = 3840): 956 / 961, and 277 / 254 at k = 1024.
// Far left of the line: 1024^3 FP32 35 / 240, split-BF16 30 / 105.  FP64
// always takes it (an LDS-tiled 64 x 64 kernel measured 3075 us at 4096^3
// against 1852, 400 against 259 at 2048^3, 18.6 against 5.8 at 256^3).
// 4 x 2 tiles (wave_shape: only where they fill the chip) move the line, split-BF16
// and two-piece FP16: u = 1/2 (2048^3) 102 / 122 and 84 / 96, 1792 x 1792 x 2500 108 /
// 140 and 91 / 107, split-BF16 u = 0.47 (2816 x 2816 x 1900) 159 / 191; u = 1 (4096 x
// 2048 x 2048) 157 / 142 and 110 / 91, so r is 0.97.
int wave_percent(const FormInfo &f, int tr) {
    return f.fam == FAM_F64 ? 101 : f.fam == FAM_F32 ? 88 : tr == 4 ? 97 : 50;
}

// MFMA tiles down and across the wave kernel's tile, and waves per workgroup;
// n(tr, tc) counts the output tiles; wide: columns padded to 96 take no more
// workspace than to 256.  Times in us, n x n x k products.
//
// A wave of the FP32 and FP64 forms spends 64 cycles on the MFMA of two cheap
// fragments: small tiles, 4 waves (FP32 2048^3: 139 with 4 waves, 193 with 2,
// 250 with 1, since workgroups of one or two waves share SIMDs while others
// idle), one wave from 8192 tiles on (FP64 3000 x 3000 x 256, 8836 tiles: 88, 105
// with 4; FP32 3000 x 2816 x 1000, 8272: 159, 160; but 2720 x 2880 x 1000, 7650: 195,
// 159).  Of these 2 x 2 tiles two workgroups fit a CU (LDS): taken from 900 tiles,
// and for FP32, where they gain little (2048^3, 1024 tiles: 134 against 140) only if
// 512 at a time fill nine tenths of the rounds (1800 x 2200 x 1000, 1050 tiles: 91 against 72).  FP64 takes them
// where they fill the rounds, or there are 64 with long sums, and little of them
// is padding: whole calls (2 x 2 / 1 x 1, and the LDS-tiled kernel), 1008 x 448 x
// 15616, 448 tiles, 316 / 550, 433; 64 x 8192 x 8192, 512, 406 / 538, 411; 512^3, 256,
// 15.2 / 16.2; 100 x 1000 x 10000, 128, 88 / 93; but 405 x 658 x 1074, 273, 31.3 / 28.8;
// 256^3, 64 short ones, 9.9 / 8.0; 33 x 5000 x 5000, a third of it padding, 163 / 159.
//
// The 16-bit and FP8 forms are bound by fragment reads, which larger tiles
// save: 2 x 2 from 256 tiles (1024^3: split-BF16 19 against 22, FP8 8.9 against
// 9.1; below, 256 x 512 x 2048, 64 tiles, refined FP8 8.6 against 6.9) with only
// as many waves as fill the SIMDs (BF16 2500^3, 1600 tiles: 53 with one wave,
// 64 with 4; 1500^3, 576: 25, 22 with 2, 24; the split forms with their longer
// chunks take 4 until 1024: split-BF16 1500^3 54 against 66 with 2).  1 x 1 tiles
// have 4 waves, 2 from 768 on (BF16 896 x 896 x 2048, 784: 23.2, 24.9 with 4; 640 x
// 640 x 2048, 400: 19.3, 18.0; between, where 2 can be the faster, 4 sum more exactly).
// Just past 256 tiles of 2 x 2 a few CUs would run two rounds: where 3 x 2 ones
// are at most 256, the 16-bit forms take these with 8 waves (1100 x 900 x 1000,
// 270 tiles against 180: split-BF16 28.4 to 23.0, two-piece FP16 20.4 to 17.4,
// BF16 13.9 to 12.8; 800 x 1100 x 3000: 62 to 43, 43 to 31, 24 to 19; FP8 gains
// nothing, 11.3 and 11.4, nor do fewer than 8 chunks); or 2 x 3 ones likewise
// (1000 x 1400 x 1400: split-BF16 35 to 29, two-piece FP16 25.4 to 21.6, BF16 16.3 to 14.6).  4 x 2 tiles need all
// registers of a SIMD for one wave; for the split forms they win where such
// waves are on nearly every SIMD, 512 tiles of two waves or 1024 of one (2 x 2
// tiles here, split-BF16 2048^3: 124 to 102, 2500 x 2500 x 1500, 800 tiles: 151 to 118;
// but 1800 x 2200 x 1000, 560: 64, 73 here), from 64 chunks (split-BF16 2048 x 2048 x
// 512: 32, 35 here) or 128 (two-piece FP16 2560 x 2560 x 1024: 60, 65 here).
//
// parts: the workgroups that mm_kernel would split a tile's step order over.  An
// FP32 sum's rounding error grows with the length of its chain, so a tile has at
// least as many waves, and 4 x 2 tiles are for products that need no more than
// their one or two: with twice the waves they lose to mm_kernel (split-BF16 2500 x
// 2500 x 2500, two parts: 215 against 177; 2048 x 1500 x 6000, four: 252 against 213;
// with one wave or two 188 and 233, at 1.4 times the error).
template <class Count>
void wave_shape(const FormInfo &f, Count n, bool wide, int64_t chunks, int parts, int *tr, int *tc, int *kg) {
    const bool slow = f.fam == FAM_F64 || f.fam == FAM_F32, b16 = f.fam == FAM_BF16 || f.fam == FAM_F16;
    const bool split = b16 && f.form != 0;
    auto fills = [](int64_t tiles, int64_t slots, int percent) {
        return tiles * 100 >= ceil_div(tiles, slots) * slots * percent;
    };
    const int64_t n22 = n(2, 2), n42 = n(4, 2);
    *tr = *tc = 1;
    if (slow) {
        const bool wide64 = (n22 >= 256 ? fills(n22, 256, 75) : n22 >= 64 && chunks >= 512) && 16 * n22 <= 5 * n(1, 1);
        if (f.fam == FAM_F64 ? n22 >= 900 || wide64 : n22 >= 900 && fills(n22, 512, 90)) *tr = *tc = 2;
        *kg = n(*tr, *tc) >= 8192 ? 1 : 4;
    } else if (split && chunks >= (f.form == 1 ? 64 : 128) && n42 > 256 && n42 <= 1024 &&
               fills(n42, n42 <= 512 ? 512 : 1024, 75) && parts <= (n42 <= 512 ? 2 : 1)) {
        *tr = 4;
        *tc = 2;
        *kg = n42 <= 512 ? 2 : 1;
    } else if (b16 && n22 > kCUs && n(3, 2) <= kCUs && chunks >= 8) {
        *tr = 3;
        *tc = 2;
        *kg = 8;
    } else if (b16 && n22 > kCUs && wide && n(2, 3) <= kCUs && chunks >= 8) {
        *tr = 2;
        *tc = 3;
        *kg = 8;
    } else if (n22 >= 256) {
        *tr = *tc = 2;
        *kg = n22 >= 1024 ? 1 : n22 >= 512 && !split ? 2 : 4;
    } else {
        *kg = n(1, 1) >= 768 ? 2 : 4;
    }
    // long sums on few tiles: 300 x 320 x 6000 BF16 13 against 15
    if (*tr == 1 && n(1, 1) <= 128 && chunks >= 256) *kg = 8;
    while (*kg > 1 && chunks < 2 * *kg) *kg /= 2;
    while (*kg < parts) *kg *= 2;
}

// Replans *P for the wave kernel where that is the faster one.  The packed
// operands never take more workspace than mm_kernel's plan (rows of a class
// are not padded, columns and chunks to smaller units) and neither do the
// planes, so a call that fits a given workspace still does.
void plan_wave(Plan *P) {
    if (P->M == 0 || P->N == 0 || P->Kd == 0) return;
    const int fam = P->f.fam;
    const int64_t tiles = (int64_t)P->K * ceil_div(P->Kt, P->G) * P->ga.GS * P->gb.GS * P->nsplit;
    Plan W = *P;
    const int64_t L = (int64_t)P->Kt * P->ga.S_r;         // rows of a residue class
    const int CBY = wave_chunk_bytes(fam);
    const int64_t nch = ceil_div(P->ga.S_k, CBY / P->f.packed_esz), chunks = P->p * nch;
    auto count = [&](int tr, int tc) {
        return (int64_t)P->K * ceil_div(L, wave_tile(fam, tr)) * ceil_div(P->N, wave_tile(fam, tc));
    };
    const bool wide = ceil_div(P->N, 96) * 96 <= P->gb.GS * P->gb.grp_rows;
    wave_shape(P->f, count, wide, chunks, P->nsplit, &W.tr, &W.tc, &W.kg);
    if (tiles * 100 >= ceil_div(tiles, kCUs) * kCUs * wave_percent(P->f, W.tr)) return;
    const int64_t wt = count(W.tr, W.tc);
    if (wt >= (int64_t)1 << 26) return;                   // 32-bit grid in threads
    const int R = wave_tile(fam, W.tr), C = wave_tile(fam, W.tc);
    OperandGeom &a = W.ga, &b = W.gb;
    a.striped = OPG_CLASSES;
    a.grp_rows = (int)std::min<int64_t>(R, L);
    a.GS = ceil_div(L, a.grp_rows);
    b.grp_rows = C; b.GS = ceil_div(P->N, C);
    a.nch = b.nch = nch;
    a.chunk_bytes = b.chunk_bytes = CBY;
    finish_geom(&a, P->p, P->K, P->K, L);
    finish_geom(&b, P->p, P->K, 1, P->N);
    const int64_t kMaxUnits = ((int64_t)1 << 32) - 512;   // 32-bit unit numbers
    if (pack_units(a, 1) > kMaxUnits || pack_units(b, 1) > kMaxUnits) return;
    int64_t ns = std::min<int64_t>({(int64_t)P->nsplit, kCUs / wt, chunks / (16 * W.kg)});
    if (ns < 2) ns = 1;
    W.sums64 = P->nsplit > 1 && W.kg > 2;                 // they stand for its planes; two round alike in FP32
    W.split_stages = (int)ceil_div(chunks, ns);
    W.nsplit = (int)ceil_div(chunks, W.split_stages);
    layout_workspace(&W);
    *P = W;
}

// Geometry of one product C[M,N] = X[M,Kd] Y[Kd,N] under schedule (p, K).
hs_status make_plan(int64_t M, int64_t N, int64_t Kd, int dt, hs_schedule s, Plan *P) {
    if (!form_info(dt, &P->f)) return HS_ERR_NOT_SUPPORTED;
    hs_schedule r;
    hs_status st = hs_schedule_resolve(s, &r);
    if (st != HS_OK) return st;
    if (M < 0 || N < 0 || Kd < 0) return HS_ERR_INVALID_VALUE;
    // every dimension below 2^31 keeps the products of two of them, and so
    // every count and byte size below, inside 64 bits
    const int64_t kMaxDim = std::numeric_limits<int32_t>::max();
    if (M > kMaxDim || N > kMaxDim || Kd > kMaxDim) return HS_ERR_NOT_SUPPORTED;
    P->p = r.p; P->K = r.K; P->Kt = r.p / r.K;
    P->M = M; P->N = N; P->Kd = Kd;
    const int BMT = mm_tile_rows(P->f.fam), BNT = mm_tile_cols(P->f.fam);
    const int CPS = mm_chunks_per_stage(P->f.fam, P->f.form);
    const int p = P->p;
    const bool fp8 = P->f.fam == FAM_FP8;
    const int CBY = fp8 ? 64 : 32;                  // chunk bytes
    const int KC = CBY / P->f.packed_esz;
    const int64_t S_r = std::max<int64_t>(1, ceil_div(M, p));
    const int64_t S_k = std::max<int64_t>(1, ceil_div(Kd, p));
    const int64_t nch = ceil_div(ceil_div(S_k, KC), CPS) * CPS;
    // a workgroup tile stacks G stripe groups of MS rows, all stripes of one
    // residue class mod K (they share every travelling block)
    const int MS = (int)std::min<int64_t>(BMT, S_r);
    P->G = (int)std::max<int64_t>(1, std::min<int64_t>(P->Kt, BMT / MS));
    const int NP = fp8 ? (P->f.form == 1 ? 2 : 1) : (P->f.form == 1 ? 3 : P->f.form == 2 ? 2 : 1);
    if (fp8) {
        // every 32-row / 32-column MFMA tile and every 64-deep chunk must lie
        // inside one 128 x 128 scale tile: whole 64-chunks per block, 32-row
        // aligned stripes and groups
        if (S_k % 64 != 0 || S_r % 32 != 0 || MS % 32 != 0) return HS_ERR_NOT_SUPPORTED;
    }

    OperandGeom &a = P->ga;
    a.R = M; a.Kd = Kd; a.striped = OPG_STRIPES; a.S_r = S_r; a.grp_rows = MS;
    a.GS = ceil_div(S_r, MS); a.p = p;
    a.S_k = S_k; a.nch = nch; a.chunk_bytes = CBY; a.pieces = NP;
    finish_geom(&a, p, P->K, p, S_r);

    OperandGeom &b = P->gb;
    b.R = N; b.Kd = Kd; b.striped = OPG_TILES; b.S_r = 0; b.grp_rows = BNT;
    b.GS = std::max<int64_t>(1, ceil_div(N, BNT)); b.p = p;
    b.S_k = S_k; b.nch = nch; b.chunk_bytes = CBY; b.pieces = NP;
    finish_geom(&b, p, P->K, 1, N);

    // grid (with padding to whole workgroup groups) must fit in 32 bits
    const int64_t nwg = (int64_t)p * a.GS * b.GS * 2 + 64;
    if (nwg > std::numeric_limits<int32_t>::max()) return HS_ERR_NOT_SUPPORTED;
    // a workgroup addresses its region of each packed operand with 32-bit
    // offsets: G groups K GS groups apart of the static operand (fewer
    // stripes per tile where that region would pass 4 GiB), one group of
    // the travelling
    const int64_t kMaxPacked = (int64_t)0xFFFFFFF0;
    auto span = [&](int G) { return ((int64_t)(G - 1) * P->K * a.GS + 1) * a.group_bytes; };
    while (P->G > 1 && span(P->G) > kMaxPacked) --P->G;
    P->a_span = span(P->G);
    if (P->a_span > kMaxPacked || b.group_bytes > kMaxPacked) return HS_ERR_NOT_SUPPORTED;
    // 32-bit indexing of the pack kernel and of the stage counter
    if (pack_units(a, 1) >= (int64_t)1 << 31 || pack_units(b, 1) >= (int64_t)1 << 31) return HS_ERR_NOT_SUPPORTED;
    if ((int64_t)p * nch >= (int64_t)1 << 31) return HS_ERR_NOT_SUPPORTED;

    // Output tiles under the CU count: split each tile's step order over
    // nsplit workgroups (at most 4, at least 64 stages each, the plain 16-bit and
    // FP8 forms' short ones counted in pairs), whose sums a fixed-order FP64 pass
    // adds (the planes below)
    {
        const int64_t spb = nch / CPS, nstages = (int64_t)p * spb;
        const int64_t tiles = (int64_t)P->K * ceil_div(P->Kt, P->G) * a.GS * b.GS;
        const int64_t pair = P->f.form == 0 && (fp8 || P->f.packed_esz == 2) ? 2 : 1;
        int64_t ns = 1;
        if (tiles > 0 && tiles < kCUs) ns = std::min<int64_t>({4, kCUs / tiles, p * ceil_div(spb, pair) / 64});
        if (ns < 2) ns = 1;
        P->split_stages = (int)ceil_div(nstages, ns);
        P->nsplit = (int)ceil_div(nstages, P->split_stages);
    }

    P->tr = P->tc = 0;
    P->kg = 0;
    P->sums64 = false;
    layout_workspace(P);
    plan_wave(P);
    if (P->f.fam == FAM_F64 && P->tr == 0 && P->total > 0) return HS_ERR_NOT_SUPPORTED;   // no other FP64 kernel
    return HS_OK;
}

bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

// ---------------------------------------------------------------------------
// kernel timing (hs_profile_begin / hs_profile_end)
// ---------------------------------------------------------------------------
bool g_prof = false;
std::vector<std::pair<hipEvent_t, hipEvent_t>> g_events;

// Two new events handed to the next timed launch, which records them itself.
bool timing_events(hipEvent_t *ev0, hipEvent_t *ev1) {
    if (hipEventCreate(ev0) != hipSuccess) return false;
    if (hipEventCreate(ev1) != hipSuccess) {
        (void)hipEventDestroy(*ev0);
        return false;
    }
    set_timed_launch(*ev0, *ev1);
    return true;
}

// After the launch call: keep the pair if a kernel took it (an empty
// problem launches nothing), else release it.
void keep_timing(hipEvent_t ev0, hipEvent_t ev1) {
    if (timed_launch_done()) {
        g_events.push_back({ev0, ev1});
    } else {
        (void)hipEventDestroy(ev0);
        (void)hipEventDestroy(ev1);
    }
}

struct Operand {
    const void *ptr;
    int64_t ld;
    int kmajor;   // 1: contraction index contiguous
    int embed;    // how a complex source is read (PackEmbed)
};

hs_status launch_status(hipError_t e) { return e == hipSuccess ? HS_OK : HS_ERR_LAUNCH_FAILED; }

// How an operand's source is read.  An MN-major one goes through LDS (16-byte
// runs of 4 FP32 or 8 16-bit rows) when its rows are 16-byte aligned and every
// run of a group lies in one stripe.
int pack_mode(const Plan &P, const Operand &X, const OperandGeom &g) {
    if (X.kmajor) return PACK_K;
    if (X.embed != EMB_NONE || P.f.pack == PK_F64) return PACK_MN;
    const int rw = 16 / P.f.in_esz;
    return X.ld % rw == 0 && aligned(X.ptr, 16) && g.grp_rows % rw == 0 && (g.striped == OPG_TILES || g.S_r % rw == 0)
               ? PACK_MN_LDS : PACK_MN;
}

PackArgs pack_args(const Plan &P, const Operand &X, const OperandGeom &g, void *dst, const int32_t *exps) {
    PackArgs a{};
    a.src = X.ptr; a.ld = X.ld; a.g = g; a.dst = dst;
    a.total_units = pack_units(g, X.kmajor);
    a.mode = pack_mode(P, X, g);
    a.exps = exps; a.exp_tiles_k = P.tiles_k; a.refine = P.f.form;
    a.embed = X.embed;
    const uint32_t upr = (uint32_t)(g.chunk_bytes / 16), units = (uint32_t)g.nch * upr;
    const bool blocks = a.mode == PACK_K;
    a.by_rows = fast_div_by(blocks ? (uint32_t)(g.grp_rows + 7) / 8 : (uint32_t)g.grp_rows);
    a.by_chunks = fast_div_by(blocks ? (units + 7) / 8 : (uint32_t)g.nch);
    a.by_p = fast_div_by((uint32_t)g.p);
    a.by_GS = fast_div_by((uint32_t)g.GS);
    a.by_run = fast_div_by(g.run);
    a.upr_log = upr == 4 ? 2 : 1;
    return a;
}

// 32 workgroups per XCD batch: grp_v class members x grp_t column tiles.
void batch_shape(int64_t nt, int64_t members, int64_t *grp_v, int64_t *grp_t) {
    int64_t gt = 1;
    while (gt * 2 <= 8 && gt * 2 <= nt) gt *= 2;
    int64_t gv = 32 / gt;
    while (gv > 1 && gv / 2 >= members) gv /= 2;
    *grp_t = gt; *grp_v = gv;
}

// One product through the hyper-systolic path.  The plan must come from
// make_plan with the same sizes; ws holds at least plan.total bytes.
hs_status run_product(const Plan &P, const Operand &X, const Operand &Y, void *out, int64_t ldo,
                      void *ws, hipStream_t stream) {
    const int f64 = P.f.out_f64;
    if (P.M == 0 || P.N == 0) return HS_OK;
    if (P.Kd == 0) return launch_status(launch_fill_zero(f64, out, P.M, P.N, ldo, stream));
    uint8_t *w = (uint8_t *)ws;
    const bool fp8 = P.f.fam == FAM_FP8;
    int32_t *ea = (int32_t *)(w + P.off_ea), *eb = (int32_t *)(w + P.off_eb);
    if (fp8) {   // per-tile exponents of both operands (operand preparation)
        Fp8ExpArgs xa{(const float *)X.ptr, X.ld, X.kmajor, P.M, P.Kd, P.tiles_k, P.f.form, ea};
        Fp8ExpArgs xb{(const float *)Y.ptr, Y.ld, Y.kmajor, P.N, P.Kd, P.tiles_k, P.f.form, eb};
        if (launch_fp8_exps(xa, P.tiles_ra * P.tiles_k, xb, P.tiles_rb * P.tiles_k, stream) != hipSuccess)
            return HS_ERR_LAUNCH_FAILED;
    }
    if (P.f.pack == PK_SPLIT2F16) {   // row amaxes of both operands (their scales)
        RowAmaxArgs xa{(const float *)X.ptr, X.ld, X.kmajor, P.M, P.Kd, (uint32_t *)ea, X.embed};
        RowAmaxArgs xb{(const float *)Y.ptr, Y.ld, Y.kmajor, P.N, P.Kd, (uint32_t *)eb, Y.embed};
        if (launch_row_amax(xa, xb, stream) != hipSuccess) return HS_ERR_LAUNCH_FAILED;
    }

    hipError_t e = launch_pack(P.f.pack, pack_args(P, X, P.ga, w + P.off_a, ea),
                               pack_args(P, Y, P.gb, w + P.off_b, eb), stream);
    if (e != hipSuccess) return HS_ERR_LAUNCH_FAILED;

    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (P.tr) {
        WaveArgs v{};
        v.A = w + P.off_a; v.a_group = P.ga.group_bytes; v.a_class = P.ga.list_bytes;
        v.B = w + P.off_b; v.b_group = P.gb.group_bytes;
        v.a_rows = P.ga.grp_rows; v.a_last = P.ga.last_rows; v.GS = P.ga.GS;
        v.a_exps = ea; v.b_exps = eb; v.a_tiles_k = P.tiles_k; v.b_tiles_k = P.tiles_k;
        v.S_k = P.ga.S_k; v.Kd = P.Kd;
        v.out = out; v.ldo = ldo;
        v.p = P.p; v.K = P.K; v.Kt = P.Kt; v.nch = P.ga.nch; v.S_r = P.ga.S_r;
        v.M = P.M; v.N = P.N; v.n_ntiles = P.gb.GS;
        batch_shape(P.gb.GS, P.ga.GS, &v.grp_v, &v.grp_t);
        v.kg = P.kg; v.sums64 = P.sums64; v.nsplit = P.nsplit; v.split_chunks = P.split_stages; v.part = w + P.off_part;
        if (g_prof && !timing_events(&ev0, &ev1)) return HS_ERR_LAUNCH_FAILED;
        e = launch_wave(P.f.fam, P.f.form, P.tr, P.tc, v, stream);
        if (g_prof) keep_timing(ev0, ev1);
        if (e == hipSuccess && P.nsplit > 1)
            e = launch_backshift(f64, v.part, P.M * P.N, P.nsplit, P.M, P.N, out, ldo, stream);
        return launch_status(e);
    }
    MainArgs m{};
    m.A = w + P.off_a; m.a_piece = P.ga.piece_bytes; m.a_group = P.ga.group_bytes;
    m.B = w + P.off_b; m.b_piece = P.gb.piece_bytes; m.b_group = P.gb.group_bytes;
    m.a_span = P.a_span;
    m.p = P.p; m.K = P.K; m.Kt = P.Kt;
    m.MS = P.ga.grp_rows; m.G = P.G; m.GS = P.ga.GS; m.nch = P.ga.nch; m.S_r = P.ga.S_r;
    m.M = P.M; m.N = P.N;
    m.a_exps = ea; m.b_exps = eb; m.a_tiles_k = P.tiles_k; m.b_tiles_k = P.tiles_k;
    m.S_k = P.ga.S_k; m.Kd = P.Kd;
    m.out = out;
    m.ldo = ldo;
    m.n_ntiles = P.gb.GS;
    m.nsplit = P.nsplit;
    m.split_stages = P.split_stages;
    m.part = w + P.off_part;
    batch_shape(P.gb.GS, ceil_div(P.Kt, P.G) * P.ga.GS, &m.grp_v, &m.grp_t);
    if (g_prof && !timing_events(&ev0, &ev1)) return HS_ERR_LAUNCH_FAILED;
    e = launch_mm(P.f.fam, P.f.form, m, stream);
    if (g_prof) keep_timing(ev0, ev1);
    if (e == hipSuccess && P.nsplit > 1)   // C = the planes' sum, fixed order, FP64
        e = launch_backshift(f64, m.part, P.M * P.N, P.nsplit, P.M, P.N, out, ldo, stream);
    return launch_status(e);
}

hs_status check_mat(const void *p, int64_t rows, int64_t cols, int64_t ld, size_t esz) {
    if (rows < 0 || cols < 0) return HS_ERR_INVALID_VALUE;
    if (ld < std::max<int64_t>(1, cols)) return HS_ERR_INVALID_VALUE;
    if (rows > 0 && cols > 0) {
        if (!p) return HS_ERR_INVALID_VALUE;
        if (!aligned(p, esz)) return HS_ERR_INVALID_VALUE;
    }
    return HS_OK;
}

hs_status check_ws(const Plan &P, const void *ws, size_t ws_bytes) {
    if (P.total == 0) return HS_OK;
    if (!ws) return HS_ERR_WORKSPACE_TOO_SMALL;
    if (!aligned(ws, kAlign)) return HS_ERR_INVALID_VALUE;
    if (ws_bytes < P.total) return HS_ERR_WORKSPACE_TOO_SMALL;
    return HS_OK;
}

#define HS_TRY(x)                          \
    do {                                   \
        hs_status _s = (x);                \
        if (_s != HS_OK) return _s;        \
    } while (0)

}  // namespace

// The n-body call's launch shape and workspace.  A workgroup's ss waves split
// the travelling bodies: 8 (n = 262144, p = 64, K = 8: 18.1 ms; 18.7 with 16; n =
// 16384 88 us, 90), or 16 where there are fewer than 1024 workgroups (n = 10000,
// p = 8, K = 1, 160 workgroups: 67 us; 82 with 8; n = 3000, p = 16, K = 4, 192: 13.2,
// 13.7), and fewer where a wave would get under 16 bodies (n = 2000, p = K = 16: 13.0
// with 4, 14.2 with 16).  From 2048 workgroups on a wave gets 96 at least: there
// the chip is full, and many replicas leave few travelling bodies to split (n =
// 61253, p = K = 256: 1197 us with 2, 1613 with 8; n = 16384, p = K = 64: 108, 128;
// n = 8000, p = K = 32: 39.6, 43.0).
hs_status nbody_plan(int64_t n, int dtype, hs_schedule s, double eps2, NbodyArgs *a, size_t *ws) {
    if (dtype != HS_F32 && dtype != HS_F64) return HS_ERR_NOT_SUPPORTED;
    hs_schedule r;
    HS_TRY(hs_schedule_resolve(s, &r));
    if (n < 0 || !std::isfinite(eps2) || eps2 < 0.0) return HS_ERR_INVALID_VALUE;
    if (dtype == HS_F32 && eps2 > (double)std::numeric_limits<float>::max()) return HS_ERR_INVALID_VALUE;
    if (n >= ((int64_t)1 << 31)) return HS_ERR_NOT_SUPPORTED;     // 32-bit positions in a block
    const int f64 = dtype == HS_F64;
    *a = NbodyArgs{};
    a->n = n;
    a->eps2 = eps2;
    a->p = r.p;
    a->K = r.K;
    a->Kt = r.p / r.K;
    a->S = (int)std::max<int64_t>(1, ceil_div(n, r.p));
    // The size limit of a call: 2^31 - 1 slices of 256 positions by replicas, a pair
    // of replicas counted once (n = 2^28, p = K = 4096: half a day of pairs).
    if ((int64_t)r.p * ceil_div(a->S, 256) * (r.K % 2 ? r.K : r.K / 2) > std::numeric_limits<int32_t>::max())
        return HS_ERR_NOT_SUPPORTED;
    a->sub = (int)ceil_div(a->S, 64);
    const int64_t gx = (int64_t)a->sub * r.K;         // times 64: at most n + 64 K, below 2^32 threads
    a->ss = gx * r.p < 1024 ? 16 : 8;
    const int least = gx * r.p < 2048 ? 16 : 96;
    while (a->ss > 1 && ((int64_t)a->Kt * a->S < least * a->ss || gx * 64 * a->ss >> 32)) a->ss /= 2;
    const size_t esz = f64 ? 8 : 4;
    *ws = r.K > 1 ? align_up((size_t)r.K * (size_t)n * 4 * esz) : 0;
    return HS_OK;
}

extern "C" {

const char *hs_status_string(int status) {
    switch (status) {
        case HS_OK: return "HS_OK";
        case HS_ERR_INVALID_VALUE: return "HS_ERR_INVALID_VALUE: invalid argument";
        case HS_ERR_NOT_SUPPORTED: return "HS_ERR_NOT_SUPPORTED: dtype or size not supported for this call";
        case HS_ERR_WORKSPACE_TOO_SMALL: return "HS_ERR_WORKSPACE_TOO_SMALL: workspace smaller than hs_workspace_size()";
        case HS_ERR_LAUNCH_FAILED: return "HS_ERR_LAUNCH_FAILED: the HIP runtime rejected a launch";
        case HS_ERR_EXCEEDS_SCRATCH:
            return "HS_ERR_EXCEEDS_SCRATCH: the call needs more workspace than hs_gemm_noalloc's static scratch holds";
    }
    return "unknown hs_status";
}

hs_status hs_schedule_resolve(hs_schedule in, hs_schedule *out) {
    if (!out) return HS_ERR_INVALID_VALUE;
    if (in.p < 1 || in.p > kMaxP || in.K < 0) return HS_ERR_INVALID_VALUE;
    int K = in.K == 0 ? default_K(in.p) : in.K;
    if (K > in.p || in.p % K != 0) return HS_ERR_INVALID_VALUE;
    out->p = in.p;
    out->K = K;
    return HS_OK;
}

hs_status hs_schedule_table(hs_schedule s, int32_t *out, size_t cap) {
    hs_schedule r;
    HS_TRY(hs_schedule_resolve(s, &r));
    const int p = r.p, K = r.K, Kt = p / K;
    if (!out || cap < (size_t)2 * p * p) return HS_ERR_INVALID_VALUE;
    size_t t = 0;
    for (int v = 0; v < p; ++v)
        for (int j = 0; j < Kt; ++j)
            for (int l = 0; l < K; ++l) {
                out[t++] = ((v - l) % p + p) % p;   // output stripe: partial c^l of v
                out[t++] = (v + j * K) % p;         // travelling block after j shifts by K
            }
    return HS_OK;
}

size_t hs_workspace_size(int op, int64_t m, int64_t n, int64_t k, int dtype, hs_schedule s) {
    const size_t bad = std::numeric_limits<size_t>::max();
    Plan P;
    switch (op) {
        case HS_OP_GEMM: {
            hs_dtype base;
            if (complex_base(dtype, &base)) {
                if (m < 0 || n < 0 || k < 0 || make_plan(m, 2 * n, 2 * k, base, s, &P) != HS_OK) return bad;
                return P.total;
            }
            if (make_plan(m, n, k, dtype, s, &P) != HS_OK) return bad;
            return P.total;
        }
        case HS_OP_GEMM_TN: {
            hs_dtype base;
            if (complex_base(dtype, &base)) {
                if (m < 0 || n < 0 || k < 0 || make_plan(m, 2 * n, 2 * k, base, s, &P) != HS_OK) return bad;
                return P.total;
            }
            if (make_plan(m, n, k, dtype, s, &P) != HS_OK) return bad;
            return P.total;
        }
        case HS_OP_GEMV: {
            if (dtype != HS_F32 && dtype != HS_F64 && dtype != HS_C32) return bad;
            hs_schedule r;
            if (hs_schedule_resolve(s, &r) != HS_OK || m < 0 || n < 0) return bad;
            return 0;
        }
        case HS_OP_NBODY: {
            NbodyArgs a;
            size_t ws;
            if (nbody_plan(m, dtype, s, 0.0, &a, &ws) != HS_OK) return bad;
            return ws;
        }
        case HS_OP_BACKWARD: {
            Plan Pa, Pb;
            hs_dtype base;
            if (complex_base(dtype, &base)) {
                if (m < 0 || n < 0 || k < 0) return bad;
                if (make_plan(m, 2 * k, 2 * n, base, s, &Pa) != HS_OK) return bad;
                if (make_plan(k, 2 * n, 2 * m, base, s, &Pb) != HS_OK) return bad;
                return std::max(Pa.total, Pb.total);
            }
            if (make_plan(m, k, n, dtype, s, &Pa) != HS_OK) return bad;
            if (make_plan(k, n, m, dtype, s, &Pb) != HS_OK) return bad;
            return std::max(Pa.total, Pb.total);
        }
    }
    return bad;
}

hs_status hs_gemm(int64_t m, int64_t n, int64_t k, int dtype, hs_schedule s,
                  const void *A, int64_t lda, const void *B, int64_t ldb,
                  void *C, int64_t ldc, void *ws, size_t ws_bytes, void *stream) {
    hs_dtype base;
    if (complex_base(dtype, &base)) {
        // one real product: A as m x 2k, B embedded as 2k x 2n, C as m x 2n
        if (m < 0 || n < 0 || k < 0) return HS_ERR_INVALID_VALUE;
        Plan P;
        HS_TRY(make_plan(m, 2 * n, 2 * k, base, s, &P));
        HS_TRY(check_mat(A, m, k, lda, 8));
        HS_TRY(check_mat(B, k, n, ldb, 8));
        HS_TRY(check_mat(C, m, n, ldc, 8));
        HS_TRY(check_ws(P, ws, ws_bytes));
        return run_product(P, Operand{A, 2 * lda, 1, EMB_NONE}, Operand{B, 2 * ldb, 0, EMB_BLOCKS}, C, 2 * ldc, ws,
                           (hipStream_t)stream);
    }
    Plan P;
    HS_TRY(make_plan(m, n, k, dtype, s, &P));
    HS_TRY(check_mat(A, m, k, lda, P.f.in_esz));
    HS_TRY(check_mat(B, k, n, ldb, P.f.in_esz));
    HS_TRY(check_mat(C, m, n, ldc, P.f.out_f64 ? 8 : 4));
    HS_TRY(check_ws(P, ws, ws_bytes));
    return run_product(P, Operand{A, lda, 1, EMB_NONE}, Operand{B, ldb, 0, EMB_NONE}, C, ldc, ws, (hipStream_t)stream);
}

hs_status hs_gemm_tn(int64_t m, int64_t n, int64_t k, int dtype, hs_schedule s,
                     const void *A, int64_t lda, const void *B, int64_t ldb,
                     void *C, int64_t ldc, void *ws, size_t ws_bytes, void *stream) {
    hs_dtype base;
    if (complex_base(dtype, &base)) {
        // A^T as m x 2k reals, read along A's columns; B embedded as 2k x 2n
        if (m < 0 || n < 0 || k < 0) return HS_ERR_INVALID_VALUE;
        Plan P;
        HS_TRY(make_plan(m, 2 * n, 2 * k, base, s, &P));
        HS_TRY(check_mat(A, k, m, lda, 8));
        HS_TRY(check_mat(B, k, n, ldb, 8));
        HS_TRY(check_mat(C, m, n, ldc, 8));
        HS_TRY(check_ws(P, ws, ws_bytes));
        return run_product(P, Operand{A, 2 * lda, 0, EMB_TRANS}, Operand{B, 2 * ldb, 0, EMB_BLOCKS}, C, 2 * ldc, ws,
                           (hipStream_t)stream);
    }
    Plan P;
    HS_TRY(make_plan(m, n, k, dtype, s, &P));
    HS_TRY(check_mat(A, k, m, lda, P.f.in_esz));
    HS_TRY(check_mat(B, k, n, ldb, P.f.in_esz));
    HS_TRY(check_mat(C, m, n, ldc, P.f.out_f64 ? 8 : 4));
    HS_TRY(check_ws(P, ws, ws_bytes));
    return run_product(P, Operand{A, lda, 0, EMB_NONE}, Operand{B, ldb, 0, EMB_NONE}, C, ldc, ws, (hipStream_t)stream);
}

hs_status hs_gemv(int64_t m, int64_t n, int dtype, hs_schedule s,
                  const void *A, int64_t lda, const void *x, void *y,
                  void *ws, size_t ws_bytes, void *stream) {
    (void)ws;
    (void)ws_bytes;
    if (dtype != HS_F32 && dtype != HS_F64 && dtype != HS_C32) return HS_ERR_NOT_SUPPORTED;
    hs_schedule r;
    HS_TRY(hs_schedule_resolve(s, &r));
    const int cplx = dtype == HS_C32;
    const size_t esz = dtype == HS_F32 ? 4 : 8;
    if (m > std::numeric_limits<int32_t>::max()) return HS_ERR_NOT_SUPPORTED;   // 4 rows per workgroup, 32-bit grid
    HS_TRY(check_mat(A, m, n, lda, esz));
    if (n > 0 && m > 0 && (!x || !aligned(x, esz))) return HS_ERR_INVALID_VALUE;
    if (m > 0 && (!y || !aligned(y, esz))) return HS_ERR_INVALID_VALUE;
    if (m == 0) return HS_OK;
    hipStream_t st = (hipStream_t)stream;
    const int f64 = dtype == HS_F64;
    if (n == 0) return launch_status(cplx ? launch_fill_zero(0, y, m, 2, 2, st) : launch_fill_zero(f64, y, m, 1, 1, st));
    GemvArgs g{};
    g.cplx = cplx;
    g.A = A; g.lda = lda; g.x = x; g.y = y; g.m = m; g.n = n;
    if (std::max<int64_t>(1, ceil_div(n, r.p)) * r.p >= ((int64_t)1 << 31)) return HS_ERR_NOT_SUPPORTED;   // 32-bit positions
    // waves per row: one, two for long rows (FP32 2500 x 16384 30 us against 34,
    // 16384 x 16384 166 against 170; but 3500 x 5000 12.0 against 11.5), four for
    // few rows that are not short (100 x 10000 4.0 us against 4.4, 250 x 16384
    // 5.3 against 7.6; but 2500 x 5000 10.2 against 8.9)
    const int64_t row_bytes = n * (int64_t)esz;
    g.waves = m < 400 && row_bytes >= 24 * 1024 ? 4 : row_bytes >= 48 * 1024 ? 2 : 1;
    // sixteen lanes a row, four rows a wave, for many short rows: a wave's sums
    // across its lanes then serve four (400000 x 122 FP32 48 us against 164 with 64
    // lanes, 100000 x 500 30, 49, 16384 x 1500 16.5, 18.8; but 32768 x 3000 63, 57, and
    // 2000 x 1500 4.7, 4.5; FP64 100000 x 122 18, 36, 32768 x 1000 38, 38)
    g.lanes = m >= 8192 && row_bytes <= 6 * 1024 ? 16 : 64;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (g_prof && !timing_events(&ev0, &ev1)) return HS_ERR_LAUNCH_FAILED;
    hipError_t e = launch_gemv(f64, g, st);
    if (g_prof) keep_timing(ev0, ev1);
    return launch_status(e);
}

hs_status hs_gemm_backward(int64_t m, int64_t n, int64_t k, int dtype, hs_schedule s,
                           const void *A, int64_t lda, const void *B, int64_t ldb,
                           const void *G, int64_t ldg,
                           void *dA, int64_t ldda, void *dB, int64_t lddb,
                           void *ws, size_t ws_bytes, void *stream) {
    hs_dtype base;
    if (complex_base(dtype, &base)) {
        // dA = G . B^H: G as m x 2n reals, B^H as the 2n x 2k block embedding
        // of conj(B)^T; dB = A^H . G: conj(A)^T as k x 2m reals, G as the
        // 2m x 2n block embedding.  Outputs as interleaved complex.
        if (m < 0 || n < 0 || k < 0) return HS_ERR_INVALID_VALUE;
        Plan Pa, Pb;
        HS_TRY(make_plan(m, 2 * k, 2 * n, base, s, &Pa));
        HS_TRY(make_plan(k, 2 * n, 2 * m, base, s, &Pb));
        HS_TRY(check_mat(G, m, n, ldg, 8));
        if (dA) {
            HS_TRY(check_mat(B, k, n, ldb, 8));
            HS_TRY(check_mat(dA, m, k, ldda, 8));
            HS_TRY(check_ws(Pa, ws, ws_bytes));
        }
        if (dB) {
            HS_TRY(check_mat(A, m, k, lda, 8));
            HS_TRY(check_mat(dB, k, n, lddb, 8));
            HS_TRY(check_ws(Pb, ws, ws_bytes));
        }
        hipStream_t st = (hipStream_t)stream;
        if (dA) HS_TRY(run_product(Pa, Operand{G, 2 * ldg, 1, EMB_NONE}, Operand{B, 2 * ldb, 1, EMB_BLOCKS_H},
                                   dA, 2 * ldda, ws, st));
        if (dB) HS_TRY(run_product(Pb, Operand{A, 2 * lda, 0, EMB_CONJ}, Operand{G, 2 * ldg, 0, EMB_BLOCKS},
                                   dB, 2 * lddb, ws, st));
        return HS_OK;
    }
    Plan Pa, Pb;
    HS_TRY(make_plan(m, k, n, dtype, s, &Pa));   // dA[m,k] = G[m,n] . B[k,n]^T
    HS_TRY(make_plan(k, n, m, dtype, s, &Pb));   // dB[k,n] = A[m,k]^T . G[m,n]
    const size_t oesz = Pa.f.out_f64 ? 8 : 4;
    HS_TRY(check_mat(G, m, n, ldg, Pa.f.in_esz));
    if (dA) {
        HS_TRY(check_mat(B, k, n, ldb, Pa.f.in_esz));
        HS_TRY(check_mat(dA, m, k, ldda, oesz));
        HS_TRY(check_ws(Pa, ws, ws_bytes));
    }
    if (dB) {
        HS_TRY(check_mat(A, m, k, lda, Pb.f.in_esz));
        HS_TRY(check_mat(dB, k, n, lddb, oesz));
        HS_TRY(check_ws(Pb, ws, ws_bytes));
    }
    hipStream_t st = (hipStream_t)stream;
    if (dA) HS_TRY(run_product(Pa, Operand{G, ldg, 1, EMB_NONE}, Operand{B, ldb, 1, EMB_NONE}, dA, ldda, ws, st));
    if (dB) HS_TRY(run_product(Pb, Operand{A, lda, 0, EMB_NONE}, Operand{G, ldg, 0, EMB_NONE}, dB, lddb, ws, st));
    return HS_OK;
}

hs_status hs_nbody(int64_t n, int dtype, hs_schedule s, const void *bodies, double eps2, void *out,
                   void *ws, size_t ws_bytes, void *stream) {
    NbodyArgs a;
    size_t need;
    HS_TRY(nbody_plan(n, dtype, s, eps2, &a, &need));
    if (n == 0) return HS_OK;
    const int f64 = dtype == HS_F64;
    const size_t row = f64 ? 32 : 16;             // one body: 4 values
    if (!bodies || !out || !aligned(bodies, row) || !aligned(out, row)) return HS_ERR_INVALID_VALUE;
    const uintptr_t b0 = (uintptr_t)bodies, o0 = (uintptr_t)out, len = (uintptr_t)n * row;
    if (b0 < o0 + len && o0 < b0 + len) return HS_ERR_INVALID_VALUE;   // out must not overlap bodies
    if (need > 0) {
        if (!ws) return HS_ERR_WORKSPACE_TOO_SMALL;
        if (!aligned(ws, kAlign)) return HS_ERR_INVALID_VALUE;
        if (ws_bytes < need) return HS_ERR_WORKSPACE_TOO_SMALL;
    }
    hipStream_t st = (hipStream_t)stream;
    void *dst = a.K > 1 ? ws : out;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (g_prof && !timing_events(&ev0, &ev1)) return HS_ERR_LAUNCH_FAILED;
    hipError_t e = launch_nbody(f64, bodies, dst, a, st);
    if (g_prof) keep_timing(ev0, ev1);
    if (e != hipSuccess) return HS_ERR_LAUNCH_FAILED;
    if (a.K > 1) return launch_status(launch_backshift(f64, ws, 4 * n, a.K, n, 4, out, 4, st));
    return HS_OK;
}

hs_status hs_profile_begin(void) {
    g_prof = true;
    return HS_OK;
}

hs_status hs_profile_end(double *total_ms, int64_t *launches) {
    if (!g_prof) return HS_ERR_INVALID_VALUE;
    g_prof = false;
    double tot = 0.0;
    int64_t n = 0;
    hs_status st = HS_OK;
    for (auto &pr : g_events) {
        float ms = 0.f;
        if (hipEventSynchronize(pr.second) != hipSuccess ||
            hipEventElapsedTime(&ms, pr.first, pr.second) != hipSuccess)
            st = HS_ERR_LAUNCH_FAILED;
        tot += ms;
        ++n;
        (void)hipEventDestroy(pr.first);
        (void)hipEventDestroy(pr.second);
    }
    g_events.clear();
    if (total_ms) *total_ms = tot;
    if (launches) *launches = n;
    return st;
}

}  // extern "C"
