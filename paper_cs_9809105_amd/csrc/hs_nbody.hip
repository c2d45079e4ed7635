// hs_nbody.hip -- the all-pairs gravitational interaction of n bodies (the
// prototype n^2-problem of Sec. 2.2) on the two-array hyper-systolic recipe
// of Sec. 4.1 with the regular bases of Def. REGULARBASE2.
//
// The bodies are cut into p blocks of S = ceil(n / p); virtual processor v
// owns block v.  With 0-based indices and K * K~ = p:
//
//   replicas  x^_t = block (v + t) mod p,   t = 0..K-1   (A = (0, 1, .., 1))
//   travel    step j: z = block (v + j K) mod p, j = 0..K~-1   (B = (0, K, .., K))
//   results   y^_t(v) += f(x^_t, z) over every step
//   collector y(b) = y^_0 + (y^_1 + ( .. + y^_{K-1}))   for body block b,
//             where y^_t comes from processor (b - t) mod p
//
// f(x, z) adds, for target body x and source body z (z != x),
//   a   += m_z (r_z - r_x) / (|r_z - r_x|^2 + eps2)^(3/2)
//   phi -= m_z / (|r_z - r_x|^2 + eps2)^(1/2).
// Every ordered pair of bodies meets exactly once (the base pair is complete
// and K K~ = p, so no multiplicity table is needed); the only pairs of a body
// with itself occur for replica t = 0 at step j = 0, where they are skipped.
//
// On the GPU a virtual processor is a group of workgroups.  A thread holds
// one body position i of the stripe in one of the K replicas (registers), and
// reads its share of the travelling blocks body by body with wave-uniform
// loads.  The collector's moves by
// -1 become addressing: replica t of processor v writes its results into
// partial plane t at the rows of the bodies it belongs to (block v + t), and
// the back-shift kernel sums the K planes per body in the order above, in
// FP64.  K = 1 (the systolic special case) writes the result directly.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hs_internal.h"

namespace hs {

#define DEVI __device__ __forceinline__

template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
    typedef float4 type;
};
template <>
struct Vec4<double> {
    typedef double4 type;
};

DEVI float inv_sqrt(float s) { return __builtin_amdgcn_rsqf(s); }
DEVI double inv_sqrt(double s) { return 1.0 / sqrt(s); }
DEVI float fma3(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
DEVI double fma3(double a, double b, double c) { return __builtin_fma(a, b, c); }

// One travelling body (zx, zy, zz, zm) against the thread's body.
// SELF: this is step j = 0 of replica t = 0, where source position jj equals
// the thread's own position i.
// 14 VALU instructions per pair (one v_rsq_f32).  The potential takes its
// own fused multiply-add from inv, independent of m / s^(1/2): forming that
// product once and subtracting it measured 15 % slower.
template <typename T, bool SELF>
DEVI void interact(const T zx, const T zy, const T zz, const T zm, const int jj, const int i, const T eps2,
                   const T px, const T py, const T pz, T &ax, T &ay, T &az, T &ph) {
    const T dx = zx - px;
    const T dy = zy - py;
    const T dz = zz - pz;
    const T s = fma3(dz, dz, fma3(dy, dy, fma3(dx, dx, eps2)));
    T inv = inv_sqrt(s);
    if (SELF) inv = (jj == i) ? (T)0 : inv;
    ph = fma3(-zm, inv, ph);                // phi -= m / s^(1/2)
    const T w = (zm * inv) * (inv * inv);   // m / s^(3/2)
    ax = fma3(w, dx, ax);
    ay = fma3(w, dy, ay);
    az = fma3(w, dz, az);
}

// Travelling bodies [jj, end) of the block at src, UB per round of
// wave-uniform loads, the last ones in rounds of half the size each.
template <typename T, bool SELF, int UB>
DEVI void travel(const T *__restrict__ src, int jj, const int end, const int i, const T eps2, const T px, const T py,
                 const T pz, T &ax, T &ay, T &az, T &ph) {
    for (; jj + UB <= end; jj += UB) {
        T z[UB][4];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
#pragma unroll
            for (int c = 0; c < 4; ++c) z[u][c] = src[(int64_t)(jj + u) * 4 + c];
        }
#pragma unroll
        for (int u = 0; u < UB; ++u)
            interact<T, SELF>(z[u][0], z[u][1], z[u][2], z[u][3], jj + u, i, eps2, px, py, pz, ax, ay, az, ph);
    }
    if constexpr (UB > 1)
        if (jj < end) travel<T, SELF, UB / 2>(src, jj, end, i, eps2, px, py, pz, ax, ay, az, ph);
}

// Grid: (sub K) x p workgroups of ss waves (host-checked): replica t = x % K,
// slice s = x / K (positions s*64 .. s*64+63 of the block), virtual processor
// v = y.
// Wave q of the workgroup takes run q of ss equal runs of the K~ S travelling
// bodies (blocks v, v + K, .. one after the other), and the waves' sums are
// added in their order through LDS: the positions of a few thousand bodies
// alone would occupy a small part of the chip.  Bound by vector ALU issue at
// the largest sizes and by filling the SIMDs below.  A thread per position and
// pair of replicas, four waves side by side along a block (256-body slices),
// measured 58 us at n = 3000 (p = 16, K = 4) against 10, 1061 against 720 at
// n = 50000 (p = 64, K = 8), 19.9 ms against 18.1 at n = 262144; two replicas
// per thread here 13.7 us, 752 us and 18.7 ms.
template <typename T>
__global__ __launch_bounds__(1024) void nbody_kernel(const T *__restrict__ bodies, T *__restrict__ out,
                                                     NbodyArgs a) {
    typedef typename Vec4<T>::type V4;
    constexpr int UB = 8;                             // FP32 n = 262144: 18.1 ms; 19.1 with 4
    extern __shared__ __attribute__((aligned(32))) uint8_t lds[];      // ss > 1: [ss][64] results
    const int p = a.p, K = a.K, S = a.S;
    const int s = (int)blockIdx.x / K, t = (int)blockIdx.x - s * K, v = (int)blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i = s * 64 + lane;                      // position in the stripe
    const T eps2 = (T)a.eps2;

    const int64_t row = (int64_t)((v + t) % p) * S + i;   // replica t: block v + t
    const bool ok = i < S && row < a.n;
    T px = 0, py = 0, pz = 0, ax = 0, ay = 0, az = 0, ph = 0;
    if (ok) {
        const V4 b = ((const V4 *)bodies)[row];
        px = b.x;
        py = b.y;
        pz = b.z;
    }

    // this wave's run [e0, e1) of the Kt S travelling positions, block by block
    const int64_t total = (int64_t)a.Kt * S;
    const int64_t e0 = total * q / a.ss, e1 = total * (q + 1) / a.ss;
    int j = (int)(e0 / S);
    int from = (int)(e0 - (int64_t)j * S);
    for (int64_t left = e1 - e0; left > 0; ++j, from = 0) {
        int to = left < S - from ? from + (int)left : S;
        left -= to - from;
        const int blk = (v + j * K) % p;              // travelling block after j shifts by K
        const int64_t base = (int64_t)blk * S;
        const int64_t have = a.n - base;              // the last block may be short or empty
        if (to > have) to = have < 0 ? 0 : (int)have;
        const T *src = bodies + base * 4;
        if (j == 0 && t == 0)
            travel<T, true, UB>(src, from, to, i, eps2, px, py, pz, ax, ay, az, ph);
        else
            travel<T, false, UB>(src, from, to, i, eps2, px, py, pz, ax, ay, az, ph);
    }

    V4 o;
    o.x = ax;
    o.y = ay;
    o.z = az;
    o.w = ph;
    if (a.ss > 1) {
        V4 *part = (V4 *)lds;
        part[q * 64 + lane] = o;
        __syncthreads();
        if (q != 0) return;
        for (int u = 1; u < a.ss; ++u) {
            const V4 b = part[u * 64 + lane];
            o.x += b.x;
            o.y += b.y;
            o.z += b.z;
            o.w += b.w;
        }
    }
    if (ok) ((V4 *)out)[t * a.n + row] = o;           // K == 1: plane 0 is the result
}

bool take_timed_launch(hipEvent_t *start, hipEvent_t *stop);   // hs_kernels.hip

hipError_t launch_nbody(int f64, const void *bodies, void *out, const NbodyArgs &a, hipStream_t st) {
    if (a.n == 0) return hipSuccess;
    const dim3 grid((unsigned)(a.sub * a.K), (unsigned)a.p), block(64 * a.ss);
    const unsigned lds = a.ss > 1 ? (unsigned)a.ss * 64 * (f64 ? 32 : 16) : 0;   // <= 32 KiB
    hipEvent_t ts, te;
    const bool timed = take_timed_launch(&ts, &te);   // hs_profile_*: events recorded by the dispatch
#define HS_NB(T)                                                                                              \
    do {                                                                                                      \
        if (timed)                                                                                            \
            hipExtLaunchKernelGGL((nbody_kernel<T>), grid, block, lds, st, ts, te, 0, (const T *)bodies,       \
                                  (T *)out, a);                                                               \
        else                                                                                                  \
            hipLaunchKernelGGL((nbody_kernel<T>), grid, block, lds, st, (const T *)bodies, (T *)out, a);      \
    } while (0)
    if (f64) HS_NB(double);
    else HS_NB(float);
#undef HS_NB
    return hipGetLastError();
}

}  // namespace hs
