// Device helpers shared by the shot kernels (mps.hip, mps_fast.hip): lane
// teams and their reductions, address-space pointers, index splits, one-sided
// Jacobi sweeps, and the small records a shot carries.
#pragma once

#include <hip/hip_runtime.h>

#include <cfloat>
#include <cstdint>

#include "kernels.h"

namespace msc {
namespace {

constexpr int NT = 256;
constexpr int NW = NT / 64;
// A team is either the whole workgroup (W == NT) or wavefront 0 (W == 64).
template <int W>
struct Team {
    static __device__ __forceinline__ int rank() { return W == 64 ? (threadIdx.x & 63) : threadIdx.x; }
    static __device__ __forceinline__ void sync() {
        if constexpr (W == NT) {
            __syncthreads();
        } else {
            // a workgroup-scope fence without the barrier: this wavefront's
            // LDS and global writes become visible to all its lanes
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
    }
    static __device__ __forceinline__ bool any(int v) {
        if constexpr (W == NT) {
            return __syncthreads_or(v) != 0;
        } else {
            sync();
            return __ballot(v) != 0ull;
        }
    }
};

// A double moved between lanes of a row of 16 by a DPP pattern (two 32-bit
// lane moves): quad_perm [1,0,3,2] = 0xB1, quad_perm [2,3,0,1] = 0x4E,
// row_half_mirror = 0x141, row_mirror = 0x140.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Sum over aligned groups of g consecutive lanes (g a power of two <= 64),
// every lane of a group receiving it: pairs within quads, then the two
// quads of each half row (mirror), then the two halves of a row (mirror),
// then across rows.
__device__ __forceinline__ double group_sum(double v, int g) {
    if (g >= 2) v += dpp_move<0xB1>(v);
    if (g >= 4) v += dpp_move<0x4E>(v);
    if (g >= 8) v += dpp_move<0x141>(v);
    if (g >= 16) v += dpp_move<0x140>(v);
    if (g >= 32) v += __shfl_xor(v, 16);
    if (g >= 64) v += __shfl_xor(v, 32);
    return v;
}

// The double held by lane l (v_readlane, the same value in every lane).
__device__ __forceinline__ double lane_read(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Sum over the whole wavefront (all lanes active), every lane receiving it:
// the row sums by DPP, then the four rows' sums read from lanes 0, 16, 32
// and 48 and added in a fixed order.
__device__ __forceinline__ double wave_sum(double v) {
    v = group_sum(v, 16);
    return (lane_read(v, 0) + lane_read(v, 16)) + (lane_read(v, 32) + lane_read(v, 48));
}

__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_move<0xB1>(v));
    v = fmax(v, dpp_move<0x4E>(v));
    v = fmax(v, dpp_move<0x141>(v));
    v = fmax(v, dpp_move<0x140>(v));
    return fmax(fmax(lane_read(v, 0), lane_read(v, 16)), fmax(lane_read(v, 32), lane_read(v, 48)));
}

template <int W, int K>
__device__ __forceinline__ void team_sum(double (&v)[K], double* red) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
    if constexpr (W == NT) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        __syncthreads();
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) red[w * K + k] = v[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < NW; ++j) s += red[j * K + k];
            v[k] = s;
        }
    }
}

template <int W>
__device__ __forceinline__ double team_max(double v, double* red) {
    v = wave_max(v);
    if constexpr (W == NT) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        __syncthreads();
        if (lane == 0) red[w] = v;
        __syncthreads();
        double m = red[0];
#pragma unroll
        for (int j = 1; j < NW; ++j) m = fmax(m, red[j]);
        v = m;
    }
    return v;
}

// Round-robin ("circle") pairing: slot 0 fixed, the others rotate each step.
__device__ __forceinline__ int player(int slot, int t, int nv) {
    if (slot == 0) return 0;
    int p = slot - 1 + t;
    if (p >= nv - 1) p -= nv - 1;
    return 1 + p;
}

// Pointers into LDS and into global memory with their address space in the
// type, so that the compiler emits ds_read/ds_write and global_load/store
// rather than generic flat accesses in the hot loops.
typedef __attribute__((address_space(3))) double ldsd;
typedef __attribute__((address_space(3))) int ldsi;
typedef __attribute__((address_space(1))) double glbd;
typedef __attribute__((address_space(1))) int glbi;

template <typename X>
__device__ __forceinline__ __attribute__((address_space(3))) X* to_lds(X* p) {
    return (__attribute__((address_space(3))) X*)p;
}
template <typename X>
__device__ __forceinline__ __attribute__((address_space(1))) X* to_glb(X* p) {
    return (__attribute__((address_space(1))) X*)p;
}

// One wavefront's asynchronous copy of `bytes` bytes from global memory to
// LDS by direct loads (global_load_lds_dwordx4: lane i's 16 bytes land at
// dst + 16 i), with no register round trip.  Both addresses are 16-byte
// aligned and both sides must have room for the size rounded up to 16
// bytes.  The data is in LDS once the wavefront's vector-memory counter has
// drained (any Team<64>::sync()).
template <typename GP>
__device__ __forceinline__ void wave_load_lds(GP src, void* dst, int bytes) {
    typedef __attribute__((address_space(1))) char gchar;
    typedef __attribute__((address_space(3))) char lchar;
    const int lane = threadIdx.x & 63;
    const int n16 = (bytes + 15) >> 4;
    gchar* s8 = (gchar*)src;
    lchar* d8 = (lchar*)dst;
    for (int b = 0; b < n16; b += 64) {
        if (b + lane < n16)
            __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)(s8 + 16 * (b + lane)),
                                             (__attribute__((address_space(3))) void*)(d8 + 16 * b), 16, 0, 0);
    }
}

// Elements of T rounded up to a multiple of 16 bytes.
// 1/sqrt(x) for a positive normal x: the hardware estimate refined by two
// Newton steps y <- y + y (1 - x y^2) / 2 (quadratic convergence), to about
// an ulp; a few fused multiply-adds instead of a correctly rounded square
// root and a division.
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
    e = fma(-x * y, y, 1.0);
    return fma(0.5 * y, e, y);
}

// 1/d for a positive divisor: the hardware estimate refined by one Newton
// step e = 1 - d y, y <- y + y e, to a relative error far below 2^-40.
__device__ __forceinline__ double rcp_nr(int d) {
    const double x = static_cast<double>(d);
    const double y = __builtin_amdgcn_rcp(x);
    return fma(y, fma(-x, y, 1.0), y);
}

// i / d for 0 <= i < 2^31 and 0 < d < 2^20 through inv = rcp_nr(d): the
// exact quotient of i + 1/2 lies at least 1/(2d) from an integer, and the
// product's error is below 2^-20, so truncation gives floor(i / d).  Three
// vector operations instead of the integer division sequence.
__device__ __forceinline__ int qdiv(int i, double inv) {
    return static_cast<int>(fma(static_cast<double>(i), inv, 0.5 * inv));
}

template <typename T>
__device__ __forceinline__ int round16(int n) {
    constexpr int q = 16 / static_cast<int>(sizeof(T));
    return (n + q - 1) / q * q;
}

// One sweep of one-sided Jacobi (Hestenes) over the nv vectors list[0..nv)
// of length len (planar FP64 at vre/vim, vector v at v*ld, ld >= len padded
// against LDS bank conflicts): every pair (p, q) once, in round-robin order
// so that the pairs of a step are disjoint and rotate in parallel (an odd
// count gets a dummy slot).  The 2x2 rotation makes the pair orthogonal:
// with gamma = x^H y, d = |y|^2 - |x|^2, the tangent t = sign(d) / (|zeta| +
// sqrt(1 + zeta^2)) of zeta = d / (2|gamma|), c = 1/sqrt(1+t^2), s = c t,
// x <- c x - s y conj(gamma)/|gamma| and y <- c y + s x gamma/|gamma| (the
// second vector keeps the phase of gamma, which leaves the pair orthogonal
// and spares a division).  With D = |d| + sqrt(d^2 + 4|gamma|^2) and
// rq = 1/sqrt(D^2 + 4|gamma|^2) this is c = D rq and s/|gamma| = 2 sign(d) rq:
// two reciprocal square roots per pair (sqrt(q) = q / sqrt(q)), each a
// refined hardware estimate.
template <int W, typename DP, typename IP>
__device__ void jacobi_sweep(DP vre, DP vim, IP list, int nv, int len, int ld, double floor2,
                             double tol) {
    const int tid = Team<W>::rank();
    if (nv < 2) return;
    const int nve = nv + (nv & 1);   // the slot nv (if odd) is a dummy
    const int npairs = nve / 2;
    int tpp = W / npairs;
    if (tpp > 64) tpp = 64;
    if (tpp < 1) tpp = 1;
    int t2 = 1;
    while (t2 * 2 <= tpp) t2 *= 2;
    tpp = t2;
    const int groups = W / tpp;
    const int gl = tid % tpp;
    const int gi = tid / tpp;
    const double tol2 = tol * tol;
    for (int t = 0; t < nve - 1; ++t) {
        for (int pb = 0; pb < npairs; pb += groups) {
            const int pi = pb + gi;
            const int sp = pi < npairs ? player(pi, t, nve) : 0;
            const int sq = pi < npairs ? player(nve - 1 - pi, t, nve) : 0;
            const bool active = pi < npairs && sp < nv && sq < nv;
            int p = 0, q = 0;
            double a = 0.0, b = 0.0, gr = 0.0, gim = 0.0;
            if (active) {
                p = list[sp];
                q = list[sq];
                DP xr = vre + (size_t)p * ld;
                DP xi = vim + (size_t)p * ld;
                DP yr = vre + (size_t)q * ld;
                DP yi = vim + (size_t)q * ld;
#pragma unroll 2
                for (int e = gl; e < len; e += tpp) {
                    double x0 = xr[e], x1 = xi[e], y0 = yr[e], y1 = yi[e];
                    a += x0 * x0 + x1 * x1;
                    b += y0 * y0 + y1 * y1;
                    gr += x0 * y0 + x1 * y1;
                    gim += x0 * y1 - x1 * y0;
                }
            }
            a = group_sum(a, tpp);
            b = group_sum(b, tpp);
            gr = group_sum(gr, tpp);
            gim = group_sum(gim, tpp);
            if (active) {
                const double g2 = gr * gr + gim * gim;
                if (a > floor2 && b > floor2 && g2 > tol2 * a * b) {
                    const double d = b - a;
                    const double q1 = d * d + 4.0 * g2;
                    const double D = fabs(d) + q1 * rsqrt_nr(q1);
                    const double rq = rsqrt_nr(D * D + 4.0 * g2);
                    const double c = D * rq;
                    const double sg = (d >= 0.0 ? 2.0 : -2.0) * rq;  // s / |gamma|
                    const double pr = sg * gr, pim = sg * gim;        // (s/|gamma|) gamma
                    DP xr = vre + (size_t)p * ld;
                    DP xi = vim + (size_t)p * ld;
                    DP yr = vre + (size_t)q * ld;
                    DP yi = vim + (size_t)q * ld;
#pragma unroll 2
                    for (int e = gl; e < len; e += tpp) {
                        const double x0 = xr[e], x1 = xi[e], y0 = yr[e], y1 = yi[e];
                        // x - (s/|g|) conj(gamma) y and y + (s/|g|) gamma x
                        xr[e] = c * x0 - (pr * y0 + pim * y1);
                        xi[e] = c * x1 - (pr * y1 - pim * y0);
                        yr[e] = c * y0 + (pr * x0 - pim * x1);
                        yi[e] = c * y1 + (pr * x1 + pim * x0);
                    }
                }
            }
        }
        Team<W>::sync();
    }
}

// Compacts the flagged vectors into list (ascending); returns their count.
template <int W, typename IP>
__device__ int flagged_list(IP flag, int nv, IP list, int* red) {
    const int tid = Team<W>::rank(), lane = tid & 63, w = tid >> 6;
    int base = 0;
    for (int b0 = 0; b0 < nv; b0 += W) {
        const int v = b0 + tid;
        const bool f = v < nv && flag[v];
        const uint64_t m = __ballot(f);
        if constexpr (W == NT) {
            __syncthreads();
            if (lane == 0) red[w] = __popcll(m);
            __syncthreads();
            int off = base;
            for (int q = 0; q < w; ++q) off += red[q];
            if (f) list[off + __popcll(m & ((1ull << lane) - 1ull))] = v;
            for (int q = 0; q < NW; ++q) base += red[q];
        } else {
            if (f) list[base + __popcll(m & ((1ull << lane) - 1ull))] = v;
            base += __popcll(m);
        }
    }
    Team<W>::sync();
    return base;
}

struct Kept {
    int r;         // vectors kept
    int want;      // vectors above the threshold (r unless the cap binds)
    double kept, dropped;
};

// A squared norm as the selection orders it: negative or NaN values (only
// ever numerical garbage) count as 0, so the order below is strict and
// every rank from 0 up is taken by exactly one vector.
__device__ __forceinline__ double sel_norm(double x) { return x > 0.0 ? x : 0.0; }

// A site tensor in the slot (global memory): real and imaginary planes.
template <typename T>
struct SiteView {
    __attribute__((address_space(1))) T* re;
    __attribute__((address_space(1))) T* im;
};

// Per-shot counters, reported by thread 0.
struct ShotAcc {
    int status = 0;
    int chi_peak = 1;
    double disc = 0.0;
    int64_t n2q = 0;
    double flops = 0.0;
    int64_t sweeps = 0;
};

// The next entry of a shared work counter, the same value in every lane of
// a one-wavefront team.
__device__ __forceinline__ int64_t wave_fetch(unsigned long long* ctr) {
    unsigned long long v = 0;
    if (Team<64>::rank() == 0) v = atomicAdd(ctr, 1ull);
    // lane 0's value, read into scalar registers: the compiler then treats
    // the shot index and everything derived from it as wave-uniform
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(v), 0);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(v >> 32), 0);
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

}  // namespace
}  // namespace msc
