// One-wavefront building blocks on v_mfma_f64_16x16x4f64, shared by the shot
// kernels: lane l = 16 g + q holds element (row q, k = g) of an A operand,
// element (k = g, column q) of a B operand, and rows g + 4 r, r = 0..3, of
// column q of a result.
#pragma once

#include <hip/hip_runtime.h>

#include "mps_common.h"

namespace msc {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mfma(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// The lane's index, opaque to the compiler: what an op derives from it (offsets,
// lane masks) is computed there and not carried through the whole shot loop
// in registers.
__device__ __forceinline__ int op_lane() {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

// Orders the wavefront's LDS and global accesses for the compiler; the
// hardware performs one wavefront's accesses to either memory in order.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Element i of a tensor plane, by a 32-bit byte offset from its (uniform) base.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T& at(
    __attribute__((address_space(1))) T* p, uint32_t i) {
    typedef __attribute__((address_space(1))) char gchar;
    return *(__attribute__((address_space(1))) T*)((gchar*)p + i * static_cast<uint32_t>(sizeof(T)));
}

// Four sums over the wavefront, every lane receiving them: a product with
// ones adds each value over the lane rows, a second one what is left of
// value j over the columns of its quad's lane j, from where it is spread.
__device__ __forceinline__ void wave_sum4(double (&v)[4]) {
    const int j = op_lane() & 3;
    const f64x4 z = {0.0, 0.0, 0.0, 0.0};
    double p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f64x4 d = mfma(v[i], 1.0, z);
        p[i] = (d[0] + d[1]) + (d[2] + d[3]);
    }
    const double x = (j & 2) ? ((j & 1) ? p[3] : p[2]) : ((j & 1) ? p[1] : p[0]);
    const double t = mfma(1.0, x, z)[0];
    v[0] = dpp_move<0x00>(t);
    v[1] = dpp_move<0x55>(t);
    v[2] = dpp_move<0xAA>(t);
    v[3] = dpp_move<0xFF>(t);
}

// Sum and maximum over the 16 lanes of a row, every lane receiving it.
__device__ __forceinline__ double row_sum(double v) { return group_sum(v, 16); }
__device__ __forceinline__ double row_max(double v) {
    v = fmax(v, dpp_move<0xB1>(v));
    v = fmax(v, dpp_move<0x4E>(v));
    v = fmax(v, dpp_move<0x141>(v));
    return fmax(v, dpp_move<0x140>(v));
}

// For a condition b on (row g, column q), the number of lanes of this lane's
// column where it holds.
__device__ __forceinline__ int column_count(bool b, uint32_t colmask) {
    const uint64_t m = __ballot(b);
    return __popc(static_cast<uint32_t>(m) & colmask) +
           __popc(static_cast<uint32_t>(m >> 32) & colmask);
}

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Gram tile of the vectors 16 tp + p and 16 tq + q at V (vector v at v * ld, its
// imaginary part lp further): entry (p, q) is x_p^H y_q, its real and
// imaginary parts in re and im (len elements, zero-padded to a multiple of 4).
template <typename DP>
__device__ __forceinline__ void gram_tile(DP V, int tp, int tq, int ld, int lp, int len, f64x4& re,
                                          f64x4& im) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    re = f64x4{0.0, 0.0, 0.0, 0.0};
    im = f64x4{0.0, 0.0, 0.0, 0.0};
    DP x = V + (16 * tp + q) * ld + g;
    DP y = V + (16 * tq + q) * ld + g;
#pragma unroll 2
    for (int e = 0; e < len; e += 4) {
        const double xr = x[e], xi = x[lp + e];
        const double yr = tp == tq ? xr : y[e], yi = tp == tq ? xi : y[lp + e];
        re = mfma(xr, yr, re);
        im = mfma(xr, yi, im);
        re = mfma(xi, yi, re);
        im = mfma(-xi, yr, im);
    }
}

// The diagonal of a diagonal Gram tile: entry (q, q), held by lane row q mod 4
// in register q / 4, is stored by that lane.
__device__ __forceinline__ void store_diagonal(const f64x4& re, ldsd* nrm) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const int r = q >> 2;
    const double d01 = (r & 1) ? re[1] : re[0], d23 = (r & 1) ? re[3] : re[2];
    if (g == (q & 3)) nrm[q] = (r & 2) ? d23 : d01;
}

// One Gram tile's overlapping pairs (rows 16 tp + g + 4 r, columns 16 tq + q,
// the upper triangle): a pair overlaps when both squared norms exceed floor2
// and |x^H y|^2 > tol2 |x|^2 |y|^2; cnt[v] counts the vectors v overlaps, mate[v]
// names one of them and gre/gim[v] hold the pair's x^H y with x its
// lower-numbered vector.  Returns 0, 1 (found some) or 2 (some vector
// overlaps more than one).
template <int SCOPE = __HIP_MEMORY_SCOPE_WAVEFRONT, typename LW>
__device__ __forceinline__ int tile_overlaps(int tp, int tq, const f64x4& gr, const f64x4& gi,
                                             LW* L, double floor2, double tol2) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const ldsd* nrm = L->nrm;
    const double b = nrm[16 * tq + q];
    int any = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double a = nrm[16 * tp + g + 4 * r];
        const double g2 = gr[r] * gr[r] + gi[r] * gi[r];
        if ((tp < tq || g + 4 * r < q) && a > floor2 && b > floor2 && g2 > tol2 * a * b) {
            const int p = 16 * tp + g + 4 * r, c = 16 * tq + q;
            ldsi* cnt = L->cnt;
            ldsi* mate = L->mate;
            ldsd* gre = L->gre;
            ldsd* gim = L->gim;
            const int o0 = __hip_atomic_fetch_add(cnt + p, 1, __ATOMIC_RELAXED,
                                                  SCOPE);
            const int o1 = __hip_atomic_fetch_add(cnt + c, 1, __ATOMIC_RELAXED,
                                                  SCOPE);
            any |= (o0 | o1) ? 2 : 1;
            mate[p] = c;
            mate[c] = p;
            gre[p] = gr[r];
            gre[c] = gr[r];
            gim[p] = gi[r];
            gim[c] = gi[r];
        }
    }
    return any;
}

}  // namespace
}  // namespace msc
