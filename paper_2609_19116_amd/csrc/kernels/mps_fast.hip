// One-wavefront shot kernel on the matrix cores: one shot per wavefront, four
// per workgroup, for slots of bond cap at most 16.
//
// Same shot loop, ops and results as the wavefront kernel of mps.hip.  What
// bounded that kernel was instruction issue and LDS traffic, not arithmetic:
// the dot products of the orthogonality check read four doubles from LDS for
// every four fused multiply-adds, loops over a few hundred elements paid an
// index split per element, and a pair of overlapping vectors was rotated by
// one step of a round-robin sweep over all flagged vectors.  Here every
// operand is loaded in the lane layout of v_mfma_f64_16x16x4f64:
//   lane l = 16 g + q holds element (row q, k = g) of an A operand, element
//   (k = g, column q) of a B operand, and rows g + 4 r, r = 0..3, of column q
//   of a result.
// A vector v of a factorisation sits in lane column q = v mod 16, its element
// e = 4 s + g in step s of lane row g, which is both operand layouts of its Gram
// matrix at once; per-vector quantities (norm, rank, scale) then belong to
// the lanes that store the vector's elements, so the kept vectors are
// permuted and scaled in registers on their way out.  The overlapping pairs
// come from the Gram matrix and rotate in one step.  All arithmetic is FP64 on
// the stored tensors (FP32 tensors are converted as they are loaded, so theta
// carries no FP32 rounding before it is stored).
//
// Measured against the wavefront kernel of mps.hip: 2^19 shots of the 49-qubit
// circuit (p = 1e-3, FP32) 138.8 -> 81.1 ms a batch, 1000 shots (one shot's
// latency) 36.3 -> 17.3 ms, 65536 17-qubit shots in FP64 64.7 -> 39.7 ms.  Per
// batch the vector instructions fell from 6.0e10 to 2.7e10 and the LDS
// instructions from 5.7e9 to 1.4e9; the matrix cores are busy a quarter of the
// time.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cstdint>

#include "kernels.h"
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

// Truncation of the factorisations: keep sigma > tau * sigma_0, at most cap
// vectors (the slot's bond cap, or chi_max below it).
struct Trunc {
    double tau;
    int chi_max, cap;
};

constexpr int kOps = 16;             // op descriptors held at a time
constexpr int kVec = 32;             // vectors of a factorisation
constexpr int kWork = 32 * 33;       // doubles: 32 vectors of 16, or 16 of 32
constexpr int kStash = 32 * 65;      // doubles: theta put aside in the slot's scratch

// LDS of one wavefront (one base address, constant offsets).
struct WaveLds {
    double work[kWork];              // the vectors of a factorisation
    double nrm[kVec], gre[kVec], gim[kVec];
    DevOp ops[kOps];
    int chi[kMaxSites + 4];          // bond dimensions
    int cnt[kVec], mate[kVec], list[kVec];
    int laste[kMaxSites];            // last measured outcome per site
};
// LDS tables of the workgroup, read-only after the start: 2x2 gates, the
// monomial 4x4 gates (phase of each row, row that a column feeds) and the
// sites' offsets within a slot.
struct TableLds {
    double g1[G1_COUNT * 8];
    double g4ph[G4_COUNT * 8];
    int g4dst[G4_COUNT * 4];
    int soff[kMaxSites], shalf[kMaxSites];
};
typedef __attribute__((address_space(3))) WaveLds LWave;
typedef __attribute__((address_space(3))) TableLds LTables;


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
__device__ __forceinline__ int tile_overlaps(int tp, int tq, const f64x4& gr, const f64x4& gi,
                                             LWave* L, double floor2, double tol2) {
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
                                                  __HIP_MEMORY_SCOPE_WAVEFRONT);
            const int o1 = __hip_atomic_fetch_add(cnt + c, 1, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WAVEFRONT);
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

// The overlapping pairs of the 16 NVT vectors at V and their squared norms
// (L->nrm).  floor2 < 0 on entry: it becomes rel_floor times the norms' sum,
// which total receives.  Returns as not_orthogonal.
template <int NVT, typename DP>
__device__ __forceinline__ int wave_overlaps(DP V, int ld, int lp, int len, LWave* L,
                                             double rel_floor, double& floor2, double tol2,
                                             double& total) {
    const int lane = op_lane(), q = lane & 15;
    ldsd* nrm = L->nrm;
    f64x4 re, im;
    if constexpr (NVT == 2) {
        gram_tile(V, 1, 1, ld, lp, len, re, im);
        store_diagonal(re, nrm + 16);
    }
    gram_tile(V, 0, 0, ld, lp, len, re, im);
    store_diagonal(re, nrm);
    if (lane < 16 * NVT) L->cnt[lane] = 0;
    wave_order();
    if (floor2 < 0.0) {
        double sum = nrm[q];
        if constexpr (NVT == 2) sum += nrm[16 + q];
        total = row_sum(sum);
        floor2 = rel_floor * total;
    }
    int any = tile_overlaps(0, 0, re, im, L, floor2, tol2);
    if constexpr (NVT == 2) {
        gram_tile(V, 0, 1, ld, lp, len, re, im);
        any |= tile_overlaps(0, 1, re, im, L, floor2, tol2);
        gram_tile(V, 1, 1, ld, lp, len, re, im);
        any |= tile_overlaps(1, 1, re, im, L, floor2, tol2);
    }
    wave_order();
    if (__ballot(any) == 0ull) return 0;
    return __ballot(any & 2) != 0ull ? 2 : 1;
}

// Selection of the kept vectors (as select_kept): rank[t] is the position
// of vector 16 t + q among them, or -1; isq[t], sq[t] its 1/sigma and sigma.
template <int NVT>
__device__ __forceinline__ Kept wave_select(LWave* L, double tau2, int capb,
                                            int (&rank)[NVT], double (&isq)[NVT],
                                            double (&sq)[NVT], int nv) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const uint32_t colmask = 0x00010001u << q;
    const ldsd* nrm = L->nrm;
    double x[NVT], y[NVT][4];
    double mx = 0.0;
#pragma unroll
    for (int t = 0; t < NVT; ++t) {
        x[t] = sel_norm(nrm[16 * t + q]);
        mx = fmax(mx, x[t]);
#pragma unroll
        for (int r = 0; r < 4; ++r) y[t][r] = sel_norm(nrm[16 * t + g + 4 * r]);
    }
    mx = row_max(mx);
    Kept k;
    k.r = 0;
    k.want = 0;
    double kept = 0.0, dropped = 0.0;
#pragma unroll
    for (int t = 0; t < NVT; ++t) {
        const int v = 16 * t + q;
        // vectors ahead of v: larger, or equal and lower-numbered
        int rk = 0;
#pragma unroll
        for (int u = 0; u < NVT; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                rk += column_count(y[u][r] > x[t] || (y[u][r] == x[t] && 16 * u + g + 4 * r < v),
                                   colmask);
        const bool above = v < nv && (x[t] > tau2 * mx || rk == 0);
        const bool keep = above && rk < capb;
        k.want += __popc(static_cast<uint32_t>(__ballot(above)) & 0xFFFFu);
        k.r += __popc(static_cast<uint32_t>(__ballot(keep)) & 0xFFFFu);
        isq[t] = rsqrt_nr(x[t]);      // (of use where x is kept: never near 0)
        sq[t] = x[t] * isq[t];
        rank[t] = keep ? rk : -1;
        kept += keep ? x[t] : 0.0;
        dropped += keep ? 0.0 : x[t];
    }
    k.kept = row_sum(kept);
    k.dropped = row_sum(dropped);
    return k;
}

// Two-site update (as twosite_update) of sites whose theta has at most
// 16 NVT vectors of at most 32 elements; the vectors live at V (LDS, or the
// slot's scratch for 32 vectors of more than 16), vector v's real part at v ld
// and its imaginary part (ld - 1) / 2 further, with ld = 33 for at most 16
// elements and 65 above (odd: no bank conflicts between vectors).
//
// When every overlapping vector has one mate, which is practically always,
// one rotation per pair orthogonalises theta, and its factors are known in
// closed form: with x' = c x - conj(b) y and y' = c y + b x, theta = sum_v
// y_v conj(W[:, v])^T, so the centre factor's vector v has sigma_v c at its own
// index and sigma_v times -b (x') or conj(b) (y') at its mate's; no projection
// is computed.  A second round of rotations (or overlaps that are not a
// matching: round-robin sweeps) falls back on the projection of theta, put
// aside in `stash` (as at V), on the rotated vectors, four MFMAs per 16x16x4
// block.
template <typename T, int NVT, typename DP>
__device__ __forceinline__ bool wave_update(const Trunc P, LWave* L, const LTables* tab,
                                            SiteView<T> A, SiteView<T> B, int k, int dir, int gate_id,
                                            ShotAcc& acc, int cl, int cm, int cr, DP V,
                                            glbd* stash) {
    typedef __attribute__((address_space(1))) T gT;
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const int m = 2 * cl, n = 2 * cr;
    const int nv = dir ? n : m, len = dir ? m : n;
    const int lp = len <= 16 ? 16 : 32, ld = 2 * lp + 1;

    // ---- theta = G (A B): plain complex product of A's rows (a, i') and B's
    // columns (j', b) in 16x16 tiles (zero outside the shapes), each entry
    // times its phase to its row and column of theta under the monomial gate
    {
        const ldsi* dst = tab->g4dst + gate_id * 4;
        const ldsd* ph = tab->g4ph + gate_id * 8;
        for (int R0 = 0; R0 < m; R0 += 16) {
            for (int C0 = 0; C0 < n; C0 += 16) {
                f64x4 sr = {0.0, 0.0, 0.0, 0.0}, si = {0.0, 0.0, 0.0, 0.0};
                const int arow = R0 + q, bcol = C0 + q;
                const bool va = arow < m, vb = bcol < n;
                const auto load = [&](int kk, T& ar, T& ai, T& br, T& bi) {
                    const bool oa = va && kk < cm, ob = vb && kk < cm;
                    const uint32_t ia = oa ? arow * cm + kk : 0;
                    const uint32_t ib = ob ? kk * n + bcol : 0;
                    ar = at(A.re, ia);
                    ai = at(A.im, ia);
                    br = at(B.re, ib);
                    bi = at(B.im, ib);
                    ar = oa ? ar : T(0);
                    ai = oa ? ai : T(0);
                    br = ob ? br : T(0);
                    bi = ob ? bi : T(0);
                };
                const auto step4 = [&](double xr, double xi, double yr, double yi) {
                    sr = mfma(xr, yr, sr);
                    si = mfma(xr, yi, si);
                    sr = mfma(-xi, yi, sr);
                    si = mfma(xi, yr, si);
                };
                for (int k0 = 0; k0 < cm; k0 += 8) {
                    T ar, ai, br, bi, cr_, ci, dr, di;
                    load(k0 + g, ar, ai, br, bi);
                    if (k0 + 4 < cm) {
                        load(k0 + 4 + g, cr_, ci, dr, di);
                        step4(ar, ai, br, bi);
                        step4(cr_, ci, dr, di);
                    } else {
                        step4(ar, ai, br, bi);
                    }
                }
                // rows R0 + g + 4 r: one i' per lane, so one entry of the gate
                const int jp = bcol >= cr ? 1 : 0, b = bcol - (jp ? cr : 0);
                const int o = dst[2 * (g & 1) + jp];
                const double pr = ph[2 * o], pi = ph[2 * o + 1];
                // entries outside theta are zeros that fill the vectors
                const int trow = R0 + (vb ? (g & 2) + (o >> 1) : g);
                const int tcol = vb ? (o & 1) * cr + b : bcol;
                DP w = V + (dir ? tcol * ld + trow : trow * ld + tcol);
                const int step = dir ? 4 : 4 * ld;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    w[0] = pr * sr[r] - pi * si[r];
                    w[lp] = pr * si[r] + pi * sr[r];
                    w += step;
                }
            }
        }
    }
    wave_order();
    const double tau2 = P.tau * P.tau;
    const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                   : 8.0 * static_cast<double>(FLT_EPSILON);
    const double tol2 = tol * tol;
    double total, floor2 = -1.0;
    int over = wave_overlaps<NVT>(V, ld, lp, len, L, 1e-4 * tau2, floor2, tol2, total);

    double wc[NVT], wr[NVT], wi[NVT];   // W: own and mate's coefficient
    int mt[NVT];
#pragma unroll
    for (int t = 0; t < NVT; ++t) {
        wc[t] = 1.0;
        wr[t] = 0.0;
        wi[t] = 0.0;
        mt[t] = -1;
    }
    int sweeps = 0;
    bool closed = true;                 // the factors follow from one rotation
    ldsi* cnt = L->cnt;
    while (over && sweeps < 40) {
        if (closed && (over == 2 || sweeps > 0)) {
            // theta, put aside for the projection (from the rotated pairs by
            // the inverse rotation: theta_v = c y_v - w y_mate)
            closed = false;
#pragma unroll
            for (int t = 0; t < NVT; ++t) {
                const int v = 16 * t + q;
                const DP x = V + v * ld + g;
                const DP y = V + (mt[t] < 0 ? v : mt[t]) * ld + g;
                for (int e = 0; e < len; e += 4) {
                    stash[v * ld + g + e] = wc[t] * x[e] - (wr[t] * y[e] - wi[t] * y[lp + e]);
                    stash[v * ld + g + lp + e] =
                        wc[t] * x[lp + e] - (wr[t] * y[lp + e] + wi[t] * y[e]);
                }
            }
            wave_order();
        }
        if (over == 1) {
            const ldsd* nrm = L->nrm;
            const ldsd* gre = L->gre;
            const ldsd* gim = L->gim;
            const ldsi* mate = L->mate;
#pragma unroll
            for (int t = 0; t < NVT; ++t) {
                const int v = 16 * t + q;
                if (cnt[v]) {
                    const int u = mate[v];
                    const bool low = v < u;
                    const double gr = gre[v], gi = gim[v];
                    const double d = low ? nrm[u] - nrm[v] : nrm[v] - nrm[u];
                    const double g2 = gr * gr + gi * gi;
                    const double q1 = d * d + 4.0 * g2;
                    const double D = fabs(d) + q1 * rsqrt_nr(q1);
                    const double rq = rsqrt_nr(D * D + 4.0 * g2);
                    const double sg = (d >= 0.0 ? 2.0 : -2.0) * rq;
                    wc[t] = D * rq;
                    // own' = c own + w mate: w = -conj(b) for the lower
                    // vector, b for the upper one, b = (s/|g|) g
                    wr[t] = low ? -(sg * gr) : sg * gr;
                    wi[t] = sg * gi;
                    mt[t] = u;
                }
            }
            // element 4 s + g of every vector at a time (both of a pair
            // are read before either is written)
            for (int e = g; e < len; e += 4) {
                double nr[NVT], ni[NVT];
#pragma unroll
                for (int t = 0; t < NVT; ++t) {
                    const DP x = V + (16 * t + q) * ld + e;
                    const DP y = V + (mt[t] < 0 ? 16 * t + q : mt[t]) * ld + e;
                    const double y0 = y[0], y1 = y[lp];
                    nr[t] = wc[t] * x[0] + (wr[t] * y0 - wi[t] * y1);
                    ni[t] = wc[t] * x[lp] + (wr[t] * y1 + wi[t] * y0);
                }
                wave_order();
#pragma unroll
                for (int t = 0; t < NVT; ++t) {
                    if (cnt[16 * t + q]) {
                        DP x = V + (16 * t + q) * ld + e;
                        x[0] = nr[t];
                        x[lp] = ni[t];
                    }
                }
            }
            wave_order();
        } else {
            int nbad;
            [[clang::always_inline]] nbad = flagged_list<64>(cnt, nv, (ldsi*)L->list, (int*)nullptr);
            [[clang::always_inline]] jacobi_sweep<64>(V, V + lp, (ldsi*)L->list, nbad, len, ld, floor2, tol);
        }
        ++sweeps;
        double tot;
        over = wave_overlaps<NVT>(V, ld, lp, len, L, 0.0, floor2, tol2, tot);
    }
    if (over) acc.status |= MSC_SHOT_NOCONV;
    acc.sweeps += sweeps;

    // ---- selection and the new tensors
    const int capb = P.cap;
    int rank[NVT];
    double isq[NVT], sq[NVT];
    const Kept kp = wave_select<NVT>(L, tau2, capb, rank, isq, sq, nv);
    if (kp.want > capb && capb < P.chi_max) return false;
    const int r = kp.r;
    acc.disc += kp.dropped;
    if (kp.dropped > 1e-12 * total && r == capb) acc.status |= MSC_SHOT_CHI_CAP;
    const double renorm = rsqrt_nr(kp.kept);
    // isometric factor: A[k][e][c] = y_c[e] / sigma_c (dir 1), A[k+1][c][e]
    // (dir 0); centre factor: A[k+1][c][u] (dir 1), A[k][u][c] (dir 0)
    gT* Ure = dir ? A.re : B.re;
    gT* Uim = dir ? A.im : B.im;
    gT* Cre = dir ? B.re : A.re;
    gT* Cim = dir ? B.im : A.im;
    const int ue = dir ? r : 1, uc = dir ? 1 : n;     // element and vector strides
    const int cu = dir ? 1 : r, cc = dir ? n : 1;     // index and vector strides
#pragma unroll
    for (int t = 0; t < NVT; ++t) {
        if (rank[t] >= 0) {
            const DP x = V + (16 * t + q) * ld;
            for (int e = g; e < len; e += 4) {
                const uint32_t ix = e * ue + rank[t] * uc;
                at(Ure, ix) = T(x[e] * isq[t]);
                at(Uim, ix) = T(x[lp + e] * isq[t]);
            }
        }
    }
    if (closed) {
#pragma unroll
        for (int t = 0; t < NVT; ++t) {
            if (rank[t] >= 0) {
                const int v = 16 * t + q;
                const double sc = sq[t] * renorm;
                const T c0 = T(sc * wc[t]), c1 = T(sc * wr[t]), c2 = T(-(sc * wi[t]));
                // conj(W): own c, mate's conj(w)
                for (int u = g; u < nv; u += 4) {
                    const uint32_t ix = u * cu + rank[t] * cc;
                    at(Cre, ix) = u == v ? c0 : u == mt[t] ? c1 : T(0);
                    at(Cim, ix) = u == mt[t] ? c2 : T(0);
                }
            }
        }
    } else {
#pragma unroll
        for (int t = 0; t < NVT; ++t) {
            for (int u0 = 0; u0 < nv; u0 += 16) {
                // (u, v): theta_u . conj(y_v) over the elements
                f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
                const glbd* th = stash + (u0 + q) * ld + g;
                const DP y = V + (16 * t + q) * ld + g;
                for (int e = 0; e < len; e += 4) {
                    const double t0 = th[e], t1 = th[lp + e], y0 = y[e], y1 = y[lp + e];
                    re = mfma(t0, y0, re);
                    im = mfma(t1, y0, im);
                    re = mfma(t1, y1, re);
                    im = mfma(-t0, y1, im);
                }
                const double sc = isq[t] * renorm;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int u = u0 + g + 4 * x;
                    if (rank[t] >= 0 && u < nv) {
                        const uint32_t ix = u * cu + rank[t] * cc;
                        at(Cre, ix) = T(re[x] * sc);
                        at(Cim, ix) = T(im[x] * sc);
                    }
                }
            }
        }
    }
    if (lane == 0) L->chi[k + 1] = r;
    acc.chi_peak = max(acc.chi_peak, r);
    ++acc.n2q;
    const double dl = cl, dm = cm, dr = cr, dk = r;
    acc.flops += 32.0 * dl * dm * dr + 32.0 * dl * dl * dr + 32.0 * dk * dl * dr + 104.0 * dl * dl * dl;
    wave_order();
    return true;
}

// Centre move (as move_fast) between sites with at most 16 vectors on the
// bond, of at most 32 elements, and a neighbour of at most 32 elements per
// vector: element 4 s + g of the vectors and of the neighbour's rows (columns)
// in the lanes of vector q, which store both at the vector's rank.  Up to 16
// elements (KS = 4) everything is loaded once and stays in registers; above
// (KS = 0) the operands are read again for the stores.
template <typename T, int KS>
__device__ __forceinline__ bool wave_move(const Trunc P, LWave* L, SiteView<T> A,
                                          SiteView<T> B, int k, int dir, ShotAcc& acc, int cl,
                                          int cm, int cr) {
    typedef __attribute__((address_space(1))) T gT;
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const int nv = cm, len = dir ? 2 * cl : 2 * cr, w = dir ? 2 * cr : 2 * cl;
    gT* Xre = dir ? A.re : B.re;
    gT* Xim = dir ? A.im : B.im;
    gT* Nre = dir ? B.re : A.re;
    gT* Nim = dir ? B.im : A.im;
    // element e of vector v, element x of the neighbour's part v
    const int xe = dir ? cm : 1, xv = dir ? 1 : len;
    const int ne = dir ? 1 : cm, nvs = dir ? w : 1;
    constexpr int K = KS ? KS : 1;
    T x0[K], x1[K], y0[K], y1[K];
    f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    const auto gram_step = [&](T a, T b, bool in) {
        const double xr = in ? static_cast<double>(a) : 0.0, xi = in ? static_cast<double>(b) : 0.0;
        re = mfma(xr, xr, re);
        im = mfma(xr, xi, im);
        re = mfma(xi, xi, re);
        im = mfma(-xi, xr, im);
    };
    if constexpr (KS != 0) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int e = 4 * s + g;
            const uint32_t ix = q < nv && e < len ? q * xv + e * xe : 0;
            const uint32_t in = q < nv && e < w ? q * nvs + e * ne : 0;
            x0[s] = at(Xre, ix);
            x1[s] = at(Xim, ix);
            y0[s] = at(Nre, in);
            y1[s] = at(Nim, in);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (4 * s < len) gram_step(x0[s], x1[s], q < nv && 4 * s + g < len);
    } else {
#pragma unroll 2
        for (int e0 = 0; e0 < len; e0 += 4) {
            const bool in = q < nv && e0 + g < len;
            const uint32_t ix = in ? q * xv + (e0 + g) * xe : 0;
            gram_step(at(Xre, ix), at(Xim, ix), in);
        }
    }
    const double tau2 = P.tau * P.tau;
    const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                   : 8.0 * static_cast<double>(FLT_EPSILON);
    ldsd* nrm = L->nrm;
    store_diagonal(re, nrm);
    wave_order();
    const double nq = nrm[q];
    const double total = row_sum(nq), floor2 = 1e-4 * tau2 * total;
    bool over = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double a = nrm[g + 4 * r];
        const double g2 = re[r] * re[r] + im[r] * im[r];
        over |= g + 4 * r < q && a > floor2 && nq > floor2 && g2 > tol * tol * a * nq;
    }
    if (__ballot(over) != 0ull) return false;
    const int capb = P.cap;
    int rank[1];
    double isq[1], sq[1];
    const Kept kp = wave_select<1>(L, tau2, capb, rank, isq, sq, nv);
    const int r = kp.r;
    acc.disc += kp.dropped;
    if (kp.dropped > 1e-12 * total && r == capb) acc.status |= MSC_SHOT_CHI_CAP;
    const double renorm = rsqrt_nr(kp.kept);
    const int ue = dir ? r : 1, uv = dir ? 1 : len;
    const int me = dir ? 1 : r, mv = dir ? w : 1;
    const double is = isq[0], sc = sq[0] * renorm;
    if constexpr (KS != 0) {
        if (rank[0] >= 0) {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int e = 4 * s + g;
                if (e < len) {
                    const uint32_t ix = e * ue + rank[0] * uv;
                    at(Xre, ix) = T(static_cast<double>(x0[s]) * is);
                    at(Xim, ix) = T(static_cast<double>(x1[s]) * is);
                }
                if (e < w) {
                    const uint32_t ix = e * me + rank[0] * mv;
                    at(Nre, ix) = T(static_cast<double>(y0[s]) * sc);
                    at(Nim, ix) = T(static_cast<double>(y1[s]) * sc);
                }
            }
        }
    } else {
        // the stores permute (and, when vectors were dropped, pack) the
        // tensors in place: every element is read before any is written
        const auto rewrite = [&](gT* re_, gT* im_, int n, int se, int sv, int de, int dv, double f) {
            T a[8], b[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int e = 4 * s + g;
                const uint32_t ix = q < nv && e < n ? q * sv + e * se : 0;
                a[s] = at(re_, ix);
                b[s] = at(im_, ix);
            }
            wave_order();
            if (rank[0] >= 0) {
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int e = 4 * s + g;
                    if (e < n) {
                        const uint32_t ix = e * de + rank[0] * dv;
                        at(re_, ix) = T(static_cast<double>(a[s]) * f);
                        at(im_, ix) = T(static_cast<double>(b[s]) * f);
                    }
                }
            }
        };
        rewrite(Xre, Xim, len, xe, xv, ue, uv, is);
        rewrite(Nre, Nim, w, ne, nvs, me, mv, sc);
    }
    if (lane == 0) L->chi[k + 1] = r;
    wave_order();
    return true;
}

// Product swap (as OP_SWAPP) with the product site's bonds pl, pr at most 16
// and the neighbour's outer bond newb at most 16: psi from the rank-1 rho, M =
// sum_i conj(psi_i) P[:, i, :] formed in the lanes that hold P in operand
// layout, the neighbour folded into it by FP64 MFMAs, psi (x) I written to
// the neighbour's site.  No LDS.
template <typename T>
__device__ __forceinline__ void wave_pswap(LWave* L, SiteView<T> Pv, SiteView<T> Ov, int k, int side, int pl,
                           int pr, int newb) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    // side 1: out = O (2 newb x pl) . M (pl x pr), side 0: M (pl x pr) . O (pr x
    // 2 newb); the summed index is kk = 4 s + g, M's other index q
    const int nk = side ? pl : pr, nm = side ? pr : pl, no = 2 * newb;
    const int mk = side ? 2 * pr : 1, mq = side ? 1 : 2 * pr;     // strides in P
    const int ok = side ? 1 : no, oq = side ? pl : 1;             // strides in O
    T p0r[4], p0i[4], p1r[4], p1i[4], orr[4], oi[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (4 * s >= nk) break;
        const int kk = 4 * s + g;
        const uint32_t i0 = q < nm && kk < nk ? kk * mk + q * mq : 0;
        p0r[s] = at(Pv.re, i0);
        p0i[s] = at(Pv.im, i0);
        p1r[s] = at(Pv.re, i0 + pr);
        p1i[s] = at(Pv.im, i0 + pr);
    }
    const auto load_o = [&](int t) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (4 * s >= nk) break;
            const int kk = 4 * s + g, o = 16 * t + q;
            const uint32_t ix = o < no && kk < nk ? kk * ok + o * oq : 0;
            orr[s] = at(Ov.re, ix);
            oi[s] = at(Ov.im, ix);
        }
    };
    load_o(0);
    double r4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (4 * s >= nk) break;
        const bool in = q < nm && 4 * s + g < nk;
        p0r[s] = in ? p0r[s] : T(0);
        p0i[s] = in ? p0i[s] : T(0);
        p1r[s] = in ? p1r[s] : T(0);
        p1i[s] = in ? p1i[s] : T(0);
        const double x0r = p0r[s], x0i = p0i[s], x1r = p1r[s], x1i = p1i[s];
        r4[0] += x0r * x0r + x0i * x0i;
        r4[1] += x1r * x1r + x1i * x1i;
        r4[2] += x0r * x1r + x0i * x1i;     // rho01 = x0 conj(x1)
        r4[3] += x0i * x1r - x0r * x1i;
    }
    wave_sum4(r4);
    // psi, unit norm: the column of rho with the larger diagonal entry
    const bool one = r4[1] > r4[0];
    const double pn = one ? r4[1] : r4[0];
    const double pd = rsqrt_nr(pn * (r4[0] + r4[1]));
    const double s0r = (one ? r4[2] : pn) * pd, s0i = one ? r4[3] * pd : 0.0;
    const double s1r = (one ? pn : r4[2]) * pd, s1i = one ? 0.0 : -(r4[3] * pd);   // rho10 = conj(rho01)
    double mr[4], mi[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (4 * s >= nk) break;
        const double x0r = p0r[s], x0i = p0i[s], x1r = p1r[s], x1i = p1i[s];
        mr[s] = s0r * x0r + s0i * x0i + s1r * x1r + s1i * x1i;
        mi[s] = s0r * x0i - s0i * x0r + s1r * x1i - s1i * x1r;
    }
    for (int t = 0; 16 * t < no; ++t) {
        if (t > 0) load_o(t);
        f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (4 * s >= nk) break;
            const bool in = 16 * t + q < no && 4 * s + g < nk;
            const double xr = in ? static_cast<double>(orr[s]) : 0.0;
            const double xi = in ? static_cast<double>(oi[s]) : 0.0;
            // side 1: rows from O, columns from M; side 0 the other way
            const double ar = side ? xr : mr[s], ai = side ? xi : mi[s];
            const double br = side ? mr[s] : xr, bi = side ? mi[s] : xi;
            re = mfma(ar, br, re);
            im = mfma(ar, bi, im);
            re = mfma(-ai, bi, re);
            im = mfma(ai, br, im);
        }
        const int rows = side ? no : pl, cols = side ? pr : no;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int row = g + 4 * x + (side ? 16 * t : 0), col = q + (side ? 0 : 16 * t);
            if (row < rows && col < cols) {
                const uint32_t ix = row * cols + col;
                at(Pv.re, ix) = T(re[x]);
                at(Pv.im, ix) = T(im[x]);
            }
        }
    }
    // the unentangled qubit on the other site: psi (x) identity
    for (int row = g; row < no; row += 4) {        // (a, i)
        if (q < newb) {
            const bool diag = q == (row >> 1), i = row & 1;
            const uint32_t ix = row * newb + q;
            at(Ov.re, ix) = T(diag ? (i ? s1r : s0r) : 0.0);
            at(Ov.im, ix) = T(diag ? (i ? s1i : s0i) : 0.0);
        }
    }
    if (lane == 0) L->chi[k + 1] = newb;
    wave_order();
}

// The shots of one wavefront in its slot: each from its fork point (or from
// |0...0>) through the op stream to its result, op by op.  EXTRA compiles in
// checkpoint recording and segment reach.
template <typename T, bool EXTRA>
__device__ __forceinline__ void run_wave(const MpsArgs& P, LWave* L, const LTables* tab, int team) {
    typedef __attribute__((address_space(1))) T gT;
    const int lane = threadIdx.x & 63;
    const int N = P.n_sites;
    gT* slot = to_glb(static_cast<T*>(P.arena) + (size_t)team * P.slot_stride);
    glbd* scr = to_glb(P.scratch + (size_t)team * P.scratch_stride);
    const Trunc trunc{P.tau, P.chi_max, N > 1 ? min(P.chi_max, P.cap[1]) : 1};
    // (k is the same in every lane)
    const auto site = [&](int k) {
        SiteView<T> v;
        v.re = slot + uni(tab->soff[k]);
        v.im = v.re + uni(tab->shalf[k]);
        return v;
    };
    const auto chi = [&](int k) { return uni(L->chi[k]); };
    const int64_t n_run = P.n_dev ? min(*P.n_dev, P.n_shots) : P.n_shots;
    for (int64_t j = wave_fetch(P.next); j < n_run; j = wave_fetch(P.next)) {
        const int64_t it = P.perm ? P.perm[j] : j;
        const int64_t shot = P.shot_idx ? P.shot_idx[it] : it;
        if (shot < 0 || shot >= P.n_csr) {
            if (lane == 0) {
                msc_shot_result bad{};
                bad.rejected_at = -1;
                P.out[it] = bad;
            }
            continue;
        }
        ShotAcc acc;
        double p_acc = 1.0, infid = 0.0;
        int rej_at = -1;
        int64_t fcur = P.shot_off[shot];
        const int64_t fend = P.shot_off[shot + 1];
        // channel of the shot's next fault, loaded ahead of its op
        int next_ch = fcur < fend ? uni(P.chan[fcur]) : -1;
        int fcode = 0;                // code of the last channel read (three-qubit faults)
        bool alive = true, retried = false;
        int start = 0, jck = -1;
        int next_seg = 0;             // next segment whose reach is unwritten
        int meas_done = 0;            // measurements projected so far
        // forked at the read-out checkpoint: its dense tensors, read in place
        const gT* final_src = nullptr;
        int next_ck = 0;              // record mode: next checkpoint to take
        int64_t ck_pos = 0;           // record mode: elements written so far
        bool ck_full = false;
        if (P.ck_mode == 2) {
            // the last checkpoint of the noiseless run before the first fault
            const int navail = uni(*P.ck_avail);
            const int jj = fcur < fend ? next_ch / P.ck_k : P.n_ck - 1;
            jck = jj < navail ? jj : navail - 1;
        }
        if (jck >= 0) {
            const CkHdr& h = P.ck_hdr[jck];
            for (int k = lane; k <= N; k += 64) L->chi[k] = h.chi[k];
            for (int k = lane; k < N; k += 64) L->laste[k] = h.laste[k];
            wave_order();
            const gT* src = to_glb(static_cast<const T*>(P.ck_data)) + P.ck_off[jck];
            if (jck == P.n_ck - 1) {
                // before the read-out: the only op left reads one site
                final_src = src;
            } else {
                for (int k = 0; k < N; ++k) {
                    const int ne = chi(k) * 2 * chi(k + 1);
                    SiteView<T> v = site(k);
                    for (int i = lane; i < ne; i += 64) {
                        v.re[i] = src[i];
                        v.im[i] = src[ne + i];
                    }
                    src += 2 * ne;
                }
            }
            p_acc = h.p_acc;
            acc.disc = h.disc;
            acc.chi_peak = h.chi_peak;
            acc.status = h.status;
            start = uni(P.ck_op[jck]);
            meas_done = h.meas_done;
            if (EXTRA && P.surv) {
                // reach of the segments before the fork: the noiseless run's
                while (next_seg < P.n_seg && P.seg_meas[next_seg] < meas_done) {
                    if (lane == 0) P.surv[it * P.n_seg + next_seg] = P.ck_pm[P.seg_meas[next_seg]];
                    ++next_seg;
                }
            }
        } else {
            // ---- initial product state |0...0> (site k in lane k)
            for (int k = lane; k <= N; k += 64) L->chi[k] = 1;
            for (int k = lane; k < N; k += 64) {
                L->laste[k] = 0;
                gT* re = slot + tab->soff[k];
                gT* im = re + tab->shalf[k];
                re[0] = T(1);
                re[1] = T(0);
                im[0] = T(0);
                im[1] = T(0);
            }
        }
        wave_order();
        int ops_lo = 0, ops_hi = 0;   // op range held in LDS

        for (int oi = start; oi < P.n_ops && alive; ++oi) {
            if (oi >= ops_hi) {
                ops_lo = oi;
                ops_hi = min(P.n_ops, oi + kOps);
                if (lane < 4 * (ops_hi - ops_lo))
                    ((__attribute__((address_space(3))) int32_t*)L->ops)[lane] =
                        reinterpret_cast<const int32_t*>(P.ops + ops_lo)[lane];
                wave_order();
            }
            if (EXTRA && P.ck_mode == 1 && !ck_full && next_ck < P.n_ck && P.ck_op[next_ck] == oi) {
                // ---- record: the state before op oi, densely, site by site
                int64_t sz = 0;
                for (int k = 0; k < N; ++k) sz += 4 * (int64_t)chi(k) * chi(k + 1);
                if (ck_pos + sz <= P.ck_cap) {
                    gT* dst = to_glb(static_cast<T*>(P.ck_data)) + ck_pos;
                    for (int k = 0; k < N; ++k) {
                        const int ne = chi(k) * 2 * chi(k + 1);
                        SiteView<T> v = site(k);
                        for (int i = lane; i < ne; i += 64) {
                            dst[i] = v.re[i];
                            dst[ne + i] = v.im[i];
                        }
                        dst += 2 * ne;
                    }
                    CkHdr& h = P.ck_hdr[next_ck];
                    for (int k = lane; k <= N; k += 64) h.chi[k] = L->chi[k];
                    for (int k = lane; k < N; k += 64) h.laste[k] = L->laste[k];
                    if (lane == 0) {
                        h.p_acc = p_acc;
                        h.meas_done = meas_done;
                        h.disc = acc.disc;
                        h.chi_peak = acc.chi_peak;
                        h.status = acc.status;
                        P.ck_off[next_ck] = ck_pos;
                        *P.ck_avail = next_ck + 1;
                    }
                    ck_pos += sz;
                    ++next_ck;
                } else {
                    ck_full = true;
                }
            }
            const int kind = uni(L->ops[oi - ops_lo].kind), a = uni(L->ops[oi - ops_lo].a);
            const int b = uni(L->ops[oi - ops_lo].b), aux = uni(L->ops[oi - ops_lo].aux);
            bool twosite = kind == OP_G2;
            int gate_id = aux;
            if (kind == OP_MOVE) {
                const int cl = chi(a), cm = chi(a + 1), cr = chi(a + 2);
                const SiteView<T> A = site(a), B = site(a + 1);
                const bool fast = max(cl, cr) <= 8
                                      ? wave_move<T, 4>(trunc, L, A, B, a, b, acc, cl, cm, cr)
                                      : wave_move<T, 0>(trunc, L, A, B, a, b, acc, cl, cm, cr);
                if (!fast) {
                    twosite = true;
                    gate_id = G4_I;
                }
            } else if (kind == OP_SWAPP) {
                const int ps = a + b, os = a + 1 - b;
                wave_pswap<T>(L, site(ps), site(os), a, b, chi(ps), chi(ps + 1),
                              b ? chi(a) : chi(a + 2));
            } else if (kind == OP_G1 || kind == OP_FAULT || kind == OP_FAULT3 || kind == OP_RESET) {
                // ---- local 2x2 on one site (two for a two-qubit fault)
                int g0 = -1, g1 = -1;
                if (kind == OP_G1) {
                    g0 = aux;
                } else if (kind == OP_RESET) {
                    if (uni(L->laste[a]) == 1) g0 = G_X;
                } else if (kind == OP_FAULT3) {
                    const int x2 = (fcode >> 4) & 1, z2 = (fcode >> 5) & 1;
                    if (x2 | z2) g0 = (x2 && z2) ? G_Y : (x2 ? G_X : G_Z);
                } else {
                    int code = 0;
                    if (fcur < fend && next_ch == aux) {
                        code = uni(P.pauli[fcur]);
                        ++fcur;
                        next_ch = fcur < fend ? uni(P.chan[fcur]) : -1;
                    }
                    fcode = code;
                    const int x0 = code & 1, z0 = (code >> 1) & 1;
                    const int x1 = (code >> 2) & 1, z1 = (code >> 3) & 1;
                    if (x0 | z0) g0 = (x0 && z0) ? G_Y : (x0 ? G_X : G_Z);
                    if ((x1 | z1) && b >= 0) g1 = (x1 && z1) ? G_Y : (x1 ? G_X : G_Z);
                }
                for (int h = 0; h < 2; ++h) {
                    const int gid = h == 0 ? g0 : g1;
                    if (gid < 0) continue;
                    const int k = h == 0 ? a : b;
                    const ldsd* m = tab->g1 + gid * 8;
                    const double m0 = m[0], m1 = m[1], m2 = m[2], m3 = m[3];
                    const double m4 = m[4], m5 = m[5], m6 = m[6], m7 = m[7];
                    const SiteView<T> v = site(k);
                    const int cl = chi(k), cr = chi(k + 1);
                    const int l = op_lane(), q = l & 15, g = l >> 4;
                    if (q < cr) {
                        for (int x = g; x < cl; x += 4) {
                            const uint32_t i0 = x * 2 * cr + q, i1 = i0 + cr;
                            const double x0r = at(v.re, i0), x0i = at(v.im, i0), x1r = at(v.re, i1),
                                         x1i = at(v.im, i1);
                            at(v.re, i0) = T(m0 * x0r - m1 * x0i + m2 * x1r - m3 * x1i);
                            at(v.im, i0) = T(m0 * x0i + m1 * x0r + m2 * x1i + m3 * x1r);
                            at(v.re, i1) = T(m4 * x0r - m5 * x0i + m6 * x1r - m7 * x1i);
                            at(v.im, i1) = T(m4 * x0i + m5 * x0r + m6 * x1i + m7 * x1r);
                        }
                    }
                    wave_order();
                }
            } else if (kind == OP_MEAS) {
                const SiteView<T> v = site(a);
                const int cl = chi(a), cr = chi(a + 1);
                const int e = uni(P.expected[aux]);
                const int l = op_lane(), q = l & 15, g = l >> 4;
                double pe2 = 0.0, po2 = 0.0;          // squared norms of the two outcomes
                T xr[4], xi[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int x = 4 * t + g;
                    xr[t] = T(0);
                    xi[t] = T(0);
                    if (q < cr && x < cl) {
                        const uint32_t ie = (x * 2 + e) * cr + q, io = (x * 2 + 1 - e) * cr + q;
                        xr[t] = at(v.re, ie);
                        xi[t] = at(v.im, ie);
                        const double er = xr[t], ei = xi[t], fr = at(v.re, io), fi = at(v.im, io);
                        pe2 += er * er + ei * ei;
                        po2 += fr * fr + fi * fi;
                    }
                }
                pe2 = wave_sum(pe2);
                po2 = wave_sum(po2);
                const double tot = pe2 + po2;
                const double pe = tot > 0.0 ? pe2 / tot : 0.0;
                if (EXTRA && P.surv) {
                    // segments starting at or before this measurement
                    while (next_seg < P.n_seg && P.seg_meas[next_seg] <= aux) {
                        if (lane == 0) P.surv[it * P.n_seg + next_seg] = p_acc;
                        ++next_seg;
                    }
                }
                if (EXTRA && P.ck_mode == 1 && P.ck_pm && lane == 0) P.ck_pm[aux] = p_acc;
                if (!(pe >= P.tau_rej)) {
                    alive = false;
                    acc.status |= MSC_SHOT_REJECTED;
                    rej_at = aux;
                    p_acc = 0.0;
                    break;
                }
                p_acc *= pe;
                meas_done = aux + 1;
                const double sc = rsqrt_nr(pe2);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int x = 4 * t + g;
                    if (q < cr && x < cl) {
                        const uint32_t ie = (x * 2 + e) * cr + q, io = (x * 2 + 1 - e) * cr + q;
                        at(v.re, ie) = T(static_cast<double>(xr[t]) * sc);
                        at(v.im, ie) = T(static_cast<double>(xi[t]) * sc);
                        at(v.re, io) = T(0);
                        at(v.im, io) = T(0);
                    }
                }
                if (lane == 0) L->laste[a] = e;
                wave_order();
            } else if (kind == OP_FINAL) {
                SiteView<T> v = site(a);
                const int cl = chi(a), cr = chi(a + 1);
                if (final_src) {
                    // site a of the dense checkpoint: planes of chi_j 2 chi_j+1
                    // elements per site, real then imaginary
                    int64_t o = 0;
                    for (int k = 0; k < a; ++k) o += 4 * (int64_t)chi(k) * chi(k + 1);
                    v.re = const_cast<gT*>(final_src + o);
                    v.im = v.re + 2 * cl * cr;
                }
                double r[4] = {0.0, 0.0, 0.0, 0.0};   // r00, r11, Re r01, Im r01
                const int l = op_lane(), q = l & 15, g = l >> 4;
                if (q < cr) {
                    for (int x = g; x < cl; x += 4) {
                        const uint32_t i0 = x * 2 * cr + q, i1 = i0 + cr;
                        const double x0r = at(v.re, i0), x0i = at(v.im, i0), x1r = at(v.re, i1), x1i = at(v.im, i1);
                        r[0] += x0r * x0r + x0i * x0i;
                        r[1] += x1r * x1r + x1i * x1i;
                        r[2] += x0r * x1r + x0i * x1i;   // rho01 = x0 conj(x1)
                        r[3] += x0i * x1r - x0r * x1i;
                    }
                }
#pragma unroll
                for (int h = 0; h < 4; ++h) r[h] = wave_sum(r[h]);
                const double tr = r[0] + r[1];
                // f = |t0|^2 rho00 + |t1|^2 rho11 + 2 Re(conj(t0) t1 rho01)
                const double ctr = P.t0r * P.t1r + P.t0i * P.t1i;   // conj(t0) t1
                const double cti = P.t0r * P.t1i - P.t0i * P.t1r;
                const double f = ((P.t0r * P.t0r + P.t0i * P.t0i) * r[0] +
                                  (P.t1r * P.t1r + P.t1i * P.t1i) * r[1] +
                                  2.0 * (ctr * r[2] - cti * r[3])) / tr;
                infid = fmax(0.0, 1.0 - f);
            }
            if (twosite) {
                const int cl = chi(a), cm = chi(a + 1), cr = chi(a + 2);
                const int nv = 2 * (b ? cr : cl), len = 2 * (b ? cl : cr);
                const SiteView<T> A = site(a), B = site(a + 1);
                bool ok;
                if (nv <= 16)
                    ok = wave_update<T, 1>(trunc, L, tab, A, B, a, b, gate_id, acc, cl, cm, cr,
                                           (ldsd*)L->work, scr);
                else if (len <= 16)
                    ok = wave_update<T, 2>(trunc, L, tab, A, B, a, b, gate_id, acc, cl, cm, cr,
                                           (ldsd*)L->work, scr);
                else
                    ok = wave_update<T, 2>(trunc, L, tab, A, B, a, b, gate_id, acc, cl, cm, cr,
                                           scr + kStash, scr);
                if (!ok) {
                    // a larger slot is needed: the shot is queued for the
                    // workgroup kernel, which runs it again from its start
                    if (lane == 0) P.retry_list[atomicAdd(P.retry_count, 1)] = it;
                    retried = true;
                    break;
                }
            }
        }
        if (lane == 0 && !retried) {
            if (EXTRA && P.surv)
                for (int s = next_seg; s < P.n_seg; ++s) P.surv[it * P.n_seg + s] = p_acc;
            msc_shot_result res;
            res.p_acc = p_acc;
            res.infid = alive ? infid : 0.0;
            res.disc_weight = acc.disc;
            res.chi_peak = acc.chi_peak;
            res.status = acc.status | (alive ? MSC_SHOT_DONE : 0);
            res.rejected_at = rej_at;
            res.fail = (alive && p_acc > 0.0 && infid > P.tau_fail) ? 1 : 0;
            res.n2q = acc.n2q;
            res.flops = acc.flops;
            res.sweeps = acc.sweeps;
            P.out[it] = res;
        }
        wave_order();
    }
}

template <typename T, bool EXTRA>
__global__ __launch_bounds__(NT, 3) void mps_fast_wave_kernel(MpsArgs P) {
    __shared__ __align__(16) WaveLds s_wave[NW];
    __shared__ __align__(16) TableLds s_tab;
    const int tid = threadIdx.x;
    for (int k = tid; k < P.n_sites; k += NT) {
        s_tab.soff[k] = static_cast<int>(P.site_off[k]);
        s_tab.shalf[k] = static_cast<int>(P.site_half[k]);
    }
    for (int i = tid; i < G1_COUNT * 8; i += NT) s_tab.g1[i] = P.g1[i];
    if (tid < G4_COUNT * 4) {
        // the nonzero of each row of each monomial 4x4 gate
        const double* m = P.g4 + (tid >> 2) * 32 + (tid & 3) * 8;
        int src = 0;
        for (int j = 1; j < 4; ++j)
            if (fabs(m[2 * j]) + fabs(m[2 * j + 1]) > fabs(m[2 * src]) + fabs(m[2 * src + 1])) src = j;
        s_tab.g4dst[(tid & ~3) + src] = tid & 3;
        s_tab.g4ph[2 * tid] = m[2 * src];
        s_tab.g4ph[2 * tid + 1] = m[2 * src + 1];
    }
    __syncthreads();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    run_wave<T, EXTRA>(P, (LWave*)(s_wave + w), (LTables*)&s_tab, blockIdx.x * NW + w);
}

}  // namespace

int mps_fast_wave_blocks_per_cu(int precision) {
    int b = 0;
    hipError_t e = precision == MSC_FP64
                       ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                             &b, mps_fast_wave_kernel<double, true>, NT, 0)
                       : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                             &b, mps_fast_wave_kernel<float, true>, NT, 0);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return b < 1 ? 1 : b;
}

hipError_t launch_mps_fast_wave(int precision, const MpsArgs& a, int grid, hipStream_t s) {
    static_assert(kWaveTeams == NW, "one team per wavefront");
    if (!a.next || !a.retry_count || !a.retry_list || a.calibrate || a.state ||
        a.scratch_stride < kStash + 32 * 65)
        return hipErrorInvalidValue;
    const bool extra = a.surv != nullptr || a.ck_mode == 1;
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(NT), 0, s, a);
        return hipGetLastError();
    };
    if (precision == MSC_FP64)
        return extra ? go(mps_fast_wave_kernel<double, true>) : go(mps_fast_wave_kernel<double, false>);
    return extra ? go(mps_fast_wave_kernel<float, true>) : go(mps_fast_wave_kernel<float, false>);
}

}  // namespace msc
