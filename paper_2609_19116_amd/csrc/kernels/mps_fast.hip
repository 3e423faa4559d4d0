// Shot kernels on the matrix cores, by the bond cap of their slots:
//   mps_fast_wave_kernel    at most 16: one shot per wavefront, four per
//                           workgroup, three workgroups per CU;
//   mps_fast_mid_kernel     at most 32: one shot per wavefront, seven per
//                           workgroup and CU;
//   mps_fast_group_kernel   at most 128: one shot per workgroup of eight
//                           wavefronts and CU.  Wavefront 0 leads: it runs the
//                           op stream and every op of bonds up to 16 alone and
//                           hands the wider two-site ops to the team (wide,
//                           follow).
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
// circuit (p = 1e-3, FP32) 138.8 -> 76.9 ms a batch, 1000 shots (one shot's
// latency) 36.3 -> 17.0 ms, 65536 17-qubit shots in FP64 64.7 -> 37.9 ms.  Per
// batch the vector instructions fell from 6.0e10 to 2.2e10 and the LDS
// instructions from 5.7e9 to 1.4e9; the matrix cores are busy 26 % of the
// time.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cstdint>

#include "kernels.h"
#include "mps_common.h"
#include "mps_mfma.h"

namespace msc {
namespace {

// Truncation of the factorisations: keep sigma > tau * sigma_0, at most cap
// vectors (the slot's bond cap, or chi_max below it).  Weight dropped with `full`
// vectors kept counts as cut by the bond cap: chi_max, as in the workgroup
// kernel, and in slots of cap 16 the slot's, as in the wavefront kernel.  (A
// slot's own cap cuts nothing: a shot that needs more leaves it.)
struct Trunc {
    double tau;
    int chi_max, cap, full;
};

constexpr int kOps = 16;             // op descriptors held at a time
constexpr int kStash = 32 * 65;      // doubles: theta put aside in the slot's scratch

// LDS of one shot (one base address, constant offsets): WORK doubles of
// work area (the vectors of a factorisation), per-vector arrays for VEC
// vectors, the shot's bonds and outcomes.
template <int VEC, int WORK>
struct ShotLds {
    static constexpr int kVec = VEC, kWork = WORK;
    double work[WORK];
    double nrm[VEC], gre[VEC], gim[VEC];
    DevOp ops[kOps];
    int chi[kMaxSites + 4];          // bond dimensions
    int cnt[VEC], mate[VEC], list[VEC];
    int laste[kMaxSites];            // last measured outcome per site
};
// The same for shots whose wider ops run by a team of NWT wavefronts: the
// rotations (wc, wr, wi, pair) and ranks of all vectors, and the team's
// partial results and command.
template <int VEC, int WORK, int NWT>
struct TeamLds : ShotLds<VEC, WORK> {
    double wc[VEC], wr[VEC], wi[VEC];
    double red[NWT * 4];
    int pair[VEC], rank[VEC];
    int flag[NWT];
    int cmd[4];
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
typedef __attribute__((address_space(3))) TableLds LTables;
// one wavefront, slots of bond cap 16: 32 vectors of 16 elements, or 16 of 32
typedef ShotLds<32, 32 * 33> WaveLds;


// The overlapping pairs of the 16 NVT vectors at V and their squared norms
// (L->nrm).  floor2 < 0 on entry: it becomes rel_floor times the norms' sum,
// which total receives.  Returns as not_orthogonal.
template <int NVT, typename DP, typename LW>
__device__ __forceinline__ int wave_overlaps(DP V, int ld, int lp, int len, LW* L,
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
template <int NVT, typename LW>
__device__ __forceinline__ Kept wave_select(LW* L, double tau2, int capb,
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

// The flops that the records count for an update (the contraction, the Gram
// matrix, a projection and an eigen-decomposition at its shapes) are those of a
// general factorisation, the unit in which all shot kernels count; the closed
// form below needs neither of the last two, two thirds of the count at equal
// bonds, and a wide centre move that counts as an update computes the Gram
// matrix alone.
//
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
template <typename T, int NVT, typename DP, typename LW>
__device__ __forceinline__ bool wave_update(const Trunc P, LW* L, const LTables* tab,
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
    if (kp.dropped > 1e-12 * total && r == P.full) acc.status |= MSC_SHOT_CHI_CAP;
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
// in the lanes of vector q, which store both at the vector's rank.
template <typename T, typename LW>
__device__ __forceinline__ bool wave_move(const Trunc P, LW* L, SiteView<T> A,
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
    f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    const auto gram_step = [&](T a, T b, bool in) {
        const double xr = in ? static_cast<double>(a) : 0.0, xi = in ? static_cast<double>(b) : 0.0;
        re = mfma(xr, xr, re);
        im = mfma(xr, xi, im);
        re = mfma(xi, xi, re);
        im = mfma(-xi, xr, im);
    };
#pragma unroll 2
    for (int e0 = 0; e0 < len; e0 += 4) {
        const bool in = q < nv && e0 + g < len;
        const uint32_t ix = in ? q * xv + (e0 + g) * xe : 0;
        gram_step(at(Xre, ix), at(Xim, ix), in);
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
    if (kp.dropped > 1e-12 * total && r == P.full) acc.status |= MSC_SHOT_CHI_CAP;
    const double renorm = rsqrt_nr(kp.kept);
    const int ue = dir ? r : 1, uv = dir ? 1 : len;
    const int me = dir ? 1 : r, mv = dir ? w : 1;
    const double is = isq[0], sc = sq[0] * renorm;
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
    if (lane == 0) L->chi[k + 1] = r;
    wave_order();
    return true;
}

// Selection among at most 8 vectors (as wave_select): lanes q and q + 8 both
// answer for vector q mod 8, so the sums over a row count every vector twice
// and are halved (exactly).
template <typename LW>
__device__ __forceinline__ Kept wave_select8(LW* L, double tau2, int capb, int& rank, double& isq,
                                             double& sq, int nv) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4, v = q & 7;
    const uint32_t colmask = 0x00010001u << q;
    const ldsd* nrm = L->nrm;
    const double x = sel_norm(nrm[v]), y0 = sel_norm(nrm[g]), y1 = sel_norm(nrm[g + 4]);
    const double mx = row_max(x);
    const int rk = column_count(y0 > x || (y0 == x && g < v), colmask) +
                   column_count(y1 > x || (y1 == x && g + 4 < v), colmask);
    const bool above = v < nv && (x > tau2 * mx || rk == 0);
    const bool keep = above && rk < capb;
    Kept k;
    k.want = __popc(static_cast<uint32_t>(__ballot(above)) & 0xFFu);
    k.r = __popc(static_cast<uint32_t>(__ballot(keep)) & 0xFFu);
    isq = rsqrt_nr(x);            // (of use where x is kept: never near 0)
    sq = x * isq;
    rank = keep ? rk : -1;
    k.kept = 0.5 * row_sum(keep ? x : 0.0);
    k.dropped = 0.5 * row_sum(keep ? 0.0 : x);
    return k;
}

// Centre move (as wave_move) between bonds of at most 8: lane column q holds one
// plane of vector q mod 8, the real one for q < 8, so one product of the 16
// columns with themselves is the Gram matrix's four real parts (re = RR + II
// and im = RI - IR, brought together by a rotation of the rows by 8), and
// every load, scale and store handles one number instead of two.  49 qubits,
// 2^19 shots: 80.6 -> 76.9 ms; 1000 17-qubit shots 2.83 -> 2.71 ms.  (Vectors of
// up to 32 elements over such a bond gained nothing: the guards of their eight
// loads cost a lone shot what the products saved.)
template <typename T, typename LW>
__device__ __forceinline__ bool wave_move8(const Trunc P, LW* L, SiteView<T> A, SiteView<T> B, int k,
                                           int dir, ShotAcc& acc, int cl, int cm, int cr) {
    typedef __attribute__((address_space(1))) T gT;
    const int lane = op_lane(), q = lane & 15, g = lane >> 4, v = q & 7;
    const int nv = cm, len = dir ? 2 * cl : 2 * cr, w = dir ? 2 * cr : 2 * cl;
    gT* X = dir ? A.re : B.re;
    gT* N = dir ? B.re : A.re;
    // this lane's plane of either site
    const uint32_t px = q < 8 ? 0 : static_cast<uint32_t>((dir ? A.im : B.im) - X);
    const uint32_t pn = q < 8 ? 0 : static_cast<uint32_t>((dir ? B.im : A.im) - N);
    const int xe = dir ? cm : 1, xv = dir ? 1 : len;
    const int ne = dir ? 1 : cm, nvs = dir ? w : 1;
    constexpr int KS = 4;
    T x[KS], y[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int e = 4 * s + g;
        x[s] = at(X, v < nv && e < len ? px + v * xv + e * xe : 0);
        y[s] = at(N, v < nv && e < w ? pn + v * nvs + e * ne : 0);
    }
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < KS; ++s)
        if (4 * s < len) {
            const double t = v < nv && 4 * s + g < len ? static_cast<double>(x[s]) : 0.0;
            d = mfma(t, t, d);
        }
    // rows g and g + 4 of columns q < 8
    const double re0 = d[0] + dpp_move<0x128>(d[2]), re1 = d[1] + dpp_move<0x128>(d[3]);
    const double im0 = dpp_move<0x128>(d[0]) - d[2], im1 = dpp_move<0x128>(d[1]) - d[3];
    const double tau2 = P.tau * P.tau;
    const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                   : 8.0 * static_cast<double>(FLT_EPSILON);
    ldsd* nrm = L->nrm;
    if (q < 8 && g == (q & 3)) nrm[q] = (q & 4) ? re1 : re0;
    wave_order();
    const double nq = nrm[v];
    const double total = 0.5 * row_sum(nq), floor2 = 1e-4 * tau2 * total;
    const double a0 = nrm[g], a1 = nrm[g + 4];
    const auto overlaps = [&](double a, double re, double im, int p) {
        return p < q && q < 8 && a > floor2 && nq > floor2 &&
               re * re + im * im > tol * tol * a * nq;
    };
    if (__ballot(overlaps(a0, re0, im0, g) || overlaps(a1, re1, im1, g + 4)) != 0ull) return false;
    const int capb = P.cap;
    int rank;
    double is, sc;
    const Kept kp = wave_select8(L, tau2, capb, rank, is, sc, nv);
    const int r = kp.r;
    acc.disc += kp.dropped;
    if (kp.dropped > 1e-12 * total && r == P.full) acc.status |= MSC_SHOT_CHI_CAP;
    sc *= rsqrt_nr(kp.kept);
    const int ue = dir ? r : 1, uv = dir ? 1 : len;
    const int me = dir ? 1 : r, mv = dir ? w : 1;
    if (rank >= 0) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int e = 4 * s + g;
            if (e < len) at(X, px + e * ue + rank * uv) = T(static_cast<double>(x[s]) * is);
            if (e < w) at(N, pn + e * me + rank * mv) = T(static_cast<double>(y[s]) * sc);
        }
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
template <typename T, typename LW>
__device__ __forceinline__ void wave_pswap(LW* L, SiteView<T> Pv, SiteView<T> Ov, int k, int side, int pl,
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

// ---------------------------------------------------------------------------
// The same ops for wider sites, by a team of NWT wavefronts (one shot per
// team): 16x16 tiles dealt to the wavefronts, FP64 MFMA.  Vectors of a
// factorisation live at V with a stride of 2 lp + 1 doubles, lp their length
// rounded up to 16 (LDS when they fit in the work area, else the slot's
// scratch).  Every wavefront returns the same values.

template <int NWT>
__device__ __forceinline__ void team_sync() {
    if constexpr (NWT == 1) wave_order();
    else __syncthreads();
}
template <int NWT>
__device__ __forceinline__ int team_wave() {
    if constexpr (NWT == 1) return 0;
    else return uni(threadIdx.x >> 6);
}

// OR of a per-lane value's bits 0 and 1 over the team (synchronises).
template <int NWT, typename LW>
__device__ __forceinline__ int team_or(LW* L, int v) {
    const int b = (__ballot(v & 1) ? 1 : 0) | (__ballot(v & 2) ? 2 : 0);
    if constexpr (NWT == 1) {
        wave_order();
        return b;
    } else {
        if ((threadIdx.x & 63) == 0) L->flag[threadIdx.x >> 6] = b;
        __syncthreads();
        int r = 0;
        for (int i = 0; i < NWT; ++i) r |= L->flag[i];
        return uni(r);
    }
}

// Sums of four wave-uniform values over the team's wavefronts, in order
// (synchronises, twice: red may be reused at once).
template <int NWT, typename LW>
__device__ __forceinline__ void team_add4(LW* L, double (&v)[4]) {
    if constexpr (NWT > 1) {
        const int w = team_wave<NWT>();
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) L->red[4 * w + j] = v[j];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = 0.0;
        for (int i = 0; i < NWT; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] += L->red[4 * i + j];
        }
        __syncthreads();
    }
}

// Sum of the squared norms nrm[0 .. n), the same order in every wavefront.
template <typename LW>
__device__ __forceinline__ double norm_total(LW* L, int n) {
    double t = 0.0;
    for (int i = op_lane(); i < n; i += 64) t += L->nrm[i];
    return wave_sum(t);
}

// Tile i of the upper triangle above the diagonal of n x n tiles.
__device__ __forceinline__ void upper_tile(int i, int n, int& tp, int& tq) {
    tp = 0;
    while (i >= n - 1 - tp) {
        i -= n - 1 - tp;
        ++tp;
    }
    tq = tp + 1 + i;
}

// wave_overlaps over the team, for the nvt Gram tiles a functor computes:
// gram(tp, tq, re, im).
template <int NWT, typename LW, typename F>
__device__ __forceinline__ int team_overlaps(F gram, int nvt, LW* L, double rel_floor,
                                             double& floor2, double tol2, double& total) {
    const int w = team_wave<NWT>();
    f64x4 re, im;
    for (int t = w; t < nvt; t += NWT) {
        gram(t, t, re, im);
        store_diagonal(re, (ldsd*)L->nrm + 16 * t);
    }
    for (int i = (int)threadIdx.x % (64 * NWT); i < 16 * nvt; i += 64 * NWT) L->cnt[i] = 0;
    team_sync<NWT>();
    if (floor2 < 0.0) {
        total = norm_total(L, 16 * nvt);
        floor2 = rel_floor * total;
    }
    constexpr int kScope = NWT == 1 ? __HIP_MEMORY_SCOPE_WAVEFRONT : __HIP_MEMORY_SCOPE_WORKGROUP;
    int any = 0;
    // the diagonal tiles (a wavefront's last one is still in registers)
    for (int t = w; t < nvt; t += NWT) {
        if (nvt > NWT) gram(t, t, re, im);
        any |= tile_overlaps<kScope>(t, t, re, im, L, floor2, tol2);
    }
    const int noff = nvt * (nvt - 1) / 2;
    for (int i = w; i < noff; i += NWT) {
        int tp, tq;
        upper_tile(i, nvt, tp, tq);
        gram(tp, tq, re, im);
        any |= tile_overlaps<kScope>(tp, tq, re, im, L, floor2, tol2);
    }
    const int r = team_or<NWT>(L, any);
    return r & 2 ? 2 : r;
}

// Selection of the kept vectors (as wave_select): rank[v] in LDS.
template <int NWT, typename LW>
__device__ __forceinline__ Kept team_select(LW* L, double tau2, int capb, int nv) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const uint32_t colmask = 0x00010001u << q;
    const int nvt = (nv + 15) >> 4, w = team_wave<NWT>();
    double mx = 0.0;
    for (int i = lane; i < 16 * nvt; i += 64) mx = fmax(mx, sel_norm(L->nrm[i]));
    mx = wave_max(mx);
    double v4[4] = {0.0, 0.0, 0.0, 0.0};    // kept, dropped, count kept, above
    for (int t = w; t < nvt; t += NWT) {
        const int v = 16 * t + q;
        const double x = sel_norm(L->nrm[v]);
        int rk = 0;
        for (int u = 0; u < nvt; ++u) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double y = sel_norm(L->nrm[16 * u + g + 4 * r]);
                rk += column_count(y > x || (y == x && 16 * u + g + 4 * r < v), colmask);
            }
        }
        const bool above = v < nv && (x > tau2 * mx || rk == 0);
        const bool keep = above && rk < capb;
        if (g == 0) L->rank[v] = keep ? rk : -1;
        v4[0] += row_sum(keep ? x : 0.0);
        v4[1] += row_sum(keep ? 0.0 : x);
        v4[2] += __popc(static_cast<uint32_t>(__ballot(keep)) & 0xFFFFu);
        v4[3] += __popc(static_cast<uint32_t>(__ballot(above)) & 0xFFFFu);
    }
    team_add4<NWT>(L, v4);
    wave_order();
    Kept k;
    k.kept = v4[0];
    k.dropped = v4[1];
    k.r = uni(static_cast<int>(v4[2] + 0.5));
    k.want = uni(static_cast<int>(v4[3] + 0.5));
    return k;
}

// What a wide op did, for the shot's record.
struct WideOp {
    bool ok;           // false: the slot's bond cap is too small, nothing written
    bool fast;         // centre move: false if vectors overlap, nothing written
    int r, sweeps, status;
    double dropped;
};

// Two-site update (as wave_update).
template <typename T, int NWT, typename LW, typename DP>
__device__ __forceinline__ WideOp team_update(const Trunc P, LW* L, const LTables* tab,
                                              SiteView<T> A, SiteView<T> B, int dir, int gate_id,
                                              int cl, int cm, int cr, DP V, glbd* stash) {
    typedef __attribute__((address_space(1))) T gT;
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const int w = team_wave<NWT>();
    const int m = 2 * cl, n = 2 * cr;
    const int nv = dir ? n : m, len = dir ? m : n;
    const int lp = (len + 15) & ~15, ld = 2 * lp + 1;
    const int nvt = (nv + 15) >> 4;
    WideOp out{true, true, 0, 0, 0, 0.0};

    // ---- theta = G (A B)
    const int rt = (m + 15) >> 4, ct = (n + 15) >> 4;
    for (int tile = w; tile < rt * ct; tile += NWT) {
        const int tr = tile / ct, R0 = 16 * tr, C0 = 16 * (tile - tr * ct);
        f64x4 sr = {0.0, 0.0, 0.0, 0.0}, si = {0.0, 0.0, 0.0, 0.0};
        const int arow = R0 + q, bcol = C0 + q;
        const bool va = arow < m, vb = bcol < n;
#pragma unroll 4
        for (int k0 = 0; k0 < cm; k0 += 4) {
            const int kk = k0 + g;
            const bool oa = va && kk < cm, ob = vb && kk < cm;
            const uint32_t ia = oa ? arow * cm + kk : 0, ib = ob ? kk * n + bcol : 0;
            const T ar = at(A.re, ia), ai = at(A.im, ia), br = at(B.re, ib), bi = at(B.im, ib);
            const double xr = oa ? ar : T(0), xi = oa ? ai : T(0);
            const double yr = ob ? br : T(0), yi = ob ? bi : T(0);
            sr = mfma(xr, yr, sr);
            si = mfma(xr, yi, si);
            sr = mfma(-xi, yi, sr);
            si = mfma(xi, yr, si);
        }
        const int jp = bcol >= cr ? 1 : 0, b = bcol - (jp ? cr : 0);
        const int o = tab->g4dst[gate_id * 4 + 2 * (g & 1) + jp];
        const double pr = tab->g4ph[gate_id * 8 + 2 * o], pi = tab->g4ph[gate_id * 8 + 2 * o + 1];
        const int trow = R0 + (vb ? (g & 2) + (o >> 1) : g);
        const int tcol = vb ? (o & 1) * cr + b : bcol;
        DP x = V + (dir ? tcol * ld + trow : trow * ld + tcol);
        const int step = dir ? 4 : 4 * ld;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            x[0] = pr * sr[r] - pi * si[r];
            x[lp] = pr * si[r] + pi * sr[r];
            x += step;
        }
    }
    for (int v = (int)threadIdx.x % (64 * NWT); v < 16 * nvt; v += 64 * NWT) {
        L->wc[v] = 1.0;
        L->wr[v] = 0.0;
        L->wi[v] = 0.0;
        L->pair[v] = -1;
    }
    team_sync<NWT>();
    const double tau2 = P.tau * P.tau;
    const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                   : 8.0 * static_cast<double>(FLT_EPSILON);
    const double tol2 = tol * tol;
    const auto gram = [&](int tp, int tq, f64x4& re, f64x4& im) {
        gram_tile(V, tp, tq, ld, lp, len, re, im);
    };
    double total, floor2 = -1.0;
    int over = team_overlaps<NWT>(gram, nvt, L, 1e-4 * tau2, floor2, tol2, total);
    bool closed = true;
    while (over && out.sweeps < 40) {
        if (closed && (over == 2 || out.sweeps > 0)) {
            // theta, put aside for the projection (as in wave_update)
            closed = false;
            for (int t = w; t < nvt; t += NWT) {
                const int v = 16 * t + q, u = L->pair[v];
                const double c = L->wc[v], br = L->wr[v], bi = L->wi[v];
                const DP x = V + v * ld + g;
                const DP y = V + (u < 0 ? v : u) * ld + g;
                for (int e = 0; e < len; e += 4) {
                    stash[v * ld + g + e] = c * x[e] - (br * y[e] - bi * y[lp + e]);
                    stash[v * ld + g + lp + e] = c * x[lp + e] - (br * y[lp + e] + bi * y[e]);
                }
            }
            team_sync<NWT>();
        }
        if (over == 1) {
            // each pair by the lanes of its lower-numbered vector
            for (int t = w; t < nvt; t += NWT) {
                const int v = 16 * t + q;
                const int u = L->cnt[v] ? (int)L->mate[v] : -1;
                if (u > v) {
                    const double gr = L->gre[v], gi = L->gim[v];
                    const double d = L->nrm[u] - L->nrm[v];
                    const double g2 = gr * gr + gi * gi;
                    const double q1 = d * d + 4.0 * g2;
                    const double D = fabs(d) + q1 * rsqrt_nr(q1);
                    const double rq = rsqrt_nr(D * D + 4.0 * g2);
                    const double sg = (d >= 0.0 ? 2.0 : -2.0) * rq;
                    // x' = c x - conj(b) y, y' = c y + b x
                    const double c = D * rq, br = sg * gr, bi = sg * gi;
                    if (g == 0) {
                        L->wc[v] = c;
                        L->wc[u] = c;
                        L->wr[v] = -br;
                        L->wr[u] = br;
                        L->wi[v] = bi;
                        L->wi[u] = bi;
                        L->pair[v] = u;
                        L->pair[u] = v;
                    }
                    DP x = V + v * ld;
                    DP y = V + u * ld;
#pragma unroll 2
                    for (int e = g; e < len; e += 4) {
                        const double x0 = x[e], x1 = x[lp + e], y0 = y[e], y1 = y[lp + e];
                        x[e] = c * x0 - (br * y0 + bi * y1);
                        x[lp + e] = c * x1 - (br * y1 - bi * y0);
                        y[e] = c * y0 + (br * x0 - bi * x1);
                        y[lp + e] = c * y1 + (br * x1 + bi * x0);
                    }
                }
            }
        } else if (w == 0) {
            int nbad;
            [[clang::always_inline]] nbad = flagged_list<64>((ldsi*)L->cnt, nv, (ldsi*)L->list, (int*)nullptr);
            [[clang::always_inline]] jacobi_sweep<64>(V, V + lp, (ldsi*)L->list, nbad, len, ld, floor2, tol);
        }
        team_sync<NWT>();
        ++out.sweeps;
        double tot;
        over = team_overlaps<NWT>(gram, nvt, L, 0.0, floor2, tol2, tot);
    }
    if (over) out.status |= MSC_SHOT_NOCONV;

    // ---- selection and the new tensors
    const Kept kp = team_select<NWT>(L, tau2, P.cap, nv);
    if (kp.want > P.cap && P.cap < P.chi_max) {
        out.ok = false;
        return out;
    }
    const int r = kp.r;
    out.r = r;
    out.dropped = kp.dropped;
    if (kp.dropped > 1e-12 * total && r == P.full) out.status |= MSC_SHOT_CHI_CAP;
    const double renorm = rsqrt_nr(kp.kept);
    gT* Ure = dir ? A.re : B.re;
    gT* Uim = dir ? A.im : B.im;
    gT* Cre = dir ? B.re : A.re;
    gT* Cim = dir ? B.im : A.im;
    const int ue = dir ? r : 1, uc = dir ? 1 : n;     // element and vector strides
    const int cu = dir ? 1 : r, cc = dir ? n : 1;     // index and vector strides
    for (int t = w; t < nvt; t += NWT) {
        const int v = 16 * t + q, c = L->rank[v];
        if (c >= 0) {
            const double x2 = L->nrm[v], is = rsqrt_nr(x2);
            const DP x = V + v * ld;
#pragma unroll 2
            for (int e = g; e < len; e += 4) {
                const uint32_t ix = e * ue + c * uc;
                at(Ure, ix) = T(x[e] * is);
                at(Uim, ix) = T(x[lp + e] * is);
            }
            if (closed) {
                const double sc = x2 * is * renorm;
                const T c0 = T(sc * L->wc[v]), c1 = T(sc * L->wr[v]), c2 = T(-(sc * L->wi[v]));
                const int mt = L->pair[v];
                for (int u = g; u < nv; u += 4) {
                    const uint32_t ix = u * cu + c * cc;
                    at(Cre, ix) = u == v ? c0 : u == mt ? c1 : T(0);
                    at(Cim, ix) = u == mt ? c2 : T(0);
                }
            }
        }
    }
    if (!closed) {
        for (int i = w; i < nvt * nvt; i += NWT) {
            // (u, v): theta_u . conj(y_v) over the elements
            const int tu = i / nvt, t = i - tu * nvt;
            f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
            const glbd* th = stash + (16 * tu + q) * ld + g;
            const DP y = V + (16 * t + q) * ld + g;
            for (int e = 0; e < len; e += 4) {
                const double t0 = th[e], t1 = th[lp + e], y0 = y[e], y1 = y[lp + e];
                re = mfma(t0, y0, re);
                im = mfma(t1, y0, im);
                re = mfma(t1, y1, re);
                im = mfma(-t0, y1, im);
            }
            const int c = L->rank[16 * t + q];
            const double sc = rsqrt_nr(L->nrm[16 * t + q]) * renorm;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int u = 16 * tu + g + 4 * x;
                if (c >= 0 && u < nv) {
                    const uint32_t ix = u * cu + c * cc;
                    at(Cre, ix) = T(re[x] * sc);
                    at(Cim, ix) = T(im[x] * sc);
                }
            }
        }
    }
    team_sync<NWT>();
    return out;
}

// Centre move (as wave_move).  The Gram matrix reads the vectors from the
// slot; in the usual case (every vector kept, in place) the tensors are scaled
// where they are, else their new elements go through the slot's scratch.
template <typename T, int NWT, typename LW>
__device__ __forceinline__ WideOp team_move(const Trunc P, LW* L, SiteView<T> A, SiteView<T> B,
                                            int dir, int cl, int cm, int cr, glbd* stash) {
    typedef __attribute__((address_space(1))) T gT;
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const int w = team_wave<NWT>();
    const int nv = cm, len = dir ? 2 * cl : 2 * cr, wn = dir ? 2 * cr : 2 * cl;
    const int nvt = (nv + 15) >> 4;
    gT* Xre = dir ? A.re : B.re;
    gT* Xim = dir ? A.im : B.im;
    gT* Nre = dir ? B.re : A.re;
    gT* Nim = dir ? B.im : A.im;
    const int xe = dir ? cm : 1, xv = dir ? 1 : len;
    const int ne = dir ? 1 : cm, nvs = dir ? wn : 1;
    WideOp out{true, true, 0, 0, 0, 0.0};
    const auto gram = [&](int tp, int tq, f64x4& re, f64x4& im) {
        re = f64x4{0.0, 0.0, 0.0, 0.0};
        im = f64x4{0.0, 0.0, 0.0, 0.0};
        const int p = 16 * tp + q, c = 16 * tq + q;
#pragma unroll 4
        for (int e0 = 0; e0 < len; e0 += 4) {
            const int e = e0 + g;
            const bool ip = p < nv && e < len, ic = c < nv && e < len;
            const uint32_t jp = ip ? p * xv + e * xe : 0, jc = ic ? c * xv + e * xe : 0;
            const T a0 = at(Xre, jp), a1 = at(Xim, jp), b0 = at(Xre, jc), b1 = at(Xim, jc);
            const double xr = ip ? a0 : T(0), xi = ip ? a1 : T(0);
            const double yr = ic ? b0 : T(0), yi = ic ? b1 : T(0);
            re = mfma(xr, yr, re);
            im = mfma(xr, yi, im);
            re = mfma(xi, yi, re);
            im = mfma(-xi, yr, im);
        }
    };
    const double tau2 = P.tau * P.tau;
    const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                   : 8.0 * static_cast<double>(FLT_EPSILON);
    double total, floor2 = -1.0;
    if (team_overlaps<NWT>(gram, nvt, L, 1e-4 * tau2, floor2, tol * tol, total)) {
        out.fast = false;
        return out;
    }
    const Kept kp = team_select<NWT>(L, tau2, P.cap, nv);
    const int r = kp.r;
    out.r = r;
    out.dropped = kp.dropped;
    if (kp.dropped > 1e-12 * total && r == P.full) out.status |= MSC_SHOT_CHI_CAP;
    const double renorm = rsqrt_nr(kp.kept);
    int moved = 0;
    for (int t = w; t < nvt; t += NWT)
        if (16 * t + q < nv && L->rank[16 * t + q] != 16 * t + q) moved = 1;
    const bool inplace = team_or<NWT>(L, moved) == 0;
    const int ue = dir ? r : 1, uv = dir ? 1 : len;
    const int me = dir ? 1 : r, mv = dir ? wn : 1;
    glbd* sx = stash;
    glbd* sn = stash + 2 * (size_t)r * len;
    for (int t = w; t < nvt; t += NWT) {
        const int v = 16 * t + q, c = v < nv ? (int)L->rank[v] : -1;
        if (c >= 0) {
            const double x2 = L->nrm[v], is = rsqrt_nr(x2), sc = x2 * is * renorm;
#pragma unroll 2
            for (int e = g; e < len; e += 4) {
                const uint32_t ix = v * xv + e * xe;
                const double a = at(Xre, ix), b = at(Xim, ix);
                if (inplace) {
                    at(Xre, ix) = T(a * is);
                    at(Xim, ix) = T(b * is);
                } else {
                    sx[e * ue + c * uv] = a * is;
                    sx[(size_t)r * len + e * ue + c * uv] = b * is;
                }
            }
#pragma unroll 2
            for (int e = g; e < wn; e += 4) {
                const uint32_t ix = v * nvs + e * ne;
                const double a = at(Nre, ix), b = at(Nim, ix);
                if (inplace) {
                    at(Nre, ix) = T(a * sc);
                    at(Nim, ix) = T(b * sc);
                } else {
                    sn[e * me + c * mv] = a * sc;
                    sn[(size_t)r * wn + e * me + c * mv] = b * sc;
                }
            }
        }
    }
    team_sync<NWT>();
    if (!inplace) {
        const int tid = (int)threadIdx.x % (64 * NWT);
        for (int i = tid; i < r * len; i += 64 * NWT) {
            at(Xre, i) = T(sx[i]);
            at(Xim, i) = T(sx[(size_t)r * len + i]);
        }
        for (int i = tid; i < r * wn; i += 64 * NWT) {
            at(Nre, i) = T(sn[i]);
            at(Nim, i) = T(sn[(size_t)r * wn + i]);
        }
        team_sync<NWT>();
    }
    return out;
}

// Product swap (as wave_pswap), with M at Mp (2 pl pr doubles: the work area
// or the slot's scratch).
template <typename T, int NWT, typename LW, typename DP>
__device__ __forceinline__ void team_pswap(LW* L, SiteView<T> Pv, SiteView<T> Ov, int side, int pl,
                                           int pr, int newb, DP Mp) {
    const int lane = op_lane(), q = lane & 15, g = lane >> 4;
    const int w = team_wave<NWT>();
    const int nk = side ? pl : pr, nm = side ? pr : pl, no = 2 * newb;
    const int mk = side ? 2 * pr : 1, mq = side ? 1 : 2 * pr;     // strides in P
    const int ok = side ? 1 : no, oq = side ? pl : 1;             // strides in O
    const int kt = (nk + 3) >> 2, mt = (nm + 15) >> 4;
    double r4[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = w; i < kt * mt; i += NWT) {
        const int a = i / mt, kk = 4 * a + g, c = 16 * (i - a * mt) + q;
        if (kk < nk && c < nm) {
            const uint32_t i0 = kk * mk + c * mq;
            const double x0r = at(Pv.re, i0), x0i = at(Pv.im, i0);
            const double x1r = at(Pv.re, i0 + pr), x1i = at(Pv.im, i0 + pr);
            r4[0] += x0r * x0r + x0i * x0i;
            r4[1] += x1r * x1r + x1i * x1i;
            r4[2] += x0r * x1r + x0i * x1i;     // rho01 = x0 conj(x1)
            r4[3] += x0i * x1r - x0r * x1i;
        }
    }
    wave_sum4(r4);
    team_add4<NWT>(L, r4);
    const bool one = r4[1] > r4[0];
    const double pn = one ? r4[1] : r4[0];
    const double pd = rsqrt_nr(pn * (r4[0] + r4[1]));
    const double s0r = (one ? r4[2] : pn) * pd, s0i = one ? r4[3] * pd : 0.0;
    const double s1r = (one ? pn : r4[2]) * pd, s1i = one ? 0.0 : -(r4[3] * pd);
    for (int i = w; i < kt * mt; i += NWT) {
        const int a = i / mt, kk = 4 * a + g, c = 16 * (i - a * mt) + q;
        if (kk < nk && c < nm) {
            const uint32_t i0 = kk * mk + c * mq;
            const double x0r = at(Pv.re, i0), x0i = at(Pv.im, i0);
            const double x1r = at(Pv.re, i0 + pr), x1i = at(Pv.im, i0 + pr);
            Mp[kk * nm + c] = s0r * x0r + s0i * x0i + s1r * x1r + s1i * x1i;
            Mp[nk * nm + kk * nm + c] = s0r * x0i - s0i * x0r + s1r * x1i - s1i * x1r;
        }
    }
    team_sync<NWT>();
    const int rows = side ? no : pl, cols = side ? pr : no;
    const int ct = (cols + 15) >> 4, nt = ((rows + 15) >> 4) * ct;
    for (int i = w; i < nt; i += NWT) {
        const int tr = i / ct, R0 = 16 * tr, C0 = 16 * (i - tr * ct);
        // O's outer index and M's other index of this lane
        const int o = (side ? R0 : C0) + q, c = (side ? C0 : R0) + q;
        f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int k0 = 0; k0 < nk; k0 += 4) {
            const int kk = k0 + g;
            const bool io = o < no && kk < nk, ic = c < nm && kk < nk;
            const uint32_t jo = io ? kk * ok + o * oq : 0;
            const int jc = ic ? kk * nm + c : 0;
            const T o0 = at(Ov.re, jo), o1 = at(Ov.im, jo);
            const double m0 = Mp[jc], m1 = Mp[nk * nm + jc];
            const double xr = io ? o0 : T(0), xi = io ? o1 : T(0);
            const double yr = ic ? m0 : 0.0, yi = ic ? m1 : 0.0;
            const double ar = side ? xr : yr, ai = side ? xi : yi;
            const double br = side ? yr : xr, bi = side ? yi : xi;
            re = mfma(ar, br, re);
            im = mfma(ar, bi, im);
            re = mfma(-ai, bi, re);
            im = mfma(ai, br, im);
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int row = R0 + g + 4 * x, col = C0 + q;
            if (row < rows && col < cols) {
                const uint32_t ix = row * cols + col;
                at(Pv.re, ix) = T(re[x]);
                at(Pv.im, ix) = T(im[x]);
            }
        }
    }
    team_sync<NWT>();
    // the unentangled qubit on the other site: psi (x) identity
    for (int row = 4 * w + g; row < no; row += 4 * NWT) {          // (a, i)
        for (int c = q; c < newb; c += 16) {
            const bool diag = c == (row >> 1), i = row & 1;
            const uint32_t ix = row * newb + c;
            at(Ov.re, ix) = T(diag ? (i ? s1r : s0r) : 0.0);
            at(Ov.im, ix) = T(diag ? (i ? s1i : s0i) : 0.0);
        }
    }
    team_sync<NWT>();
}

// A wide op (kind OP_MOVE, OP_SWAPP or OP_G2 of sites a, a + 1; b its
// direction or side) by the whole team.  A product swap's new bond is set
// here; the caller sets the others' from the result.
template <typename T, int NWT, typename LW>
__device__ __forceinline__ WideOp wide_op(const Trunc P, LW* L, const LTables* tab, int kind, int a,
                                          int b, int gate_id, SiteView<T> A, SiteView<T> B,
                                          glbd* scr) {
    const int cl = uni(L->chi[a]), cm = uni(L->chi[a + 1]), cr = uni(L->chi[a + 2]);
    if (kind == OP_SWAPP) {
        const int pl = b ? cm : cl, pr = b ? cr : cm, newb = b ? cl : cr;
        const SiteView<T> Pv = b ? B : A, Ov = b ? A : B;
        if (2 * pl * pr <= LW::kWork)
            team_pswap<T, NWT>(L, Pv, Ov, b, pl, pr, newb, (ldsd*)L->work);
        else
            team_pswap<T, NWT>(L, Pv, Ov, b, pl, pr, newb, scr);
        return WideOp{true, true, newb, 0, 0, 0.0};
    }
    if (kind == OP_MOVE) return team_move<T, NWT>(P, L, A, B, b, cl, cm, cr, scr);
    const int nv = 2 * (b ? cr : cl), len = 2 * (b ? cl : cr);
    const int rows = (nv + 15) & ~15, ld = 2 * ((len + 15) & ~15) + 1;
    if (rows * ld <= LW::kWork)
        return team_update<T, NWT>(P, L, tab, A, B, b, gate_id, cl, cm, cr, (ldsd*)L->work, scr);
    return team_update<T, NWT>(P, L, tab, A, B, b, gate_id, cl, cm, cr, scr + (size_t)rows * ld, scr);
}

// The shots of one wavefront in its slot: each from its fork point (or from
// |0...0>) through the op stream to its result, op by op.  EXTRA compiles in
// checkpoint recording and segment reach.  NWT > 0: ops on bonds above 16 run
// by the team of NWT wavefronts this one leads (a wide centre move counts as
// the identity update it stands for, as in the workgroup kernel, whose LDS
// vectors hold 32); NWT = 0: the slots' bonds stay within 16.
template <typename T, bool EXTRA, int NWT, typename LW>
__device__ __forceinline__ void run_wave(const MpsArgs& P, LW* L, const LTables* tab, int team) {
    typedef __attribute__((address_space(1))) T gT;
    const int lane = threadIdx.x & 63;
    const int N = P.n_sites;
    gT* slot = to_glb(static_cast<T*>(P.arena) + (size_t)team * P.slot_stride);
    glbd* scr = to_glb(P.scratch + (size_t)team * P.scratch_stride);
    const int cap = N > 1 ? min(P.chi_max, P.cap[1]) : 1;
    const Trunc trunc{P.tau, P.chi_max, cap, NWT > 0 ? P.chi_max : cap};
    // (k is the same in every lane)
    const auto site = [&](int k) {
        SiteView<T> v;
        v.re = slot + uni(tab->soff[k]);
        v.im = v.re + uni(tab->shalf[k]);
        return v;
    };
    const auto chi = [&](int k) { return uni(L->chi[k]); };
    const int lane0 = lane == 0;
    // Hands a wide op to the team.  The followers read the command and, in
    // wide_op, the bonds after the barrier here and before the op's first one,
    // so every wide op passes at least one barrier of the whole workgroup on
    // every path (also where it returns early) and all wavefronts return from
    // it alike; only then may the leader write a bond or the next command.
    const auto wide = [&](int kind, int a, int b, int gate_id) {
        if constexpr (NWT > 1) {
            if (lane0) {
                L->cmd[0] = kind;
                L->cmd[1] = a;
                L->cmd[2] = b;
                L->cmd[3] = gate_id;
            }
            __syncthreads();
        }
        if constexpr (NWT > 0)
            return wide_op<T, NWT>(trunc, L, tab, kind, a, b, gate_id, site(a), site(a + 1), scr);
        else
            return WideOp{};
    };
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
#pragma unroll 4
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
                bool fast;
                if (NWT > 0 && (cm > 16 || max(cl, cr) > 16)) {
                    const WideOp o = wide(OP_MOVE, a, b, 0);
                    fast = o.fast;
                    if (fast) {
                        acc.disc += o.dropped;
                        acc.status |= o.status;
                        if (lane0) L->chi[a + 1] = o.r;
                        if (cm > 32 || (b ? cl : cr) > 16) {
                            // an identity update in the records
                            const double dl = cl, dm = cm, dr = cr, dk = o.r;
                            ++acc.n2q;
                            acc.chi_peak = max(acc.chi_peak, o.r);
                            acc.flops += 32.0 * dl * dm * dr + 32.0 * dl * dl * dr +
                                         32.0 * dk * dl * dr + 104.0 * dl * dl * dl;
                        }
                        wave_order();
                    }
                } else {
                    const SiteView<T> A = site(a), B = site(a + 1);
                    fast = max(max(cl, cr), cm) <= 8
                               ? wave_move8<T>(trunc, L, A, B, a, b, acc, cl, cm, cr)
                               : wave_move<T>(trunc, L, A, B, a, b, acc, cl, cm, cr);
                }
                if (!fast) {
                    twosite = true;
                    gate_id = G4_I;
                }
            } else if (kind == OP_SWAPP) {
                const int ps = a + b, os = a + 1 - b;
                const int pl = chi(ps), pr = chi(ps + 1), newb = b ? chi(a) : chi(a + 2);
                if (NWT > 0 && max(max(pl, pr), newb) > 16) {
                    wide(OP_SWAPP, a, b, 0);
                    if (lane0) L->chi[a + 1] = newb;
                    wave_order();
                } else {
                    wave_pswap<T>(L, site(ps), site(os), a, b, pl, pr, newb);
                }
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
                    for (int y = q; y < cr; y += 16) {
#pragma unroll 4
                        for (int x = g; x < cl; x += 4) {
                            const uint32_t i0 = x * 2 * cr + y, i1 = i0 + cr;
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
                const bool wide_site = NWT > 0 && max(cl, cr) > 16;
                if (!wide_site) {
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
                } else {
                    for (int y = q; y < cr; y += 16) {
#pragma unroll 2
                        for (int x = g; x < cl; x += 4) {
                            const uint32_t ie = (x * 2 + e) * cr + y, io = (x * 2 + 1 - e) * cr + y;
                            const double er = at(v.re, ie), ei = at(v.im, ie);
                            const double fr = at(v.re, io), fi = at(v.im, io);
                            pe2 += er * er + ei * ei;
                            po2 += fr * fr + fi * fi;
                        }
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
                if (!wide_site) {
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
                } else {
                    for (int y = q; y < cr; y += 16) {
#pragma unroll 2
                        for (int x = g; x < cl; x += 4) {
                            const uint32_t ie = (x * 2 + e) * cr + y, io = (x * 2 + 1 - e) * cr + y;
                            at(v.re, ie) = T(static_cast<double>(at(v.re, ie)) * sc);
                            at(v.im, ie) = T(static_cast<double>(at(v.im, ie)) * sc);
                            at(v.re, io) = T(0);
                            at(v.im, io) = T(0);
                        }
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
                for (int y = q; y < cr; y += 16) {
                    for (int x = g; x < cl; x += 4) {
                        const uint32_t i0 = x * 2 * cr + y, i1 = i0 + cr;
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
                if (nv <= 16 && len <= 32)
                    ok = wave_update<T, 1>(trunc, L, tab, A, B, a, b, gate_id, acc, cl, cm, cr,
                                           (ldsd*)L->work, scr);
                else if (nv <= 32 && len <= 16)
                    ok = wave_update<T, 2>(trunc, L, tab, A, B, a, b, gate_id, acc, cl, cm, cr,
                                           (ldsd*)L->work, scr);
                else if constexpr (NWT == 0)
                    ok = wave_update<T, 2>(trunc, L, tab, A, B, a, b, gate_id, acc, cl, cm, cr,
                                           scr + kStash, scr);
                else {
                    const WideOp o = wide(OP_G2, a, b, gate_id);
                    ok = o.ok;
                    if (ok) {
                        const double dl = cl, dm = cm, dr = cr, dk = o.r;
                        acc.disc += o.dropped;
                        acc.status |= o.status;
                        acc.sweeps += o.sweeps;
                        acc.chi_peak = max(acc.chi_peak, o.r);
                        ++acc.n2q;
                        acc.flops += 32.0 * dl * dm * dr + 32.0 * dl * dl * dr + 32.0 * dk * dl * dr +
                                     104.0 * dl * dl * dl;
                        if (lane0) L->chi[a + 1] = o.r;
                        wave_order();
                    }
                }
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
    if constexpr (NWT > 1) {
        if (lane0) L->cmd[0] = -1;
        __syncthreads();
    }
}

// The other wavefronts of a team: they join every wide op until the leader
// has no shots left (the barriers pair with wide() and those inside the op; a
// wide op that some wavefront left without passing its barriers would hang the
// workgroup or let the leader overwrite a command still to be read).
template <typename T, int NWT, typename LW>
__device__ __forceinline__ void follow(const MpsArgs& P, LW* L, const LTables* tab, int team) {
    typedef __attribute__((address_space(1))) T gT;
    gT* slot = to_glb(static_cast<T*>(P.arena) + (size_t)team * P.slot_stride);
    glbd* scr = to_glb(P.scratch + (size_t)team * P.scratch_stride);
    const Trunc trunc{P.tau, P.chi_max, P.n_sites > 1 ? min(P.chi_max, P.cap[1]) : 1, P.chi_max};
    for (;;) {
        __syncthreads();
        const int kind = uni(L->cmd[0]), a = uni(L->cmd[1]), b = uni(L->cmd[2]),
                  gate_id = uni(L->cmd[3]);
        if (kind < 0) return;
        SiteView<T> A, B;
        A.re = slot + uni(tab->soff[a]);
        A.im = A.re + uni(tab->shalf[a]);
        B.re = slot + uni(tab->soff[a + 1]);
        B.im = B.re + uni(tab->shalf[a + 1]);
        wide_op<T, NWT>(trunc, L, tab, kind, a, b, gate_id, A, B, scr);
    }
}

// The workgroup's tables (nt threads; ends synchronised).
__device__ __forceinline__ void fill_tables(const MpsArgs& P, TableLds& s_tab, int nt) {
    const int tid = threadIdx.x;
    for (int k = tid; k < P.n_sites; k += nt) {
        s_tab.soff[k] = static_cast<int>(P.site_off[k]);
        s_tab.shalf[k] = static_cast<int>(P.site_half[k]);
    }
    for (int i = tid; i < G1_COUNT * 8; i += nt) s_tab.g1[i] = P.g1[i];
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
}

template <typename T, bool EXTRA>
__global__ __launch_bounds__(NT, 3) void mps_fast_wave_kernel(MpsArgs P) {
    __shared__ __align__(16) WaveLds s_wave[NW];
    __shared__ __align__(16) TableLds s_tab;
    fill_tables(P, s_tab, NT);
    const int w = uni(threadIdx.x >> 6);
    run_wave<T, EXTRA, 0>(P, (__attribute__((address_space(3))) WaveLds*)(s_wave + w),
                          (LTables*)&s_tab, blockIdx.x * NW + w);
}

// Bond cap 32: still one shot per wavefront, seven per workgroup and CU (LDS:
// 64 vectors of 16 elements, 32 of 32 or 16 of 64 each; wider factorisations
// in the slot's scratch).
typedef TeamLds<64, 64 * 33, 1> MidLds;
template <typename T>
__global__ __launch_bounds__(64 * kMidTeams, 1) void mps_fast_mid_kernel(MpsArgs P) {
    __shared__ __align__(16) MidLds s_wave[kMidTeams];
    __shared__ __align__(16) TableLds s_tab;
    fill_tables(P, s_tab, 64 * kMidTeams);
    const int w = uni(threadIdx.x >> 6);
    run_wave<T, true, 1>(P, (__attribute__((address_space(3))) MidLds*)(s_wave + w),
                         (LTables*)&s_tab, blockIdx.x * kMidTeams + w);
}

// Bond cap 128: one shot per workgroup of kGroupWaves wavefronts, one
// workgroup per CU (LDS: 128 vectors of 64 elements or 64 of 128).
typedef TeamLds<256, 128 * 129, kGroupWaves> GroupLds;
template <typename T>
__global__ __launch_bounds__(64 * kGroupWaves, 1) void mps_fast_group_kernel(MpsArgs P) {
    __shared__ __align__(16) GroupLds s_shot;
    __shared__ __align__(16) TableLds s_tab;
    fill_tables(P, s_tab, 64 * kGroupWaves);
    auto* L = (__attribute__((address_space(3))) GroupLds*)&s_shot;
    if (uni(threadIdx.x >> 6) == 0)
        run_wave<T, true, kGroupWaves>(P, L, (LTables*)&s_tab, blockIdx.x);
    else
        follow<T, kGroupWaves>(P, L, (LTables*)&s_tab, blockIdx.x);
}

}  // namespace

FastKernel fast_kernel(int cap) {
    FastKernel k{};
    k.teams = cap <= kFastWaveBond ? kWaveTeams : cap <= kFastMidBond ? kMidTeams : 1;
    k.blocks_per_cu = cap <= kFastWaveBond ? 3 : 1;
    return k;
}

hipError_t launch_mps_fast(int precision, int cap, const MpsArgs& a, int grid, hipStream_t s) {
    static_assert(kWaveTeams == NW, "one team per wavefront");
    static_assert(sizeof(WaveLds) * NW + sizeof(TableLds) <= 160 * 1024 / 3, "three workgroups per CU");
    static_assert(sizeof(MidLds) * kMidTeams + sizeof(TableLds) <= 160 * 1024, "LDS of one CU");
    static_assert(sizeof(GroupLds) + sizeof(TableLds) <= 160 * 1024, "LDS of one CU");
    static_assert(2 * kStash <= fast_scratch(1), "theta and the vectors of a cap-16 slot");
    if (!a.next || !a.retry_count || !a.retry_list || a.calibrate || a.state || cap < 1 ||
        cap > kFastGroupBond || a.scratch_stride < fast_scratch(cap))
        return hipErrorInvalidValue;
    const auto go = [&](auto kernel, int nt) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(nt), 0, s, a);
        return hipGetLastError();
    };
    const bool d = precision == MSC_FP64;
    if (cap > kFastMidBond)
        return d ? go(mps_fast_group_kernel<double>, 64 * kGroupWaves)
                 : go(mps_fast_group_kernel<float>, 64 * kGroupWaves);
    if (cap > kFastWaveBond)
        return d ? go(mps_fast_mid_kernel<double>, 64 * kMidTeams)
                 : go(mps_fast_mid_kernel<float>, 64 * kMidTeams);
    const bool extra = a.surv != nullptr || a.ck_mode == 1;
    if (d) return extra ? go(mps_fast_wave_kernel<double, true>, NT) : go(mps_fast_wave_kernel<double, false>, NT);
    return extra ? go(mps_fast_wave_kernel<float, true>, NT) : go(mps_fast_wave_kernel<float, false>, NT);
}

}  // namespace msc
