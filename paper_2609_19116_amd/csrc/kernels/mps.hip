// Persistent batched MPS shot kernel for gfx950.
//
// One workgroup (4 wavefronts, one per SIMD) owns one MPS slot in HBM and
// runs whole shots through the compiled op stream, taking shots blockIdx.x,
// blockIdx.x + gridDim.x, ...  Each shot has its own ragged bond
// dimensions, kept in LDS, and stops at the first measurement whose
// expected outcome has probability below tau_rej (online screening,
// Section 4.3), so a rejected shot frees its workgroup for the next one at
// once.
//
// Per op (Section 3.1 for the MPS, Section 4 for the shot semantics):
//  * 1q gates and Pauli faults act on one site tensor (chi_l x 2 x chi_r);
//  * a two-site update contracts A[k] A[k+1] (complex, in the tensor
//    precision T), applies the 4x4 gate, and factorises the result exactly:
//    one-sided Jacobi (Hestenes) SVD in FP64 on the columns (centre moves
//    right) or rows (centre moves left) of theta, held in LDS when both
//    sides are at most SMAX, else in the slot's HBM scratch; singular values
//    sigma_i <= tau * sigma_0 are dropped (numerical zeros), the bond becomes
//    the number kept, the isometric factor is the normalised orthogonal
//    vectors and the centre factor is the projection of theta on them,
//    renormalised in FP64 (Section 3.1, "exact regime" of Section 5.1);
//  * a measurement, taken with the centre on the site, computes
//    p_e = ||A[:, e, :]||^2 / ||A||^2 in FP64, rejects if p_e < tau_rej,
//    otherwise projects, renormalises and multiplies P_acc by p_e;
//  * the final op reads the seed qubit's reduced density matrix and the
//    fidelity with the target (Appendix "Post-selection and logical error").
//
// Latency, not arithmetic, bounds a shot: the ops are small and strictly
// sequential.  Small factorisations (both sides of theta at most 32, the
// bulk of the updates) and centre moves therefore run on wavefront 0 alone
// with wave-level synchronisation while the other three wavefronts wait at
// the op's one workgroup barrier; larger ones use the whole workgroup.  Op
// descriptors, gate tables and the slot layout are served from LDS.
#include <hip/hip_runtime.h>

#include <algorithm>

#include <cfloat>
#include <cstdint>

#include "kernels.h"
#include "mps_common.h"

namespace msc {
namespace {

constexpr int MAXV = 2 * kMaxChiKernel;   // vectors in a two-site SVD
constexpr int kStage = 2048;               // doubles of LDS staging per workgroup
constexpr int kOpBuf = 128;                // op descriptors per LDS refill
constexpr int kWaveSide = 16;              // largest theta side factorised by one wave

// Squared norms of nv vectors (stride ld) into nrm.  When the team has
// lanes to spare, g consecutive lanes (g a power of two <= 16, within a
// wavefront) share a vector: each sums every g-th element, then the group
// adds the partial sums by DPP moves.
template <int W, typename DP>
__device__ void vector_norms(DP vre, DP vim, int nv, int len, int ld, DP nrm) {
    const int tid = Team<W>::rank();
    int g = 1;
    while (g < 16 && nv * g * 2 <= W) g *= 2;
    const int per = W / g, sub = tid & (g - 1), vi = tid / g;
    for (int v0 = 0; v0 < nv; v0 += per) {
        const int v = v0 + vi;
        double s0 = 0.0, s1 = 0.0;
        if (v < nv) {
            DP xr = vre + (size_t)v * ld;
            DP xi = vim + (size_t)v * ld;
#pragma unroll 2
            for (int e = sub; e < len; e += g) {
                s0 += xr[e] * xr[e];
                s1 += xi[e] * xi[e];
            }
        }
        const double sum = group_sum(s0 + s1, g);
        if (v < nv && sub == 0) nrm[v] = sum;
    }
    Team<W>::sync();
}

// One parallel pass over every pair of vectors whose squared norms exceed
// floor2 (only pairs with a vector flagged in `only`, if given): marks in
// `bad` every vector of a pair that overlaps by more than tol and returns
// true (team-uniform) if there is one.
template <int W, typename DP, typename IP>
__device__ bool not_orthogonal(DP vre, DP vim, int nv, int len, int ld, DP nrm, double floor2,
                               double tol, IP bad, IP only) {
    const int tid = Team<W>::rank();
    for (int v = tid; v < nv; v += W) bad[v] = 0;
    Team<W>::sync();
    int any = 0;
    const int npair = nv * (nv - 1) / 2;
    const double tol2 = tol * tol;
    // pair index t -> (p, q), p < q, walking the upper triangle row by row
    int p = 0, rowlen = nv - 1, t0 = 0;
    for (int t = tid; t < npair; t += W) {
        while (t >= t0 + rowlen) {
            t0 += rowlen;
            ++p;
            --rowlen;
        }
        const int q = p + 1 + (t - t0);
        if (only && !(only[p] | only[q])) continue;
        const double a = nrm[p], b = nrm[q];
        if (!(a > floor2 && b > floor2)) continue;
        DP xr = vre + (size_t)p * ld;
        DP xi = vim + (size_t)p * ld;
        DP yr = vre + (size_t)q * ld;
        DP yi = vim + (size_t)q * ld;
        double gr = 0.0, gim = 0.0;
#pragma unroll 2
        for (int e = 0; e < len; ++e) {
            gr += xr[e] * yr[e] + xi[e] * yi[e];
            gim += xr[e] * yi[e] - xi[e] * yr[e];
        }
        if (gr * gr + gim * gim > tol2 * a * b) {
            any = 1;
            bad[p] = 1;   // benign race: every writer stores 1
            bad[q] = 1;
        }
    }
    return Team<W>::any(any);
}

// Keep the vectors with sigma^2 > tau2 * sigma_0^2 (at most capb), ordered by
// decreasing norm: sel[0..r) are their indices, isq[c] = 1/sigma and
// sq[c] = sigma of the c-th kept vector (each computed once here).
template <int W, typename DP, typename IP>
__device__ Kept select_kept(DP nrm, int nv, double tau2, int capb, IP sel, DP isq, DP sq,
                            double* red) {
    const int tid = Team<W>::rank();
    double mx = 0.0;
    for (int v = tid; v < nv; v += W) mx = fmax(mx, sel_norm(nrm[v]));
    mx = team_max<W>(mx, red);
    double kd[4] = {0.0, 0.0, 0.0, 0.0};
    // one wavefront with a lane per vector: the other vectors' norms are
    // read from their lanes, not from memory
    const bool lanes = W == 64 && nv <= 64;
    const double xl = (lanes && tid < nv) ? sel_norm(nrm[tid]) : 0.0;
    for (int v = tid; v < nv; v += W) {
        const double x = lanes ? xl : sel_norm(nrm[v]);
        int rank = 0;
        if (lanes) {
            for (int u = 0; u < nv; ++u) {
                const double y = lane_read(xl, u);
                rank += (y > x) || (y == x && u < v);
            }
        } else {
            for (int u = 0; u < nv; ++u) {
                const double y = sel_norm(nrm[u]);
                rank += (y > x) || (y == x && u < v);
            }
        }
        const bool above = x > tau2 * mx || rank == 0;
        kd[3] += above ? 1.0 : 0.0;
        const bool keep = above && rank < capb;
        if (keep) {
            // (only an all-zero theta keeps a vector of norm near 0)
            const bool nrm_ok = x > 1e-290;
            const double is = nrm_ok ? rsqrt_nr(x) : 1.0 / sqrt(x);
            sel[rank] = v;
            sq[rank] = nrm_ok ? x * is : sqrt(x);
            isq[rank] = is;
            kd[0] += 1.0;
            kd[1] += x;
        } else {
            kd[2] += x;
        }
    }
    team_sum<W, 4>(kd, red);
    Team<W>::sync();
    Kept k;
    k.r = static_cast<int>(kd[0] + 0.5);
    k.want = static_cast<int>(kd[3] + 0.5);
    k.kept = kd[1];
    k.dropped = kd[2];
    return k;
}

// LDS of a team (the workgroup, or one wavefront of the wavefront kernel),
// shared by the op implementations.
struct Smem {
    int* chi;            // [kMaxSites + 1] bond dimensions
    int* laste;          // [kMaxSites] last measured outcome per site
    int* flag;           // [1]
    DevOp* ops;          // op descriptors, a window of the op stream
    const int32_t* soff; // [kMaxSites] site offsets within a slot
    const int32_t* shalf;
    const double* g1;    // [G1_COUNT * 8] 2x2 gates
    int n_u;             // doubles of staging at u
    int n_work = 0;      // doubles from vre on (vectors and staging) usable as one
                         // area by a wide factorisation (one-wavefront teams)
    int n_vmax = 0;      // capacity of the per-vector arrays in LDS (wide case)
    double* vre;         // SVD vectors (SMAX x (SMAX + 1)), planar
    double* vim;
    double* nrm;         // [SMAX]
    double* isq;         // [SMAX]
    double* sq;          // [SMAX]
    int* sel;
    int* bad;
    int* list;
    int* ired;           // [NW]
    double* red;         // [NW * 4]
    const int* cap;      // [kMaxSites + 1] bond capacities
    double* u;           // [kStage] staging
    const int* g4src;    // [G4_COUNT * 4] monomial 4x4 gates: source column
    const double* g4ph;  // [G4_COUNT * 8] and phase of each row
};

// Per-vector work arrays of a factorisation: in LDS or in the slot's HBM
// scratch (DP, IP carry the address space).
template <typename DP, typename IP>
struct Vecs {
    DP vre, vim, nrm, isq, sq;
    IP sel, bad, list;
};

// Centre move from site k to k+1 (dir 1) or k+1 to k (dir 0) when the
// centre site's vectors (columns for dir 1, rows for dir 0) are already
// orthogonal, as they are after a split that left the centre there: a
// selection of the kept vectors, their normalisation and a rescaling of the
// neighbour.  Returns false (team-uniform) when a pair overlaps; the caller
// then falls back to a two-site identity update.  The vectors live in V
// (LDS, or the slot's scratch); the rescaled neighbour is staged in V's
// vector arrays when it fits in vcap doubles each, else at the start of the
// slot's scratch (which then must not hold V).
template <typename T, int W, typename DP, typename IP>
__device__ bool move_fast(const MpsArgs& P, const Smem& S, SiteView<T> A, SiteView<T> B, int k,
                          int dir, const Vecs<DP, IP>& V, int64_t vcap, double* scr, ShotAcc& acc) {
    typedef __attribute__((address_space(1))) T gT;
    typedef __attribute__((address_space(3))) T lT;
    const int tid = Team<W>::rank();
    const int cl = S.chi[k], cm = S.chi[k + 1], cr = S.chi[k + 2];
    const int nv = cm, len = dir ? 2 * cl : 2 * cr, ld = len + 1;
    // one wavefront: the neighbour that gets rescaled (B for dir 1, A for
    // dir 0) is copied to the staging area by direct loads now, so that its
    // global read overlaps the vectors' and the rescale reads LDS
    const int ne = dir ? cm * 2 * cr : 2 * cl * cm;
    const int ne16 = round16<T>(ne);
    const bool pre = W == 64 && (size_t)2 * ne16 * sizeof(T) <= (size_t)S.n_u * sizeof(double);
    lT* ure = to_lds(reinterpret_cast<T*>(S.u));
    lT* uim = ure + ne16;
    if (pre) {
        wave_load_lds(dir ? B.re : A.re, S.u, ne * sizeof(T));
        wave_load_lds(dir ? B.im : A.im, reinterpret_cast<T*>(S.u) + ne16, ne * sizeof(T));
    }
    DP vre = V.vre;
    DP vim = V.vim;
    DP nrm = V.nrm;
    DP isq = V.isq;
    DP sq = V.sq;
    IP sel = V.sel;
    gT* Are = A.re;
    gT* Aim = A.im;
    gT* Bre = B.re;
    gT* Bim = B.im;
    {
        gT* Xre = dir ? Are : Bre;
        gT* Xim = dir ? Aim : Bim;
        const double inv_len = rcp_nr(len);
        for (int idx = tid; idx < nv * len; idx += W) {
            const int v = qdiv(idx, inv_len), e = idx - v * len;
            const int at = dir ? e * cm + v : v * len + e;
            vre[v * ld + e] = static_cast<double>(Xre[at]);
            vim[v * ld + e] = static_cast<double>(Xim[at]);
        }
    }
    Team<W>::sync();
    vector_norms<W>(vre, vim, nv, len, ld, nrm);
    double tsum[1] = {0.0};
    for (int v = tid; v < nv; v += W) tsum[0] += nrm[v];
    team_sum<W, 1>(tsum, S.red);
    const double tau2 = P.tau * P.tau;
    const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                   : 8.0 * static_cast<double>(FLT_EPSILON);
    if (not_orthogonal<W>(vre, vim, nv, len, ld, nrm, 1e-4 * tau2 * tsum[0], tol, V.bad, (IP)nullptr))
        return false;
    const int capb = min(P.chi_max, S.cap[k + 1]);
    const Kept kp = select_kept<W>(nrm, nv, tau2, capb, sel, isq, sq, S.red);
    const int r = kp.r;
    acc.disc += kp.dropped;
    if (kp.dropped > 1e-12 * tsum[0] && r == capb) acc.status |= MSC_SHOT_CHI_CAP;
    const double renorm = 1.0 / sqrt(kp.kept);
    if (dir) {
        // A[k] <- normalised columns; A[k+1] <- its selected rows, rescaled
        // (rows c of the new A[k+1] are rows sel[c] of the old one, so they
        // are read before any is written: staged first)
        const double inv_r = rcp_nr(r);
        for (int idx = tid; idx < 2 * cl * r; idx += W) {
            const int e = qdiv(idx, inv_r), c = idx - e * r;
            const int v = sel[c];
            const double is = isq[c];
            Are[idx] = T(vre[v * ld + e] * is);
            Aim[idx] = T(vim[v * ld + e] * is);
        }
        const int w = 2 * cr;
        Team<W>::sync();
        if (pre) {
            // the old rows from the LDS copy, the new ones straight to B
            const double inv_w = rcp_nr(w);
            for (int idx = tid; idx < r * w; idx += W) {
                const int c = qdiv(idx, inv_w), x = idx - c * w;
                const int v = sel[c];
                const double sc = sq[c] * renorm;
                Bre[idx] = T(static_cast<double>(ure[v * w + x]) * sc);
                Bim[idx] = T(static_cast<double>(uim[v * w + x]) * sc);
            }
        } else if (r * w <= vcap) {
            const double inv_w = rcp_nr(w);
            for (int idx = tid; idx < r * w; idx += W) {
                const int c = qdiv(idx, inv_w), x = idx - c * w;
                const int v = sel[c];
                const double sc = sq[c] * renorm;
                vre[idx] = static_cast<double>(Bre[v * w + x]) * sc;
                vim[idx] = static_cast<double>(Bim[v * w + x]) * sc;
            }
            Team<W>::sync();
            for (int idx = tid; idx < r * w; idx += W) {
                Bre[idx] = T(vre[idx]);
                Bim[idx] = T(vim[idx]);
            }
        } else {
            glbd* tr_ = to_glb(scr);
            glbd* ti_ = tr_ + (size_t)r * w;
            const double inv_w = rcp_nr(w);
            for (int idx = tid; idx < r * w; idx += W) {
                const int c = qdiv(idx, inv_w), x = idx - c * w;
                const int v = sel[c];
                const double sc = sq[c] * renorm;
                tr_[idx] = static_cast<double>(Bre[v * w + x]) * sc;
                ti_[idx] = static_cast<double>(Bim[v * w + x]) * sc;
            }
            Team<W>::sync();
            for (int idx = tid; idx < r * w; idx += W) {
                Bre[idx] = T(tr_[idx]);
                Bim[idx] = T(ti_[idx]);
            }
        }
    } else {
        // A[k+1] <- normalised rows; A[k] <- its selected columns, rescaled
        const int w = 2 * cr;
        const double inv_w = rcp_nr(w);
        for (int idx = tid; idx < r * w; idx += W) {
            const int c = qdiv(idx, inv_w), e = idx - c * w;
            const int v = sel[c];
            const double is = isq[c];
            Bre[idx] = T(vre[v * ld + e] * is);
            Bim[idx] = T(vim[v * ld + e] * is);
        }
        Team<W>::sync();
        if (pre) {
            const double inv_r = rcp_nr(r);
            for (int idx = tid; idx < 2 * cl * r; idx += W) {
                const int row = qdiv(idx, inv_r), c = idx - row * r;
                const int v = sel[c];
                const double sc = sq[c] * renorm;
                Are[idx] = T(static_cast<double>(ure[row * cm + v]) * sc);
                Aim[idx] = T(static_cast<double>(uim[row * cm + v]) * sc);
            }
        } else if (2 * cl * r <= vcap) {
            const double inv_r = rcp_nr(r);
            for (int idx = tid; idx < 2 * cl * r; idx += W) {
                const int row = qdiv(idx, inv_r), c = idx - row * r;
                const int v = sel[c];
                const double sc = sq[c] * renorm;
                vre[idx] = static_cast<double>(Are[row * cm + v]) * sc;
                vim[idx] = static_cast<double>(Aim[row * cm + v]) * sc;
            }
            Team<W>::sync();
            for (int idx = tid; idx < 2 * cl * r; idx += W) {
                Are[idx] = T(vre[idx]);
                Aim[idx] = T(vim[idx]);
            }
        } else {
            glbd* tr_ = to_glb(scr);
            glbd* ti_ = tr_ + (size_t)2 * cl * r;
            const double inv_r = rcp_nr(r);
            for (int idx = tid; idx < 2 * cl * r; idx += W) {
                const int row = qdiv(idx, inv_r), c = idx - row * r;
                const int v = sel[c];
                const double sc = sq[c] * renorm;
                tr_[idx] = static_cast<double>(Are[row * cm + v]) * sc;
                ti_[idx] = static_cast<double>(Aim[row * cm + v]) * sc;
            }
            Team<W>::sync();
            for (int idx = tid; idx < 2 * cl * r; idx += W) {
                Are[idx] = T(tr_[idx]);
                Aim[idx] = T(ti_[idx]);
            }
        }
    }
    Team<W>::sync();
    if (tid == 0) S.chi[k + 1] = r;
    return true;
}

// theta = G . (A[k] A[k+1]) for the rows a of A[k]: written into the vectors
// (columns of theta for dir 1, rows for dir 0) with their total squared
// norm returned per thread.
template <typename T, int W, typename AP, typename DP>
__device__ double contract(AP Ar, AP Ai, AP Br, AP Bi, int cl, int cm, int cr, const int* gsrc,
                           const double* gph, int dir, int ld, DP vre, DP vim) {
    const int tid = Team<W>::rank();
    double nsum = 0.0;
    const double inv_cr = rcp_nr(cr);
    for (int idx = tid; idx < cl * cr; idx += W) {
        const int a = qdiv(idx, inv_cr), b = idx - a * cr;
        T sr[4] = {T(0), T(0), T(0), T(0)}, si[4] = {T(0), T(0), T(0), T(0)};
        AP a0r = Ar + (a * 2) * cm;
        AP a0i = Ai + (a * 2) * cm;
#pragma unroll 2
        for (int c = 0; c < cm; ++c) {
            const T x0r = a0r[c], x0i = a0i[c], x1r = a0r[cm + c], x1i = a0i[cm + c];
            const int b0 = (c * 2) * cr + b, b1 = b0 + cr;
            const T y0r = Br[b0], y0i = Bi[b0], y1r = Br[b1], y1i = Bi[b1];
            // S[i'j'] += A[a,i',c] B[c,j',b]
            sr[0] += x0r * y0r - x0i * y0i; si[0] += x0r * y0i + x0i * y0r;
            sr[1] += x0r * y1r - x0i * y1i; si[1] += x0r * y1i + x0i * y1r;
            sr[2] += x1r * y0r - x1i * y0i; si[2] += x1r * y0i + x1i * y0r;
            sr[3] += x1r * y1r - x1i * y1i; si[3] += x1r * y1i + x1i * y1r;
        }
        // monomial gate: output o = phase[o] * S[src[o]]
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const int j = gsrc[o];
            const double xr = static_cast<double>(sr[j]), xi = static_cast<double>(si[j]);
            const double pr = gph[2 * o], pim = gph[2 * o + 1];
            const double tr_ = pr * xr - pim * xi;
            const double ti_ = pr * xi + pim * xr;
            const int i = o >> 1, jj = o & 1;
            const int row = a * 2 + i, col = jj * cr + b;
            const size_t vi = dir ? (size_t)col * ld + row : (size_t)row * ld + col;
            vre[vi] = tr_;
            vim[vi] = ti_;
            nsum += tr_ * tr_ + ti_ * ti_;
        }
    }
    return nsum;
}

// Projection of theta (m x n, planar FP64 at thr/thi) on the kept vectors:
// R[c][col] = sum_row conj(U[row][c]) theta[row][col] into B (dir 1), or
// L[row][c] = sum_col theta[row][col] conj(V[c][col]) into A (dir 0).
template <typename T, int W, typename DP, typename IP, typename TP>
__device__ void project(TP thr, TP thi, int m, int n, int r, int dir, int ld, const Vecs<DP, IP>& V,
                        double renorm, __attribute__((address_space(1))) T* ore,
                        __attribute__((address_space(1))) T* oim) {
    const int tid = Team<W>::rank();
    if (dir) {
        const double inv_n = rcp_nr(n);
        for (int idx = tid; idx < r * n; idx += W) {
            const int c = qdiv(idx, inv_n), col = idx - c * n;
            const int v = V.sel[c];
            const double is = renorm * V.isq[c];
            DP ur = V.vre + (size_t)v * ld;
            DP ui = V.vim + (size_t)v * ld;
            double xr = 0.0, xi = 0.0;
#pragma unroll 2
            for (int row = 0; row < m; ++row) {
                const double a0 = ur[row], a1 = ui[row];
                const double t0 = thr[(size_t)row * n + col], t1 = thi[(size_t)row * n + col];
                xr += a0 * t0 + a1 * t1;
                xi += a0 * t1 - a1 * t0;
            }
            ore[idx] = T(xr * is);
            oim[idx] = T(xi * is);
        }
    } else {
        const double inv_r = rcp_nr(r);
        for (int idx = tid; idx < m * r; idx += W) {
            const int row = qdiv(idx, inv_r), c = idx - row * r;
            const int v = V.sel[c];
            const double is = renorm * V.isq[c];
            DP wr = V.vre + (size_t)v * ld;
            DP wi = V.vim + (size_t)v * ld;
            double xr = 0.0, xi = 0.0;
#pragma unroll 2
            for (int col = 0; col < n; ++col) {
                const double t0 = thr[(size_t)row * n + col], t1 = thi[(size_t)row * n + col];
                const double b0 = wr[col], b1 = wi[col];
                xr += t0 * b0 + t1 * b1;
                xi += t1 * b0 - t0 * b1;
            }
            ore[idx] = T(xr * is);
            oim[idx] = T(xi * is);
        }
    }
}

// Two-site update of sites k, k+1 with the 4x4 gate gate_id; the centre
// ends on k+1 (dir 1) or k (dir 0).  Sets chi[k+1] to the new bond.  V holds
// the vectors (LDS for sides <= SMAX, else the slot's scratch).  Returns
// false, having written nothing, when the slot's bond capacity is below
// chi_max and more vectors than it holds pass the threshold and the caller
// asked for that check (grow): the shot then needs a larger slot.
template <typename T, int SMAX, int W, typename DP, typename IP>
__device__ bool twosite_update(const MpsArgs& P, const Smem& S, SiteView<T> A, SiteView<T> B,
                               int k, int dir, int gate_id, double* scr, const Vecs<DP, IP>& V,
                               ShotAcc& acc, bool grow = false, int ldv = 0) {
    typedef __attribute__((address_space(1))) T gT;
    typedef __attribute__((address_space(3))) T lT;
    const int tid = Team<W>::rank();
    const int cl = S.chi[k], cm = S.chi[k + 1], cr = S.chi[k + 2];
    const int m = 2 * cl, n = 2 * cr;
    const int nv = dir ? n : m, len = dir ? m : n;
    // ldv > 0: the vectors take the team's whole work area (its staging
    // included, so theta's copy goes to the scratch), each vector's real and
    // imaginary parts side by side at the odd stride ldv (no bank conflicts
    // between vectors)
    const bool packed = ldv > 0;
    const int ld = packed ? ldv : len + 1;
    const int n_u = packed ? 0 : S.n_u;
    DP vre = V.vre, vim = packed ? V.vre + len : V.vim, nrm = V.nrm;
    IP sel = V.sel, bad = V.bad, list = V.list;
    gT* Are = A.re;
    gT* Aim = A.im;
    gT* Bre = B.re;
    gT* Bim = B.im;
    // the 4x4 gates of the op stream are monomial: one nonzero per row
    const int* gsrc = S.g4src + gate_id * 4;
    const double* gph = S.g4ph + gate_id * 8;
    // both site tensors into LDS with one coalesced pass when they fit: the
    // contraction then reads each element from LDS
    const int na = cl * 2 * cm, nb = cm * 2 * cr;
    double nsum[1];
    // planes at 16-byte offsets (one wavefront stages them by direct loads)
    const int na16 = round16<T>(na), nb16 = round16<T>(nb);
    if ((size_t)2 * (na16 + nb16) * sizeof(T) <= (size_t)n_u * sizeof(double)) {
        lT* st = to_lds(reinterpret_cast<T*>(S.u));
        if constexpr (W == 64) {
            T* u = reinterpret_cast<T*>(S.u);
            wave_load_lds(Are, u, na * sizeof(T));
            wave_load_lds(Aim, u + na16, na * sizeof(T));
            wave_load_lds(Bre, u + 2 * na16, nb * sizeof(T));
            wave_load_lds(Bim, u + 2 * na16 + nb16, nb * sizeof(T));
        } else {
            for (int i = tid; i < na; i += W) {
                st[i] = Are[i];
                st[na16 + i] = Aim[i];
            }
            for (int i = tid; i < nb; i += W) {
                st[2 * na16 + i] = Bre[i];
                st[2 * na16 + nb16 + i] = Bim[i];
            }
        }
        Team<W>::sync();
        nsum[0] = contract<T, W>(st, st + na16, st + 2 * na16, st + 2 * na16 + nb16, cl, cm, cr,
                                 gsrc, gph, dir, ld, vre, vim);
    } else {
        nsum[0] = contract<T, W>(Are, Aim, Bre, Bim, cl, cm, cr, gsrc, gph, dir, ld, vre, vim);
    }
    team_sum<W, 1>(nsum, S.red);
    Team<W>::sync();
    const double total = nsum[0];
    const double tau2 = P.tau * P.tau;
    const double floor2 = 1e-4 * tau2 * total;
    // orthogonality tolerance: a few ulps of the tensor precision
    const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                   : 8.0 * static_cast<double>(FLT_EPSILON);
    // squared norms, then one parallel pass over every pair: if all vectors
    // are already orthogonal (the common case) no Jacobi sweep is needed
    vector_norms<W>(vre, vim, nv, len, ld, nrm);
    const bool rotated = not_orthogonal<W>(vre, vim, nv, len, ld, nrm, floor2, tol, bad, (IP)nullptr);
    // theta's copy for the projection: LDS staging when it fits
    const bool th_lds = 2 * (size_t)m * n <= (size_t)n_u;
    if (rotated) {
        // keep theta for the projection (the vectors still hold it)
        if (th_lds) {
            ldsd* thr = to_lds(S.u);
            ldsd* thi = thr + (size_t)m * n;
            const double inv_n = rcp_nr(n);
            for (int idx = tid; idx < m * n; idx += W) {
                const int row = qdiv(idx, inv_n), col = idx - row * n;
                const size_t vi = dir ? (size_t)col * ld + row : (size_t)row * ld + col;
                thr[idx] = vre[vi];
                thi[idx] = vim[vi];
            }
        } else {
            glbd* thr = to_glb(scr);
            glbd* thi = thr + (size_t)m * n;
            const double inv_n = rcp_nr(n);
            for (int idx = tid; idx < m * n; idx += W) {
                const int row = qdiv(idx, inv_n), col = idx - row * n;
                const size_t vi = dir ? (size_t)col * ld + row : (size_t)row * ld + col;
                thr[idx] = vre[vi];
                thi[idx] = vim[vi];
            }
        }
        // sweep until the parallel check finds every pair orthogonal; only
        // vectors of an overlapping pair need rotating: the others stay
        // orthogonal to every combination of them
        int sweeps = 0;
        bool again = true;
        while (again && sweeps < 40) {
            const int nbad = flagged_list<W>(bad, nv, list, S.ired);
            jacobi_sweep<W>(vre, vim, list, nbad, len, ld, floor2, tol);
            ++sweeps;
            vector_norms<W>(vre, vim, nv, len, ld, nrm);
            for (int v = tid; v < nv; v += W) sel[v] = bad[v];
            Team<W>::sync();
            again = not_orthogonal<W>(vre, vim, nv, len, ld, nrm, floor2, tol, bad, sel);
        }
        if (again) acc.status |= MSC_SHOT_NOCONV;
        acc.sweeps += sweeps;
    }
    const int capb = min(P.chi_max, S.cap[k + 1]);
    const Kept kp = select_kept<W>(nrm, nv, tau2, capb, sel, V.isq, V.sq, S.red);
    if (grow && kp.want > capb && capb < P.chi_max) return false;
    const int r = kp.r;
    acc.disc += kp.dropped;
    if (kp.dropped > 1e-12 * total && r == capb) acc.status |= MSC_SHOT_CHI_CAP;
    const double renorm = 1.0 / sqrt(kp.kept);
    // isometric factor: normalised vectors; centre factor: the projection
    // of theta on them.  When no rotation was needed the vectors are
    // theta's own columns (rows), so the projection is sigma_c on the
    // selected column (row) and zero elsewhere, up to overlaps below the
    // orthogonality tolerance.
    if (dir) {
        // A[k] (cl,2,r): U[row][c] = w_sel[c][row] / |w|
        const double inv_r = rcp_nr(r);
        for (int idx = tid; idx < m * r; idx += W) {
            const int row = qdiv(idx, inv_r), c = idx - row * r;
            const int v = sel[c];
            const double is = V.isq[c];
            Are[idx] = T(vre[(size_t)v * ld + row] * is);
            Aim[idx] = T(vim[(size_t)v * ld + row] * is);
        }
    } else {
        // A[k+1] (r,2,cr): V[c][col] = w_sel[c][col] / |w|
        const double inv_n = rcp_nr(n);
        for (int idx = tid; idx < r * n; idx += W) {
            const int c = qdiv(idx, inv_n), col = idx - c * n;
            const int v = sel[c];
            const double is = V.isq[c];
            Bre[idx] = T(vre[(size_t)v * ld + col] * is);
            Bim[idx] = T(vim[(size_t)v * ld + col] * is);
        }
    }
    if (!rotated) {
        if (dir) {
            const double inv_n = rcp_nr(n);
            for (int idx = tid; idx < r * n; idx += W) {
                const int c = qdiv(idx, inv_n), col = idx - c * n;
                const int v = sel[c];
                Bre[idx] = T(col == v ? V.sq[c] * renorm : 0.0);
                Bim[idx] = T(0);
            }
        } else {
            const double inv_r = rcp_nr(r);
            for (int idx = tid; idx < m * r; idx += W) {
                const int row = qdiv(idx, inv_r), c = idx - row * r;
                const int v = sel[c];
                Are[idx] = T(row == v ? V.sq[c] * renorm : 0.0);
                Aim[idx] = T(0);
            }
        }
    } else {
        // the vectors as this update laid them out
        Vecs<DP, IP> Vw = V;
        Vw.vim = vim;
        if (th_lds) {
            ldsd* thr = to_lds(S.u);
            project<T, W>(thr, thr + (size_t)m * n, m, n, r, dir, ld, Vw, renorm,
                          dir ? Bre : Are, dir ? Bim : Aim);
        } else {
            glbd* thr = to_glb(scr);
            project<T, W>(thr, thr + (size_t)m * n, m, n, r, dir, ld, Vw, renorm,
                          dir ? Bre : Are, dir ? Bim : Aim);
        }
    }
    if (tid == 0) S.chi[k + 1] = r;
    acc.chi_peak = max(acc.chi_peak, r);
    ++acc.n2q;
    const double dl = cl, dm = cm, dr = cr, dk = r;
    acc.flops += 32.0 * dl * dm * dr + 32.0 * dl * dl * dr + 32.0 * dk * dl * dr + 104.0 * dl * dl * dl;
    return true;
}

// The fold of a product swap: with psi the unentangled qubit's state on
// site ps (tensor P, pl x 2 x pr), M = sum_i conj(psi_i) P[:, i, :] is
// formed in FP64 at mr/mi (fold_m; when P has at most W elements each lane
// passes the pair P[a, 0, b], P[a, 1, b] it already holds in x), then the
// product site receives the neighbour times M: A[k] M (side 1, neighbour
// ol x 2 x pl) or M A[k+1] (side 0, neighbour pr x 2 x ocr) (fold_apply).
// Whole team; fold_m ends with the team synchronised, fold_apply after its
// writes are issued.
template <typename T, int W, typename MP>
__device__ void fold_m(MP mr, MP mi, SiteView<T> Pv, double p0r, double p0i, double p1r,
                       double p1i, int pl, int pr, const double (&x)[4]) {
    const int tid = Team<W>::rank();
    if (pl * pr <= W) {
        if (tid < pl * pr) {
            mr[tid] = p0r * x[0] + p0i * x[1] + p1r * x[2] + p1i * x[3];
            mi[tid] = p0r * x[1] - p0i * x[0] + p1r * x[3] - p1i * x[2];
        }
    } else {
        const double inv_pr = rcp_nr(pr);
        for (int idx = tid; idx < pl * pr; idx += W) {
            const int a = qdiv(idx, inv_pr), b = idx - a * pr;
            const int i0 = (a * 2) * pr + b, i1 = i0 + pr;
            const double x0r = Pv.re[i0], x0i = Pv.im[i0], x1r = Pv.re[i1], x1i = Pv.im[i1];
            mr[idx] = p0r * x0r + p0i * x0i + p1r * x1r + p1i * x1i;
            mi[idx] = p0r * x0i - p0i * x0r + p1r * x1i - p1i * x1r;
        }
    }
    Team<W>::sync();
}

template <typename T, int W, typename MP, typename OP>
__device__ void fold_apply(MP mr, MP mi, OP ore, OP oim, SiteView<T> Pv, int side, int ol,
                           int pl, int pr, int ocr) {
    const int tid = Team<W>::rank();
    if (side) {
        // product on k+1: new A[k+1] = A[k] M  (ol, 2, pr)
        const double inv_pr = rcp_nr(pr);
        for (int idx = tid; idx < ol * 2 * pr; idx += W) {
            const int row = qdiv(idx, inv_pr), c = idx - row * pr;
            double xr = 0.0, xi = 0.0;
#pragma unroll 2
            for (int b = 0; b < pl; ++b) {
                const double ar = ore[row * pl + b], ai = oim[row * pl + b];
                const double br = mr[b * pr + c], bi = mi[b * pr + c];
                xr += ar * br - ai * bi;
                xi += ar * bi + ai * br;
            }
            Pv.re[idx] = T(xr);
            Pv.im[idx] = T(xi);
        }
    } else {
        // product on k: new A[k] = M A[k+1]  (pl, 2, ocr)
        const int w = 2 * ocr;
        const double inv_w = rcp_nr(w);
        for (int idx = tid; idx < pl * w; idx += W) {
            const int a = qdiv(idx, inv_w), rem = idx - a * w;
            double xr = 0.0, xi = 0.0;
#pragma unroll 2
            for (int b = 0; b < pr; ++b) {
                const double ar = mr[a * pr + b], ai = mi[a * pr + b];
                const double br = ore[b * w + rem], bi = oim[b * w + rem];
                xr += ar * br - ai * bi;
                xi += ar * bi + ai * br;
            }
            Pv.re[idx] = T(xr);
            Pv.im[idx] = T(xi);
        }
    }
}

// Resident workgroups per CU the register budget is capped for: the shots
// are latency-bound, so more resident shots raise the throughput more than
// the spills of a tighter register cap cost.  The batched FP32 instance
// (39.6 KB of LDS with SMAX = 32) runs four per CU with 128 VGPRs; the
// others three (FP64 at SMAX = 32) or what their LDS allows (SMAX = 64).
template <typename T, int SMAX>
constexpr int kMpsWavesPerSimd = (sizeof(T) == sizeof(float) && SMAX == 32) ? 4 : 3;

// The team's LDS vectors as a Vecs.
__device__ __forceinline__ Vecs<ldsd*, ldsi*> lds_vecs(const Smem& S) {
    return Vecs<ldsd*, ldsi*>{to_lds(S.vre), to_lds(S.vim), to_lds(S.nrm), to_lds(S.isq),
                              to_lds(S.sq),  to_lds(S.sel), to_lds(S.bad), to_lds(S.list)};
}

// The shots of one team (a workgroup, or one wavefront of the wavefront
// kernel) in its slot `team` of n_teams: each from its fork point (or from
// |0...0>) through the op stream to its result, op by op.  S is the team's
// LDS; NOPS op descriptors are held at a time.
template <typename T, int SMAX, int W, int NOPS, bool EXTRA = true>
__device__ void run_team(const MpsArgs& P, const Smem& S, const int team, const int n_teams) {
    // modes compiled in: parking and calibration (the workgroup kernel
    // only), checkpoint recording and segment reach (EXTRA); a kernel built
    // without a mode keeps none of its arguments in registers
    constexpr bool kPark = W != 64;
    constexpr bool kExtra = EXTRA;
    const int tid = Team<W>::rank();
    const int N = P.n_sites;
    T* slot_base = static_cast<T*>(P.arena) + (size_t)team * P.slot_stride;
    double* scr = P.scratch + (size_t)team * P.scratch_stride;
    // per-vector arrays of SVDs too large for LDS, at the end of the slot's scratch
    double* g_nrm = scr + P.scratch_stride - 6 * MAXV;
    double* g_isq = g_nrm + MAXV;
    double* g_sq = g_isq + MAXV;
    int* g_sel = reinterpret_cast<int*>(g_sq + MAXV);
    int* g_bad = g_sel + MAXV;
    int* g_list = g_bad + MAXV;

    auto site = [&](int k) {
        SiteView<T> v;
        v.re = to_glb(slot_base + S.soff[k]);
        v.im = v.re + S.shalf[k];
        return v;
    };

    const int64_t n_run = P.n_dev ? min(*P.n_dev, P.n_shots) : P.n_shots;
    // with slot states the grid is the slot count and every launch picks up
    // where the slot's last one stopped
    ShotState* const st = kPark && P.state ? P.state + team : nullptr;
    int64_t j0 = team;
    bool resume = false;
    if (st) {
        const int status = st->status;
        if (status == kSlotDone || status == kSlotParked) return;
        if (status == kSlotResume) {
            resume = true;
            j0 = st->j;
        }
    }
    const bool can_park = st && P.park_side > 0;
    // the wavefront kernel takes its shots from a shared counter, the
    // workgroup kernel every n_teams-th one
    const auto next_j = [&](int64_t jj) -> int64_t {
        if constexpr (W == 64) {
            if (P.next) return wave_fetch(P.next);
        }
        return jj + n_teams;
    };
    if constexpr (W == 64) {
        if (P.next && !resume) j0 = wave_fetch(P.next);
    }
    for (int64_t j = j0; j < n_run; j = next_j(j)) {
        const int64_t it = P.perm ? P.perm[j] : j;
        const int64_t shot = P.shot_idx ? P.shot_idx[it] : it;
        if (shot < 0 || shot >= P.n_csr) {
            if (tid == 0) {
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
        int next_ch = fcur < fend ? P.chan[fcur] : -1;
        int fcode = 0;     // code of the last channel read (three-qubit faults)
        bool alive = true;
        int start = 0;
        int jck = -1;
        int next_seg = 0;             // next segment whose reach is unwritten
        int meas_done = 0;            // measurements projected so far
        if (P.ck_mode == 2) {
            // fork from the last checkpoint of the noiseless run before the
            // shot's first fault (the ops before it are fault-free here)
            const int navail = *P.ck_avail;
            const int jj = fcur < fend ? next_ch / P.ck_k : P.n_ck - 1;
            jck = jj < navail ? jj : navail - 1;
        }
        bool retried = false;         // handed to the workgroup kernel
        // forked at the read-out checkpoint: its dense tensors, read in place
        const __attribute__((address_space(1))) T* final_src = nullptr;
        int next_ck = 0;              // record mode: next checkpoint to take
        int64_t ck_pos = 0;           // record mode: elements written so far
        bool ck_full = false;
        if (resume) {
            // ---- continue a parked shot after its large update
            for (int k = tid; k <= N; k += W) S.chi[k] = st->chi[k];
            for (int k = tid; k < N; k += W) S.laste[k] = st->laste[k];
            fcur = st->fcur;
            next_ch = st->next_ch;
            fcode = st->fcode;
            p_acc = st->p_acc;
            infid = st->infid;
            rej_at = st->rej_at;
            alive = st->alive != 0;
            start = st->oi;
            meas_done = st->meas_done;
            next_seg = st->next_seg;
            next_ck = st->next_ck;
            ck_pos = st->ck_pos;
            ck_full = st->ck_full != 0;
            acc.status = st->shot_status;
            acc.chi_peak = st->chi_peak;
            acc.disc = st->disc;
            acc.n2q = st->n2q;
            acc.flops = st->flops;
            acc.sweeps = st->sweeps;
            jck = -2;                 // no fork, no initial state
            resume = false;
        }
        if (jck >= 0) {
            const CkHdr& h = P.ck_hdr[jck];
            for (int k = tid; k <= N; k += W) S.chi[k] = h.chi[k];
            for (int k = tid; k < N; k += W) S.laste[k] = h.laste[k];
            Team<W>::sync();
            const __attribute__((address_space(1))) T* src =
                to_glb(static_cast<const T*>(P.ck_data)) + P.ck_off[jck];
            if (jck == P.n_ck - 1) {
                // the checkpoint before the read-out: the only op left reads
                // one site, so the shot reads the checkpoint in place
                final_src = src;
            } else {
                int64_t o = 0;
                for (int k = 0; k < N; ++k) {
                    const int ne = S.chi[k] * 2 * S.chi[k + 1];
                    SiteView<T> v = site(k);
                    for (int idx = tid; idx < ne; idx += W) {
                        v.re[idx] = src[o + idx];
                        v.im[idx] = src[o + ne + idx];
                    }
                    o += 2 * ne;
                }
            }
            p_acc = h.p_acc;
            acc.disc = h.disc;
            acc.chi_peak = h.chi_peak;
            acc.status = h.status;
            start = P.ck_op[jck];
            meas_done = h.meas_done;
            // reach of the segments before the fork: the noiseless run's
            // running P_acc, as this shot would have computed it
            if (kExtra && P.surv) {
                while (next_seg < P.n_seg && P.seg_meas[next_seg] < meas_done) {
                    if (tid == 0) P.surv[it * P.n_seg + next_seg] = P.ck_pm[P.seg_meas[next_seg]];
                    ++next_seg;
                }
            }
        } else if (jck == -1) {
            // ---- initial product state |0...0>
            for (int k = tid; k <= N; k += W) S.chi[k] = 1;
            for (int k = tid; k < N; k += W) {
                S.laste[k] = 0;
                SiteView<T> v = site(k);
                v.re[0] = T(1);
                v.re[1] = T(0);
                v.im[0] = T(0);
                v.im[1] = T(0);
            }
        }
        Team<W>::sync();
        int ops_lo = 0, ops_hi = 0;   // op range held in s_ops

        for (int oi = start; oi < P.n_ops && alive; ++oi) {
            if (oi >= ops_hi) {
                Team<W>::sync();
                ops_lo = oi;
                ops_hi = min(P.n_ops, oi + NOPS);
                for (int i = tid; i < ops_hi - ops_lo; i += W) S.ops[i] = P.ops[ops_lo + i];
                Team<W>::sync();
            }
            if (kExtra && P.ck_mode == 1 && !ck_full && next_ck < P.n_ck && P.ck_op[next_ck] == oi) {
                // ---- record: the state before op oi, densely, site by site
                int64_t sz = 0;
                for (int k = 0; k < N; ++k) sz += 4 * (int64_t)S.chi[k] * S.chi[k + 1];
                if (ck_pos + sz <= P.ck_cap) {
                    __attribute__((address_space(1))) T* dst = to_glb(static_cast<T*>(P.ck_data)) + ck_pos;
                    int64_t o = 0;
                    for (int k = 0; k < N; ++k) {
                        const int ne = S.chi[k] * 2 * S.chi[k + 1];
                        SiteView<T> v = site(k);
                        for (int idx = tid; idx < ne; idx += W) {
                            dst[o + idx] = v.re[idx];
                            dst[o + ne + idx] = v.im[idx];
                        }
                        o += 2 * ne;
                    }
                    CkHdr& h = P.ck_hdr[next_ck];
                    for (int k = tid; k <= N; k += W) h.chi[k] = S.chi[k];
                    for (int k = tid; k < N; k += W) h.laste[k] = S.laste[k];
                    if (tid == 0) {
                        h.p_acc = p_acc;
                        h.meas_done = meas_done;
                        h.disc = acc.disc;
                        h.chi_peak = acc.chi_peak;
                        h.status = acc.status;
                        P.ck_off[next_ck] = ck_pos;
                    }
                    ck_pos += sz;
                    Team<W>::sync();
                    if (tid == 0) *P.ck_avail = next_ck + 1;
                    ++next_ck;
                } else {
                    ck_full = true;
                }
            }
            const DevOp op = S.ops[oi - ops_lo];
            bool twosite = op.kind == OP_G2;
            int gate_id = op.aux;
            if (op.kind == OP_MOVE) {
                // ---- move the centre by one site: one wavefront does the
                // usual case (orthogonal vectors, small sides)
                const int k = op.a, dir = op.b;
                const int cl = S.chi[k], cm = S.chi[k + 1], cr = S.chi[k + 2];
                const int nv = cm, len = dir ? 2 * cl : 2 * cr;
                SiteView<T> A = site(k), B = site(k + 1);
                bool fast = false;
                if constexpr (W == 64) {
                    // one wavefront: LDS vectors, or the slot's scratch after
                    // the staging area of the rescaled neighbour
                    if (nv <= SMAX && len <= SMAX) {
                        fast = move_fast<T, 64>(P, S, A, B, k, dir, lds_vecs(S), SMAX * (SMAX + 1),
                                                scr, acc);
                    } else {
                        glbd* vre = to_glb(scr + 4 * (size_t)cm * max(cl, cr));
                        const Vecs<glbd*, glbi*> V{vre, vre + (size_t)nv * (len + 1),
                                                   to_glb(g_nrm), to_glb(g_isq), to_glb(g_sq),
                                                   to_glb(g_sel), to_glb(g_bad), to_glb(g_list)};
                        fast = move_fast<T, 64>(P, S, A, B, k, dir, V, 0, scr, acc);
                    }
                    Team<W>::sync();
                } else if (nv <= SMAX && len <= SMAX) {
                    if (nv <= kWaveSide && len <= kWaveSide) {
                        if (tid < 64) {
                            const bool f = move_fast<T, 64>(P, S, A, B, k, dir, lds_vecs(S),
                                                            SMAX * (SMAX + 1), scr, acc);
                            if (tid == 0) S.flag[0] = f;
                        }
                        Team<W>::sync();
                        fast = S.flag[0] != 0;
                    } else {
                        fast = move_fast<T, NT>(P, S, A, B, k, dir, lds_vecs(S), SMAX * (SMAX + 1),
                                                scr, acc);
                        Team<W>::sync();
                    }
                }
                if (!fast) {
                    twosite = true;
                    gate_id = G4_I;
                }
            }
            if (op.kind == OP_G1 || op.kind == OP_FAULT || op.kind == OP_FAULT3 ||
                op.kind == OP_RESET) {
                // ---- local 2x2 on one site (two for a two-qubit fault)
                int g0 = -1, g1 = -1;
                if (op.kind == OP_G1) {
                    g0 = op.aux;
                } else if (op.kind == OP_RESET) {
                    if (S.laste[op.a] == 1) g0 = G_X;
                } else if (op.kind == OP_FAULT3) {
                    const int x2 = (fcode >> 4) & 1, z2 = (fcode >> 5) & 1;
                    if (x2 | z2) g0 = (x2 && z2) ? G_Y : (x2 ? G_X : G_Z);
                } else {
                    int code = 0;
                    if (fcur < fend && next_ch == op.aux) {
                        code = P.pauli[fcur];
                        ++fcur;
                        next_ch = fcur < fend ? P.chan[fcur] : -1;
                    }
                    fcode = code;
                    const int x0 = code & 1, z0 = (code >> 1) & 1;
                    const int x1 = (code >> 2) & 1, z1 = (code >> 3) & 1;
                    if (x0 | z0) g0 = (x0 && z0) ? G_Y : (x0 ? G_X : G_Z);
                    if ((x1 | z1) && op.b >= 0) g1 = (x1 && z1) ? G_Y : (x1 ? G_X : G_Z);
                }
                for (int h = 0; h < 2; ++h) {
                    const int gid = h == 0 ? g0 : g1;
                    if (gid < 0) continue;
                    const int k = h == 0 ? op.a : op.b;
                    const double* m = S.g1 + gid * 8;
                    const double m0 = m[0], m1 = m[1], m2 = m[2], m3 = m[3];
                    const double m4 = m[4], m5 = m[5], m6 = m[6], m7 = m[7];
                    SiteView<T> v = site(k);
                    const int cl = S.chi[k], cr = S.chi[k + 1];
                    const double inv_cr = rcp_nr(cr);
                    for (int idx = tid; idx < cl * cr; idx += W) {
                        const int a = qdiv(idx, inv_cr), b = idx - a * cr;
                        const int i0 = (a * 2) * cr + b, i1 = i0 + cr;
                        const double x0r = v.re[i0], x0i = v.im[i0], x1r = v.re[i1], x1i = v.im[i1];
                        v.re[i0] = T(m0 * x0r - m1 * x0i + m2 * x1r - m3 * x1i);
                        v.im[i0] = T(m0 * x0i + m1 * x0r + m2 * x1i + m3 * x1r);
                        v.re[i1] = T(m4 * x0r - m5 * x0i + m6 * x1r - m7 * x1i);
                        v.im[i1] = T(m4 * x0i + m5 * x0r + m6 * x1i + m7 * x1r);
                    }
                    Team<W>::sync();
                }
            } else if (op.kind == OP_SWAPP) {
                // ---- SWAP with a qubit that is unentangled in every shot:
                // its tensor is psi (x) M, so the swap moves psi to the other
                // site as psi (x) I and folds M into the neighbour (no SVD;
                // canonical form is kept because psi is normalised)
                const int k = op.a, side = op.b;
                const int ps = k + side, os = k + 1 - side;
                SiteView<T> Pv = site(ps), Ov = site(os);
                const int pl = S.chi[ps], pr = S.chi[ps + 1];
                const int ol = S.chi[k], ocr = S.chi[k + 2];
                const int on = side ? ol * 2 * pl : pr * 2 * ocr;   // neighbour elements
                const int on16 = round16<T>(on);
                // in LDS (neighbour staged) when it fits; one wavefront
                // stages it by direct loads now, overlapping the reads below
                const bool lds_fold = pl * pr <= SMAX * (SMAX + 1) &&
                                      (size_t)2 * on16 * sizeof(T) <= (size_t)S.n_u * sizeof(double);
                if (W == 64 && lds_fold) {
                    wave_load_lds(Ov.re, S.u, on * sizeof(T));
                    wave_load_lds(Ov.im, reinterpret_cast<T*>(S.u) + on16, on * sizeof(T));
                }
                double r4[4] = {0.0, 0.0, 0.0, 0.0};
                double xk[4] = {0.0, 0.0, 0.0, 0.0};   // this lane's first pair, for M
                const double inv_pr = rcp_nr(pr);
                for (int idx = tid; idx < pl * pr; idx += W) {
                    const int a = qdiv(idx, inv_pr), b = idx - a * pr;
                    const int i0 = (a * 2) * pr + b, i1 = i0 + pr;
                    const double x0r = Pv.re[i0], x0i = Pv.im[i0], x1r = Pv.re[i1], x1i = Pv.im[i1];
                    if (idx == tid) {
                        xk[0] = x0r;
                        xk[1] = x0i;
                        xk[2] = x1r;
                        xk[3] = x1i;
                    }
                    r4[0] += x0r * x0r + x0i * x0i;
                    r4[1] += x1r * x1r + x1i * x1i;
                    r4[2] += x0r * x1r + x0i * x1i;     // rho01 = x0 conj(x1)
                    r4[3] += x0i * x1r - x0r * x1i;
                }
                team_sum<W, 4>(r4, S.red);
                const double tr = r4[0] + r4[1];
                double p0r, p0i, p1r, p1i;               // psi, unit norm
                if (r4[1] > r4[0]) {
                    const double d = 1.0 / sqrt(r4[1] * tr);
                    p0r = r4[2] * d;
                    p0i = r4[3] * d;
                    p1r = r4[1] * d;
                    p1i = 0.0;
                } else {
                    const double d = 1.0 / sqrt(r4[0] * tr);
                    p0r = r4[0] * d;
                    p0i = 0.0;
                    p1r = r4[2] * d;                     // rho10 = conj(rho01)
                    p1i = -r4[3] * d;
                }
                // M = sum_i conj(psi_i) P[:, i, :] (pl x pr, FP64), then the
                // neighbour times M
                const int newb = side ? ol : ocr;
                // the unentangled qubit on the other site: psi (x) identity
                const auto write_psi = [&]() {
                    const double inv_newb = rcp_nr(newb);
                    const double inv_2xnewb = rcp_nr(2 * newb);
                    for (int idx = tid; idx < newb * 2 * newb; idx += W) {
                        const int a = qdiv(idx, inv_2xnewb), rem = idx - a * 2 * newb;
                        const int i = qdiv(rem, inv_newb), a2 = rem - i * newb;
                        const bool diag = a == a2;
                        Ov.re[idx] = T(diag ? (i ? p1r : p0r) : 0.0);
                        Ov.im[idx] = T(diag ? (i ? p1i : p0i) : 0.0);
                    }
                };
                if (lds_fold) {
                    typedef __attribute__((address_space(3))) T lT;
                    lT* st = to_lds(reinterpret_cast<T*>(S.u));
                    if (W != 64) {
                        for (int idx = tid; idx < on; idx += W) {
                            st[idx] = Ov.re[idx];
                            st[on16 + idx] = Ov.im[idx];
                        }
                    }
                    fold_m<T, W>(to_lds(S.vre), to_lds(S.vim), Pv, p0r, p0i, p1r, p1i, pl, pr, xk);
                    // the neighbour's staging loads have completed (the
                    // psi reads issued after them were waited for; the
                    // explicit wait on the vector-memory counter states it),
                    // so its site is rewritten alongside the fold
                    if (W == 64) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
                    write_psi();
                    fold_apply<T, W>(to_lds(S.vre), to_lds(S.vim), st, st + on16, Pv, side, ol, pl,
                                     pr, ocr);
                } else {
                    glbd* mr = to_glb(scr);
                    fold_m<T, W>(mr, mr + (size_t)pl * pr, Pv, p0r, p0i, p1r, p1i, pl, pr, xk);
                    fold_apply<T, W>(mr, mr + (size_t)pl * pr, Ov.re, Ov.im, Pv, side, ol, pl, pr,
                                     ocr);
                    Team<W>::sync();
                    write_psi();
                }
                if (tid == 0) S.chi[k + 1] = newb;
                Team<W>::sync();
            } else if (op.kind == OP_MEAS) {
                const int k = op.a;
                SiteView<T> v = site(k);
                const int cl = S.chi[k], cr = S.chi[k + 1];
                double pp[2] = {0.0, 0.0};
                const double inv_cr = rcp_nr(cr);
                for (int idx = tid; idx < cl * cr; idx += W) {
                    const int a = qdiv(idx, inv_cr), b = idx - a * cr;
                    const int i0 = (a * 2) * cr + b, i1 = i0 + cr;
                    const double x0r = v.re[i0], x0i = v.im[i0], x1r = v.re[i1], x1i = v.im[i1];
                    pp[0] += x0r * x0r + x0i * x0i;
                    pp[1] += x1r * x1r + x1i * x1i;
                }
                team_sum<W, 2>(pp, S.red);
                const double tot = pp[0] + pp[1];
                int e;
                const bool calib = kPark && P.calibrate;
                if (calib) e = pp[1] > pp[0] ? 1 : 0;
                else e = P.expected[op.aux];
                const double raw = pp[e];
                const double pe = tot > 0.0 ? raw / tot : 0.0;
                if (calib && tid == 0) {
                    P.cal_p[op.aux] = pe;
                    P.cal_e[op.aux] = static_cast<uint8_t>(e);
                }
                if (kExtra && P.surv) {
                    // segments starting at or before this measurement
                    while (next_seg < P.n_seg && P.seg_meas[next_seg] <= op.aux) {
                        if (tid == 0) P.surv[it * P.n_seg + next_seg] = p_acc;
                        ++next_seg;
                    }
                }
                if (kExtra && P.ck_mode == 1 && P.ck_pm && tid == 0) P.ck_pm[op.aux] = p_acc;
                if (!(pe >= P.tau_rej)) {
                    alive = false;
                    acc.status |= MSC_SHOT_REJECTED;
                    rej_at = op.aux;
                    p_acc = 0.0;
                    break;
                }
                p_acc *= pe;
                meas_done = op.aux + 1;
                const double sc = 1.0 / sqrt(raw);
                for (int idx = tid; idx < cl * cr; idx += W) {
                    const int a = qdiv(idx, inv_cr), b = idx - a * cr;
                    const int ie = (a * 2 + e) * cr + b, io = (a * 2 + 1 - e) * cr + b;
                    v.re[ie] = T(static_cast<double>(v.re[ie]) * sc);
                    v.im[ie] = T(static_cast<double>(v.im[ie]) * sc);
                    v.re[io] = T(0);
                    v.im[io] = T(0);
                }
                if (tid == 0) S.laste[k] = e;
                Team<W>::sync();
            } else if (op.kind == OP_FINAL) {
                const int k = op.a;
                SiteView<T> v = site(k);
                if (final_src) {
                    // site k of the dense checkpoint: planes of chi_j 2 chi_j+1
                    // elements per site, real then imaginary
                    int64_t o = 0;
                    for (int q = 0; q < k; ++q) o += 4 * (int64_t)S.chi[q] * S.chi[q + 1];
                    v.re = const_cast<__attribute__((address_space(1))) T*>(final_src + o);
                    v.im = v.re + 2 * S.chi[k] * S.chi[k + 1];
                }
                const int cl = S.chi[k], cr = S.chi[k + 1];
                double r[4] = {0.0, 0.0, 0.0, 0.0};   // r00, r11, Re r01, Im r01
                const double inv_cr = rcp_nr(cr);
                for (int idx = tid; idx < cl * cr; idx += W) {
                    const int a = qdiv(idx, inv_cr), b = idx - a * cr;
                    const int i0 = (a * 2) * cr + b, i1 = i0 + cr;
                    const double x0r = v.re[i0], x0i = v.im[i0], x1r = v.re[i1], x1i = v.im[i1];
                    r[0] += x0r * x0r + x0i * x0i;
                    r[1] += x1r * x1r + x1i * x1i;
                    // rho01 = x0 * conj(x1)
                    r[2] += x0r * x1r + x0i * x1i;
                    r[3] += x0i * x1r - x0r * x1i;
                }
                team_sum<W, 4>(r, S.red);
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
                // ---- two-site update on sites k, k+1
                const int k = op.a, dir = op.b;
                const int m = 2 * S.chi[k], n = 2 * S.chi[k + 2];
                SiteView<T> A = site(k), B = site(k + 1);
                if (can_park && max(m, n) > P.park_side) {
                    // ---- hand the update to the batched engine: save the
                    // shot, queue the slot and free the workgroup
                    for (int q = tid; q <= N; q += W) st->chi[q] = S.chi[q];
                    for (int q = tid; q < N; q += W) st->laste[q] = S.laste[q];
                    if (tid == 0) {
                        st->j = j;
                        st->fcur = fcur;
                        st->fend = fend;
                        st->ck_pos = ck_pos;
                        st->n2q = acc.n2q;
                        st->sweeps = acc.sweeps;
                        st->p_acc = p_acc;
                        st->infid = infid;
                        st->disc = acc.disc;
                        st->flops = acc.flops;
                        st->oi = oi + 1;
                        st->next_ch = next_ch;
                        st->fcode = fcode;
                        st->meas_done = meas_done;
                        st->next_seg = next_seg;
                        st->rej_at = rej_at;
                        st->alive = alive ? 1 : 0;
                        st->next_ck = next_ck;
                        st->ck_full = ck_full ? 1 : 0;
                        st->shot_status = acc.status;
                        st->chi_peak = acc.chi_peak;
                        st->k = k;
                        st->dir = dir;
                        st->gate_id = gate_id;
                        st->status = kSlotParked;
                        P.park_list[atomicAdd(P.park_count, 1)] = team;
                    }
                    return;
                }
                // the wavefront kernel's slots hold smaller bonds than
                // chi_max: a shot that outgrows them is handed on (grow)
                const bool grow = P.retry_list != nullptr;
                bool ok = true;
                // a wide update of a one-wavefront team whose vectors fit in
                // the team's whole LDS work area
                const int nvw = dir ? n : m, lenw = dir ? m : n;
                const bool wide_lds = W == 64 && !(m <= SMAX && n <= SMAX) && nvw <= S.n_vmax &&
                                      nvw * (2 * lenw + 1) <= S.n_work;
                if ((m <= SMAX && n <= SMAX) || wide_lds) {
                    if constexpr (W == 64) {
                        ok = twosite_update<T, SMAX, 64>(P, S, A, B, k, dir, gate_id, scr,
                                                         lds_vecs(S), acc, grow,
                                                         wide_lds ? 2 * lenw + 1 : 0);
                    } else if (m <= kWaveSide && n <= kWaveSide) {
                        if (tid < 64)
                            twosite_update<T, SMAX, 64>(P, S, A, B, k, dir, gate_id, scr,
                                                        lds_vecs(S), acc);
                    } else {
                        twosite_update<T, SMAX, NT>(P, S, A, B, k, dir, gate_id, scr, lds_vecs(S),
                                                    acc);
                    }
                } else {
                    // vectors in the slot's scratch after theta's copy
                    const int nv = dir ? n : m, ld = (dir ? m : n) + 1;
                    glbd* vre = to_glb(scr + 2 * (size_t)m * n);
                    const Vecs<glbd*, glbi*> V{vre, vre + (size_t)nv * ld, to_glb(g_nrm),
                                               to_glb(g_isq), to_glb(g_sq), to_glb(g_sel),
                                               to_glb(g_bad), to_glb(g_list)};
                    ok = twosite_update<T, SMAX, W>(P, S, A, B, k, dir, gate_id, scr, V, acc, grow);
                }
                Team<W>::sync();
                if (!ok) {
                    // a larger slot is needed: the shot is queued for the
                    // workgroup kernel, which runs it again from its start
                    if (tid == 0) P.retry_list[atomicAdd(P.retry_count, 1)] = it;
                    retried = true;
                    break;
                }
            }
        }
        if (tid == 0 && !retried) {
            if (kExtra && P.surv)
                for (int g = next_seg; g < P.n_seg; ++g) P.surv[it * P.n_seg + g] = p_acc;
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
        Team<W>::sync();
    }
    if (st && tid == 0) st->status = kSlotDone;
}

template <typename T, int SMAX>
__global__ __launch_bounds__(NT, (kMpsWavesPerSimd<T, SMAX>)) void mps_kernel(MpsArgs P) {
    __shared__ int s_chi[kMaxSites + 1];
    __shared__ int s_laste[kMaxSites];
    __shared__ double s_vre[SMAX * (SMAX + 1)];
    __shared__ double s_vim[SMAX * (SMAX + 1)];
    __shared__ double s_nrm[SMAX];
    __shared__ double s_isq[SMAX];
    __shared__ double s_sq[SMAX];
    __shared__ int s_sel[SMAX];
    __shared__ int s_bad[SMAX];
    __shared__ int s_list[SMAX];
    __shared__ int s_ired[NW];
    __shared__ double s_red[NW * 4];
    __shared__ int s_flag[1];
    // gate tables, per-site layout of the slot and bond caps, read once
    __shared__ double s_g1[G1_COUNT * 8];
    __shared__ int s_g4src[G4_COUNT * 4];
    __shared__ double s_g4ph[G4_COUNT * 8];
    __shared__ int32_t s_soff[kMaxSites];    // offsets within a slot (< 2^31 elements)
    __shared__ int32_t s_shalf[kMaxSites];
    __shared__ int s_cap[kMaxSites + 1];
    // op descriptors, kOpBuf at a time
    __shared__ DevOp s_ops[kOpBuf];
    // staging: the two site tensors of an update (tensor type), then the
    // copy of theta kept for the projection (FP64)
    __shared__ __align__(16) double s_u[kStage];

    const int tid = threadIdx.x;

    for (int k = tid; k < P.n_sites; k += NT) {
        s_soff[k] = P.site_off[k];
        s_shalf[k] = P.site_half[k];
    }
    for (int k = tid; k <= P.n_sites; k += NT) s_cap[k] = P.cap[k];
    for (int i = tid; i < G1_COUNT * 8; i += NT) s_g1[i] = P.g1[i];
    if (tid < G4_COUNT * 4) {
        // the nonzero of each row of each monomial 4x4 gate, found once
        const double* g = P.g4 + (tid >> 2) * 32 + (tid & 3) * 8;
        int src = 0;
        for (int j = 1; j < 4; ++j)
            if (fabs(g[2 * j]) + fabs(g[2 * j + 1]) > fabs(g[2 * src]) + fabs(g[2 * src + 1]))
                src = j;
        s_g4src[tid] = src;
        s_g4ph[2 * tid] = g[2 * src];
        s_g4ph[2 * tid + 1] = g[2 * src + 1];
    }
    __syncthreads();

    Smem S;
    S.chi = s_chi;
    S.vre = s_vre;
    S.vim = s_vim;
    S.nrm = s_nrm;
    S.isq = s_isq;
    S.sq = s_sq;
    S.sel = s_sel;
    S.bad = s_bad;
    S.list = s_list;
    S.ired = s_ired;
    S.red = s_red;
    S.cap = s_cap;
    S.u = s_u;
    S.g4src = s_g4src;
    S.g4ph = s_g4ph;
    S.laste = s_laste;
    S.flag = s_flag;
    S.ops = s_ops;
    S.soff = s_soff;
    S.shalf = s_shalf;
    S.g1 = s_g1;
    S.n_u = kStage;
    run_team<T, SMAX, NT, kOpBuf>(P, S, blockIdx.x, gridDim.x);
}


// One shot per wavefront, four per workgroup, for shots whose bonds stay
// small: no workgroup barrier after the tables are loaded, so the waves of a
// workgroup run their shots independently and a CU holds twelve resident
// shots instead of four.  The slots' bonds are capped below chi_max; a shot
// that outgrows them is queued (retry_list) and run again from its start by
// the workgroup kernel.  Factorisations with both theta sides <= kWaveSmax
// keep their vectors in LDS; wider ones (up to twice the slot's bond cap)
// take the wavefront's whole LDS work area when their nv vectors of length
// len fit in it at a stride of 2 len + 1 doubles, else the slot's scratch.
constexpr int kWaveSmax = 16;
constexpr int kWaveOps = 16;
constexpr int kWaveStage = 512;
constexpr int kWaveVec = kWaveSmax * (kWaveSmax + 1);     // doubles per plane, small sides
constexpr int kWaveWork = 2 * kWaveVec + kWaveStage;      // vectors + staging
constexpr int kWaveMaxV = 2 * kWaveSmax;                  // vectors of a wide update

template <typename T, bool EXTRA>
__global__ __launch_bounds__(NT, 3) void mps_wave_kernel(MpsArgs P) {
    // per wavefront
    __shared__ int s_chi[NW][kMaxSites + 1];
    __shared__ int s_laste[NW][kMaxSites];
    // the SVD vectors of small sides (planar) and the staging area, one
    // contiguous work area that a wide factorisation takes whole
    __shared__ __align__(16) double s_work[NW][kWaveWork];
    __shared__ double s_nrm[NW][kWaveMaxV];
    __shared__ double s_isq[NW][kWaveMaxV];
    __shared__ double s_sq[NW][kWaveMaxV];
    __shared__ int s_sel[NW][kWaveMaxV];
    __shared__ int s_bad[NW][kWaveMaxV];
    __shared__ int s_list[NW][kWaveMaxV];
    __shared__ int s_flag[NW][1];
    __shared__ DevOp s_ops[NW][kWaveOps];
    // per workgroup, read-only after the start
    __shared__ double s_g1[G1_COUNT * 8];
    __shared__ int s_g4src[G4_COUNT * 4];
    __shared__ double s_g4ph[G4_COUNT * 8];
    __shared__ int32_t s_soff[kMaxSites];
    __shared__ int32_t s_shalf[kMaxSites];
    __shared__ int s_cap[kMaxSites + 1];

    const int tid = threadIdx.x;
    for (int k = tid; k < P.n_sites; k += NT) {
        s_soff[k] = P.site_off[k];
        s_shalf[k] = P.site_half[k];
    }
    for (int k = tid; k <= P.n_sites; k += NT) s_cap[k] = P.cap[k];
    for (int i = tid; i < G1_COUNT * 8; i += NT) s_g1[i] = P.g1[i];
    if (tid < G4_COUNT * 4) {
        const double* g = P.g4 + (tid >> 2) * 32 + (tid & 3) * 8;
        int src = 0;
        for (int j = 1; j < 4; ++j)
            if (fabs(g[2 * j]) + fabs(g[2 * j + 1]) > fabs(g[2 * src]) + fabs(g[2 * src + 1]))
                src = j;
        s_g4src[tid] = src;
        s_g4ph[2 * tid] = g[2 * src];
        s_g4ph[2 * tid + 1] = g[2 * src + 1];
    }
    __syncthreads();
    // the wavefront's index, as a scalar: its LDS arrays and slot are then
    // addressed with scalar registers
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    Smem S;
    S.chi = s_chi[w];
    S.laste = s_laste[w];
    S.vre = s_work[w];
    S.vim = s_work[w] + kWaveVec;
    S.nrm = s_nrm[w];
    S.isq = s_isq[w];
    S.sq = s_sq[w];
    S.sel = s_sel[w];
    S.bad = s_bad[w];
    S.list = s_list[w];
    S.ired = nullptr;   // one-wavefront teams reduce in registers
    S.red = nullptr;
    S.flag = s_flag[w];
    S.ops = s_ops[w];
    S.u = s_work[w] + 2 * kWaveVec;
    S.n_u = kWaveStage;
    S.n_work = kWaveWork;
    S.n_vmax = kWaveMaxV;
    S.cap = s_cap;
    S.g4src = s_g4src;
    S.g4ph = s_g4ph;
    S.soff = s_soff;
    S.shalf = s_shalf;
    S.g1 = s_g1;
    run_team<T, kWaveSmax, 64, kWaveOps, EXTRA>(P, S, blockIdx.x * NW + w, gridDim.x * NW);
}

// ---------------------------------------------------------------------------
// Factor step of the batched engine for large two-site updates (the
// contraction and the Gram matrix come from lx.hip).  One workgroup per
// parked shot, with theta (tensor type T) and G = V^H V (FP64) of its
// vectors V (theta's columns when the centre moves right, rows when left):
//  * the vectors' squared norms are G's diagonal; a pair (p, q) overlaps if
//    |G_pq|^2 > tol^2 G_pp G_qq (the same test and tolerance as the shot
//    kernel's orthogonality check); the flagged vectors F are those of an
//    overlapping pair, the others are already orthogonal to everything;
//  * if |F| <= kLxFactorMax the block G_FF is diagonalised in LDS by cyclic
//    two-sided Jacobi in FP64, W^H G_FF W = diag, and the rotated vectors
//    Y = X_F W are formed in FP64 from theta; their squared norms are taken
//    from Y itself, so a direction of G's null space gets a norm of order
//    eps |X| rather than the sqrt(eps) |X| its eigenvalue carries.  Since X_F
//    = Y W^H, theta = sum_u y_u conj(W[:, u])^T: the isometric factor is
//    y_u / sigma_u and the centre factor's row (column) u is sigma_u
//    conj(W[:, u]) on F (sigma_u e_v for an unflagged vector v), with no
//    second product;
//  * otherwise the flagged vectors are orthogonalised by one-sided Jacobi
//    sweeps in the workspace (as the shot kernel does for wide theta) and the
//    centre factor is the projection of theta on the isometric factor;
//  * the kept vectors (sigma_u > tau sigma_0, at most the bond cap) are
//    written as the new A[k], A[k+1] in FP64-renormalised form, the slot's
//    state gets the new bond and counters and is marked for resumption.
// Two-sided Jacobi on a Hermitian pair block [[a, g], [conj(g), b]]: with
// g = |g| e^{i phi}, zeta = (b - a) / (2 |g|), t = sign(zeta) / (|zeta| +
// sqrt(1 + zeta^2)), c = 1 / sqrt(1 + t^2), s = c t, the unitary
// J = diag(1, e^{-i phi}) [[c, s], [-s, c]] makes J^H A J diagonal (the
// phase makes the pair's off-diagonal real, the real rotation removes it).
constexpr int FM = kLxFactorMax;
constexpr int FLD = FM + 1;

template <typename T>
__global__ __launch_bounds__(NT) void lx_factor_kernel(LxArgs a, LxFactor f) {
    __shared__ double s_gr[FM * FLD], s_gi[FM * FLD];   // G_FF, then staging
    __shared__ double s_wr[FM * FLD], s_wi[FM * FLD];   // W
    __shared__ double s_pc[FM / 2], s_ps[FM / 2], s_pr[FM / 2], s_pi[FM / 2];
    __shared__ int s_pp[FM / 2], s_pq[FM / 2];
    __shared__ double s_red[NW * 4];
    __shared__ int s_ired[NW];
    __shared__ int s_any;
    const int tid = threadIdx.x;
    const LxPlan* pl = a.plan;
    const int cnt = pl->count;
    for (int pi = blockIdx.x; pi < cnt; pi += gridDim.x) {
        const int slot = pl->slot[pi];
        ShotState* st = const_cast<ShotState*>(a.state) + slot;
        const int k = st->k, dir = st->dir;
        const int cl = st->chi[k], cm = st->chi[k + 1], cr = st->chi[k + 2];
        const int m = 2 * cl, n = 2 * cr;
        const int nv = dir ? n : m, len = dir ? m : n;
        typedef __attribute__((address_space(1))) T gT;
        const gT* Tr = to_glb(static_cast<const T*>(a.theta) + (size_t)slot * a.theta_stride);
        const gT* Ti = Tr + (size_t)m * n;
        glbd* G = to_glb(a.gram + (size_t)slot * a.gram_stride);
        const glbd* Gr = G;
        const glbd* Gi = G + (size_t)nv * nv;
        // per-vector arrays after the workspace (sides up to smax = 2 chi_max)
        const int64_t smax = 2 * (int64_t)f.chi_max;
        glbd* d = G + 2 * smax * (smax + 1);
        glbd* nrm = d + smax;
        glbd* isq = nrm + smax;
        glbd* sq = isq + smax;
        glbi* sel = reinterpret_cast<glbi*>(sq + smax);
        glbi* bad = sel + smax;
        glbi* list = bad + smax;
        glbi* fpos = list + smax;
        // the slot's site tensors
        T* base = static_cast<T*>(a.arena) + (size_t)slot * a.slot_stride;
        gT* Are = to_glb(base + a.site_off[k]);
        gT* Aim = Are + a.site_half[k];
        gT* Bre = to_glb(base + a.site_off[k + 1]);
        gT* Bim = Bre + a.site_half[k + 1];
        auto X = [&](int v, int e, int plane) -> double {   // vector v, element e
            const size_t at = dir ? (size_t)e * n + v : (size_t)v * n + e;
            return static_cast<double>(plane ? Ti[at] : Tr[at]);
        };

        // ---- norms and the overlap flags from G
        double tot[1] = {0.0};
        for (int v = tid; v < nv; v += NT) {
            const double x = Gr[(size_t)v * nv + v];
            d[v] = x;
            bad[v] = 0;
            tot[0] += x;
        }
        team_sum<NT, 1>(tot, s_red);
        const double total = tot[0];
        const double tau2 = f.tau * f.tau;
        const double floor2 = 1e-4 * tau2 * total;
        const double tol = sizeof(T) == sizeof(double) ? static_cast<double>(len) * DBL_EPSILON
                                                       : 8.0 * static_cast<double>(FLT_EPSILON);
        const double tol2 = tol * tol;
        __syncthreads();
        {
            const int npair = nv * (nv - 1) / 2;
            int p = 0, rowlen = nv - 1, t0 = 0;
            for (int t = tid; t < npair; t += NT) {
                while (t >= t0 + rowlen) {
                    t0 += rowlen;
                    ++p;
                    --rowlen;
                }
                const int q = p + 1 + (t - t0);
                const double dp = d[p], dq = d[q];
                if (!(dp > floor2 && dq > floor2)) continue;
                const double gr = Gr[(size_t)p * nv + q], gi = Gi[(size_t)p * nv + q];
                if (gr * gr + gi * gi > tol2 * dp * dq) {
                    bad[p] = 1;   // benign race: every writer stores 1
                    bad[q] = 1;
                }
            }
        }
        __syncthreads();
        const int nf = flagged_list<NT>(bad, nv, list, s_ired);
        for (int v = tid; v < nv; v += NT) fpos[v] = -1;
        __syncthreads();
        for (int j = tid; j < nf; j += NT) fpos[list[j]] = j;
        int sweeps = 0;
        bool noconv = false;
        bool polished = false;   // Y rotated after the eigen-decomposition
        const bool small = nf <= FM;
        // workspace of the rotated vectors: planar FP64, vector j at j * ldy
        const int ldy = len + 1;
        glbd* Yr = G;
        glbd* Yi = G + (size_t)nf * ldy;
        if (nf > 0 && small) {
            // ---- G_FF into LDS (Hermitian from the upper triangle), W = I
            for (int idx = tid; idx < nf * nf; idx += NT) {
                const int r = idx / nf, c = idx - r * nf;
                const int p = list[r], q = list[c];
                double gr, gi;
                if (p <= q) {
                    gr = Gr[(size_t)p * nv + q];
                    gi = Gi[(size_t)p * nv + q];
                } else {
                    gr = Gr[(size_t)q * nv + p];
                    gi = -Gi[(size_t)q * nv + p];
                }
                if (p == q) gi = 0.0;
                s_gr[r * FLD + c] = gr;
                s_gi[r * FLD + c] = gi;
                s_wr[r * FLD + c] = r == c ? 1.0 : 0.0;
                s_wi[r * FLD + c] = 0.0;
            }
            __syncthreads();
            // ---- cyclic two-sided Jacobi, round-robin pairs
            const int nve = nf + (nf & 1);
            const int npairs = nve / 2;
            bool again = true;
            while (again && sweeps < 40) {
                if (tid == 0) s_any = 0;
                __syncthreads();
                for (int t = 0; t < nve - 1; ++t) {
                    if (tid < npairs) {
                        const int sp = player(tid, t, nve), sq2 = player(nve - 1 - tid, t, nve);
                        double c = 1.0, sn = 0.0, er = 1.0, ei = 0.0;
                        int p = -1, q = -1;
                        if (sp < nf && sq2 < nf) {
                            p = sp < sq2 ? sp : sq2;
                            q = sp < sq2 ? sq2 : sp;
                            const double aa = s_gr[p * FLD + p], bb = s_gr[q * FLD + q];
                            const double gr = s_gr[p * FLD + q], gi = s_gi[p * FLD + q];
                            const double g2 = gr * gr + gi * gi;
                            if (aa > floor2 && bb > floor2 && g2 > tol2 * aa * bb) {
                                // e = exp(-i phi): the columns take J's e^{-i phi},
                                // the rows its conjugate
                                const double ga = sqrt(g2);
                                er = gr / ga;
                                ei = -gi / ga;
                                const double zeta = (bb - aa) / (2.0 * ga);
                                const double tt = (zeta >= 0.0 ? 1.0 : -1.0) /
                                                  (fabs(zeta) + sqrt(1.0 + zeta * zeta));
                                c = 1.0 / sqrt(1.0 + tt * tt);
                                sn = c * tt;
                                s_any = 1;
                            } else {
                                p = -1;
                            }
                        }
                        s_pp[tid] = p;
                        s_pq[tid] = q;
                        s_pc[tid] = c;
                        s_ps[tid] = sn;
                        s_pr[tid] = er;
                        s_pi[tid] = ei;
                    }
                    __syncthreads();
                    // columns: A <- A J and W <- W J
                    for (int idx = tid; idx < npairs * nf; idx += NT) {
                        const int pr = idx / nf, r = idx - pr * nf;
                        const int p = s_pp[pr];
                        if (p < 0) continue;
                        const int q = s_pq[pr];
                        const double c = s_pc[pr], sn = s_ps[pr], er = s_pr[pr], ei = s_pi[pr];
                        for (int mat = 0; mat < 2; ++mat) {
                            double* Mr = mat ? s_wr : s_gr;
                            double* Mi = mat ? s_wi : s_gi;
                            const double xr = Mr[r * FLD + p], xi = Mi[r * FLD + p];
                            const double yr = Mr[r * FLD + q], yi = Mi[r * FLD + q];
                            // e y
                            const double eyr = er * yr - ei * yi, eyi = er * yi + ei * yr;
                            Mr[r * FLD + p] = c * xr - sn * eyr;
                            Mi[r * FLD + p] = c * xi - sn * eyi;
                            Mr[r * FLD + q] = sn * xr + c * eyr;
                            Mi[r * FLD + q] = sn * xi + c * eyi;
                        }
                    }
                    __syncthreads();
                    // rows: A <- J^H A
                    for (int idx = tid; idx < npairs * nf; idx += NT) {
                        const int pr = idx / nf, col = idx - pr * nf;
                        const int p = s_pp[pr];
                        if (p < 0) continue;
                        const int q = s_pq[pr];
                        const double c = s_pc[pr], sn = s_ps[pr], er = s_pr[pr], ei = -s_pi[pr];
                        const double xr = s_gr[p * FLD + col], xi = s_gi[p * FLD + col];
                        const double yr = s_gr[q * FLD + col], yi = s_gi[q * FLD + col];
                        // conj(e) y
                        const double eyr = er * yr - ei * yi, eyi = er * yi + ei * yr;
                        s_gr[p * FLD + col] = c * xr - sn * eyr;
                        s_gi[p * FLD + col] = c * xi - sn * eyi;
                        s_gr[q * FLD + col] = sn * xr + c * eyr;
                        s_gi[q * FLD + col] = sn * xi + c * eyi;
                    }
                    __syncthreads();
                }
                ++sweeps;
                again = s_any != 0;
                __syncthreads();
            }
            noconv = again;
            // ---- Y = X_F W in FP64, 64 elements of every flagged vector staged
            // in LDS (the G_FF arrays are free now)
            for (int e0 = 0; e0 < len; e0 += FM) {
                const int ne = min(FM, len - e0);
                for (int idx = tid; idx < nf * ne; idx += NT) {
                    const int j = idx / ne, e = idx - j * ne;
                    s_gr[j * FLD + e] = X(list[j], e0 + e, 0);
                    s_gi[j * FLD + e] = X(list[j], e0 + e, 1);
                }
                __syncthreads();
                for (int idx = tid; idx < nf * ne; idx += NT) {
                    const int i = idx / ne, e = idx - i * ne;
                    double yr = 0.0, yi = 0.0;
                    for (int j = 0; j < nf; ++j) {
                        const double xr = s_gr[j * FLD + e], xi = s_gi[j * FLD + e];
                        const double wr = s_wr[j * FLD + i], wi = s_wi[j * FLD + i];
                        yr += xr * wr - xi * wi;
                        yi += xr * wi + xi * wr;
                    }
                    Yr[(size_t)i * ldy + e0 + e] = yr;
                    Yi[(size_t)i * ldy + e0 + e] = yi;
                }
                __syncthreads();
            }
            // ---- polish Y: eigenvectors of G leave the rotated vectors
            // orthogonal only to about eps |G| / (sigma_u sigma_v), and a
            // null-space direction with a norm near eps sigma_0^3 /
            // sigma_min^2, which can pass the exact regime's threshold; one-
            // sided Jacobi on Y (quadratically convergent from here) brings
            // both to the tensor precision's resolution.  The centre factor
            // is then the projection of theta on the isometric factor.
            for (int j = tid; j < nf; j += NT) sel[j] = j;
            __syncthreads();
            vector_norms<NT>(Yr, Yi, nf, len, ldy, nrm);
            bool again2 = not_orthogonal<NT>(Yr, Yi, nf, len, ldy, nrm, floor2, tol, bad,
                                             (glbi*)nullptr);
            polished = again2;
            int psweeps = 0;
            while (again2 && psweeps < 40) {
                const int nb2 = flagged_list<NT>(bad, nf, sel, s_ired);
                jacobi_sweep<NT>(Yr, Yi, sel, nb2, len, ldy, floor2, tol);
                ++psweeps;
                vector_norms<NT>(Yr, Yi, nf, len, ldy, nrm);
                again2 = not_orthogonal<NT>(Yr, Yi, nf, len, ldy, nrm, floor2, tol, bad,
                                            (glbi*)nullptr);
            }
            sweeps += psweeps;
            noconv = noconv || again2;
        } else if (nf > 0) {
            // ---- many overlapping vectors: one-sided Jacobi in the workspace
            for (int idx = tid; idx < nf * len; idx += NT) {
                const int j = idx / len, e = idx - j * len;
                Yr[(size_t)j * ldy + e] = X(list[j], e, 0);
                Yi[(size_t)j * ldy + e] = X(list[j], e, 1);
            }
            for (int j = tid; j < nf; j += NT) sel[j] = j;   // identity list
            __syncthreads();
            vector_norms<NT>(Yr, Yi, nf, len, ldy, nrm);
            bool again = true;
            for (int j = tid; j < nf; j += NT) bad[j] = 1;
            __syncthreads();
            while (again && sweeps < 40) {
                const int nb2 = flagged_list<NT>(bad, nf, sel, s_ired);
                jacobi_sweep<NT>(Yr, Yi, sel, nb2, len, ldy, floor2, tol);
                ++sweeps;
                vector_norms<NT>(Yr, Yi, nf, len, ldy, nrm);
                again = not_orthogonal<NT>(Yr, Yi, nf, len, ldy, nrm, floor2, tol, bad,
                                           (glbi*)nullptr);
            }
            noconv = again;
        }
        __syncthreads();
        // ---- squared norms of all vectors (rotated ones from Y itself)
        for (int v = tid; v < nv; v += NT) {
            const int j = fpos[v];
            if (j < 0) {
                nrm[v] = d[v];
            } else {
                double s0 = 0.0, s1 = 0.0;
                const glbd* yr = Yr + (size_t)j * ldy;
                const glbd* yi = Yi + (size_t)j * ldy;
                for (int e = 0; e < len; ++e) {
                    s0 += yr[e] * yr[e];
                    s1 += yi[e] * yi[e];
                }
                nrm[v] = s0 + s1;
            }
        }
        __syncthreads();
        const int capb = min(f.chi_max, f.cap[k + 1]);
        const Kept kp = select_kept<NT>(nrm, nv, tau2, capb, sel, isq, sq, s_red);
        const int r = kp.r;
        const double renorm = 1.0 / sqrt(kp.kept);
        // ---- isometric factor: the kept vectors, normalised
        // (element e of kept vector c)
        auto kept_elem = [&](int c, int e, double& xr, double& xi) {
            const int v = sel[c];
            const int j = fpos[v];
            if (j < 0) {
                xr = X(v, e, 0);
                xi = X(v, e, 1);
            } else {
                xr = Yr[(size_t)j * ldy + e];
                xi = Yi[(size_t)j * ldy + e];
            }
        };
        if (dir) {
            for (int idx = tid; idx < m * r; idx += NT) {
                const int row = idx / r, c = idx - row * r;
                double xr, xi;
                kept_elem(c, row, xr, xi);
                Are[idx] = T(xr * isq[c]);
                Aim[idx] = T(xi * isq[c]);
            }
        } else {
            for (int idx = tid; idx < r * n; idx += NT) {
                const int c = idx / n, col = idx - c * n;
                double xr, xi;
                kept_elem(c, col, xr, xi);
                Bre[idx] = T(xr * isq[c]);
                Bim[idx] = T(xi * isq[c]);
            }
        }
        // ---- centre factor
        if (nf == 0 || (small && !polished)) {
            // sigma_u conj(W[:, u]) on the flagged positions, sigma_u e_v for
            // an unflagged vector v (entry (u, v) of Sigma W~^H)
            auto centre = [&](int c, int v, double& xr, double& xi) {
                const int u = sel[c];
                const int ju = fpos[u], jv = fpos[v];
                const double sc = sq[c] * renorm;
                if (ju < 0) {
                    xr = v == u ? sc : 0.0;
                    xi = 0.0;
                } else if (jv < 0) {
                    xr = 0.0;
                    xi = 0.0;
                } else {
                    xr = sc * s_wr[jv * FLD + ju];
                    xi = -sc * s_wi[jv * FLD + ju];
                }
            };
            if (dir) {
                for (int idx = tid; idx < r * n; idx += NT) {
                    const int c = idx / n, col = idx - c * n;
                    double xr, xi;
                    centre(c, col, xr, xi);
                    Bre[idx] = T(xr);
                    Bim[idx] = T(xi);
                }
            } else {
                for (int idx = tid; idx < m * r; idx += NT) {
                    const int row = idx / r, c = idx - row * r;
                    double xr, xi;
                    centre(c, row, xr, xi);
                    Are[idx] = T(xr);
                    Aim[idx] = T(xi);
                }
            }
        } else {
            // projection of theta on the isometric factor just written
            __syncthreads();
            if (dir) {
                // A[k+1][c][col] = sum_row conj(U[row][c]) theta[row][col]
                for (int idx = tid; idx < r * n; idx += NT) {
                    const int c = idx / n, col = idx - c * n;
                    double xr = 0.0, xi = 0.0;
                    for (int row = 0; row < m; ++row) {
                        const double ur = static_cast<double>(Are[row * r + c]);
                        const double ui = static_cast<double>(Aim[row * r + c]);
                        const double tr = X(col, row, 0), ti = X(col, row, 1);
                        xr += ur * tr + ui * ti;
                        xi += ur * ti - ui * tr;
                    }
                    Bre[idx] = T(xr * renorm);
                    Bim[idx] = T(xi * renorm);
                }
            } else {
                // A[k][row][c] = sum_col theta[row][col] conj(V[c][col])
                for (int idx = tid; idx < m * r; idx += NT) {
                    const int row = idx / r, c = idx - row * r;
                    double xr = 0.0, xi = 0.0;
                    for (int col = 0; col < n; ++col) {
                        const double vr = static_cast<double>(Bre[c * n + col]);
                        const double vi = static_cast<double>(Bim[c * n + col]);
                        const double tr = X(row, col, 0), ti = X(row, col, 1);
                        xr += tr * vr + ti * vi;
                        xi += ti * vr - tr * vi;
                    }
                    Are[idx] = T(xr * renorm);
                    Aim[idx] = T(xi * renorm);
                }
            }
        }
        // ---- the slot's state: new bond, counters, resume
        if (tid == 0) {
            atomicAdd(a.counts + (small ? 0 : 1), 1ull);
            atomicAdd(a.counts + 2, static_cast<unsigned long long>(nf));
            atomicAdd(a.counts + 3, static_cast<unsigned long long>(sweeps));
            st->chi[k + 1] = r;
            st->disc += kp.dropped;
            if (kp.dropped > 1e-12 * total && r == capb) st->shot_status |= MSC_SHOT_CHI_CAP;
            if (noconv) st->shot_status |= MSC_SHOT_NOCONV;
            st->sweeps += sweeps;
            st->chi_peak = max(st->chi_peak, r);
            st->n2q += 1;
            const double dl = cl, dm = cm, dr = cr, dk = r;
            st->flops += 32.0 * dl * dm * dr + 32.0 * dl * dl * dr + 32.0 * dk * dl * dr +
                         104.0 * dl * dl * dl;
            st->status = kSlotResume;
        }
        __syncthreads();
    }
}

// Processing order of the shots: a stable counting sort into 16 buckets,
// the longest-running shots first so that the tail of the persistent grid
// stays short.  Without checkpoints the key is the fault count (capped at
// 15): low-weight shots are the ones that run to the end of the circuit,
// online screening stops the others early.  With checkpoints a shot starts
// at its first fault, so the key is the position of that channel in the
// circuit (fault-free shots, which only read out, last).
// Three launches over chunks of kOrderChunk entries: per-chunk key counts,
// one exclusive scan of them in (key, chunk) order, and a stable scatter in
// which each workgroup ranks its chunk's entries by ballots.
constexpr int OT = 256;
constexpr int kOrderItems = 16;
constexpr int kOrderChunk = OT * kOrderItems;

__device__ __forceinline__ int order_key(int64_t j, const int64_t* shot_off,
                                         const int64_t* shot_idx, int64_t n_csr,
                                         const int32_t* chan, int32_t n_channels) {
    const int64_t sh = shot_idx ? shot_idx[j] : j;
    int c = 15;
    if (sh >= 0 && sh < n_csr) {
        const int64_t f0 = shot_off[sh], f = shot_off[sh + 1] - f0;
        if (n_channels > 0) {
            const int64_t ch = f > 0 ? chan[f0] : n_channels;
            c = ch < 0 ? 0 : ch >= n_channels ? 15 : static_cast<int>(ch * 15 / n_channels);
        } else {
            c = f < 15 ? static_cast<int>(f) : 15;
        }
    }
    return c;
}

// cnt[key * nblk + block]: entries of the chunk with that key
__global__ __launch_bounds__(OT) void order_count_kernel(int64_t n, const int64_t* n_dev,
                                                         const int64_t* shot_off,
                                                         const int64_t* shot_idx, int64_t n_csr,
                                                         const int32_t* chan, int32_t n_channels,
                                                         int32_t* cnt, int nblk) {
    __shared__ int s_cnt[16];
    if (n_dev && *n_dev < n) n = *n_dev;
    const int tid = threadIdx.x;
    if (tid < 16) s_cnt[tid] = 0;
    __syncthreads();
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kOrderChunk;
    for (int i = 0; i < kOrderItems; ++i) {
        const int64_t j = j0 + static_cast<int64_t>(i) * OT + tid;
        if (j < n) atomicAdd(&s_cnt[order_key(j, shot_off, shot_idx, n_csr, chan, n_channels)], 1);
    }
    __syncthreads();
    if (tid < 16) cnt[tid * nblk + blockIdx.x] = s_cnt[tid];
}

// base[e] = sum of cnt[0 .. e) over the 16 * nblk entries (one workgroup)
__global__ __launch_bounds__(OT) void order_scan_kernel(const int32_t* cnt, int64_t* base,
                                                        int64_t total) {
    __shared__ int64_t s_part[OT];
    const int tid = threadIdx.x;
    const int64_t per = (total + OT - 1) / OT;
    const int64_t e0 = min(total, tid * per), e1 = min(total, e0 + per);
    int64_t sum = 0;
    for (int64_t e = e0; e < e1; ++e) sum += cnt[e];
    s_part[tid] = sum;
    __syncthreads();
    if (tid == 0) {
        int64_t run = 0;
        for (int q = 0; q < OT; ++q) {
            const int64_t v = s_part[q];
            s_part[q] = run;
            run += v;
        }
    }
    __syncthreads();
    int64_t run = s_part[tid];
    for (int64_t e = e0; e < e1; ++e) {
        base[e] = run;
        run += cnt[e];
    }
}

// perm[base + rank] = j for the chunk's entries, in index order per key
__global__ __launch_bounds__(OT) void order_scatter_kernel(int64_t n, const int64_t* n_dev,
                                                           const int64_t* shot_off,
                                                           const int64_t* shot_idx,
                                                           int64_t n_csr, const int32_t* chan,
                                                           int32_t n_channels,
                                                           const int64_t* base, int nblk,
                                                           int64_t* perm) {
    __shared__ int64_t s_base[16];
    __shared__ int s_wc[OT / 64][16];
    if (n_dev && *n_dev < n) n = *n_dev;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid < 16) s_base[tid] = base[tid * nblk + blockIdx.x];
    __syncthreads();
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kOrderChunk;
    const uint64_t below = (1ull << lane) - 1ull;
    for (int i = 0; i < kOrderItems; ++i) {
        const int64_t j = j0 + static_cast<int64_t>(i) * OT + tid;
        const int key = j < n ? order_key(j, shot_off, shot_idx, n_csr, chan, n_channels) : -1;
        uint64_t mine = 0;
        int wc = 0;
        for (int k = 0; k < 16; ++k) {
            const uint64_t m = __ballot(key == k);
            if (key == k) mine = m;
            if (lane == k) wc = __popcll(m);
        }
        if (lane < 16) s_wc[w][lane] = wc;
        __syncthreads();
        if (key >= 0) {
            int64_t pos = s_base[key];
            for (int q = 0; q < w; ++q) pos += s_wc[q][key];
            perm[pos + __popcll(mine & below)] = j;
        }
        __syncthreads();
        if (tid < 16) {
            int t = 0;
            for (int q = 0; q < OT / 64; ++q) t += s_wc[q][tid];
            s_base[tid] += t;
        }
        __syncthreads();
    }
}

}  // namespace

int mps_blocks_per_cu(int precision, bool small) {
    int b = 0;
    hipError_t e;
    if (precision == MSC_FP64)
        e = small ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, mps_kernel<double, 32>, NT, 0)
                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, mps_kernel<double, 64>, NT, 0);
    else
        e = small ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, mps_kernel<float, 32>, NT, 0)
                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, mps_kernel<float, 64>, NT, 0);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return b < 1 ? 1 : b;
}

int mps_wave_blocks_per_cu(int precision) {
    int b = 0;
    hipError_t e = precision == MSC_FP64
                       ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, mps_wave_kernel<double, true>, NT, 0)
                       : hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, mps_wave_kernel<float, true>, NT, 0);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return b < 1 ? 1 : b;
}

hipError_t launch_mps_wave(int precision, const MpsArgs& a, int grid, hipStream_t s) {
    static_assert(kWaveTeams == NW, "one team per wavefront");
    if (!a.next || !a.retry_count || !a.retry_list || a.calibrate || a.state)
        return hipErrorInvalidValue;
    // the kernel without checkpoint recording and segment reach when the
    // run needs neither (the benchmark's): fewer arguments held in registers
    const bool extra = a.surv != nullptr || a.ck_mode == 1;
    if (precision == MSC_FP64) {
        if (extra) hipLaunchKernelGGL((mps_wave_kernel<double, true>), dim3(grid), dim3(NT), 0, s, a);
        else hipLaunchKernelGGL((mps_wave_kernel<double, false>), dim3(grid), dim3(NT), 0, s, a);
    } else {
        if (extra) hipLaunchKernelGGL((mps_wave_kernel<float, true>), dim3(grid), dim3(NT), 0, s, a);
        else hipLaunchKernelGGL((mps_wave_kernel<float, false>), dim3(grid), dim3(NT), 0, s, a);
    }
    return hipGetLastError();
}

int64_t order_tmp_bytes(int64_t n) {
    const int64_t nblk = (std::max<int64_t>(n, 1) + kOrderChunk - 1) / kOrderChunk;
    return 16 * nblk * static_cast<int64_t>(sizeof(int32_t) + sizeof(int64_t));
}

hipError_t launch_order(int64_t n, const int64_t* n_dev, const int64_t* shot_off,
                        const int64_t* shot_idx, int64_t n_csr, const int32_t* chan,
                        int32_t n_channels, int64_t* perm, void* tmp, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t nblk = (n + kOrderChunk - 1) / kOrderChunk;
    if (nblk > (int64_t(1) << 24)) return hipErrorInvalidValue;
    int64_t* base = static_cast<int64_t*>(tmp);
    int32_t* cnt = reinterpret_cast<int32_t*>(base + 16 * nblk);
    const int nb = static_cast<int>(nblk);
    hipLaunchKernelGGL(order_count_kernel, dim3(nb), dim3(OT), 0, s, n, n_dev, shot_off, shot_idx,
                       n_csr, chan, n_channels, cnt, nb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(order_scan_kernel, dim3(1), dim3(OT), 0, s, cnt, base, 16 * nblk);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(order_scatter_kernel, dim3(nb), dim3(OT), 0, s, n, n_dev, shot_off,
                       shot_idx, n_csr, chan, n_channels, base, nb, perm);
    return hipGetLastError();
}

hipError_t launch_lx_factor(int precision, const LxArgs& a, const LxFactor& f, int grid,
                            hipStream_t s) {
    if (precision == MSC_FP64)
        hipLaunchKernelGGL(lx_factor_kernel<double>, dim3(grid), dim3(NT), 0, s, a, f);
    else
        hipLaunchKernelGGL(lx_factor_kernel<float>, dim3(grid), dim3(NT), 0, s, a, f);
    return hipGetLastError();
}

hipError_t launch_mps(int precision, bool small, const MpsArgs& a, int grid, hipStream_t s) {
    if (precision == MSC_FP64) {
        if (small) hipLaunchKernelGGL((mps_kernel<double, 32>), dim3(grid), dim3(NT), 0, s, a);
        else hipLaunchKernelGGL((mps_kernel<double, 64>), dim3(grid), dim3(NT), 0, s, a);
    } else {
        if (small) hipLaunchKernelGGL((mps_kernel<float, 32>), dim3(grid), dim3(NT), 0, s, a);
        else hipLaunchKernelGGL((mps_kernel<float, 64>), dim3(grid), dim3(NT), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace msc
