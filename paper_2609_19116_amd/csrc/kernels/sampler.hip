// Subset-sampling fault draws on the device (Section 4.1), one shot per
// lane.
//
// The draws are the same pure function of (seed, shot index) as the host
// sampler: SplitMix64 (Steele, Lea, Flood 2014) seeded with
// mix(seed ^ mix(shot)); a weight w either given per shot or found by
// inverting the FP64 cumulative Bin(M, p) table against u = (x >> 11) 2^-53;
// Floyd's uniform w-subset of the M channels with Lemire's bounded integers;
// the subset in ascending order; one uniform non-identity Pauli per chosen
// channel (3, 15 or 63 choices for a one-, two- or three-qubit depolarising
// channel, X for an X flip).  Only integer and IEEE basic operations are
// used, so every bit of the CSR matches the host's.
//
// Three steps: (1) every lane draws its shot's weight, the block's total goes
// out; (2) a scan of the block totals; (3) the block's offsets, channels and
// Paulis (draw_kernel), written only where a shot's slice ends within the
// caller's capacity, so an undersized output is never written past its end.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.h"

namespace msc {
namespace {

// the one-workgroup scans use 256 threads: small enough to find room beside
// resident shot kernels of other streams
constexpr int kScanT = 256;

constexpr int ST = 256;   // shots per block
constexpr int kSup = 256; // blocks per superblock of the offset scan
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

struct DevRng {
    uint64_t s;
    __device__ DevRng(uint64_t seed, uint64_t shot) : s(mix64(seed ^ mix64(shot))) {}
    __device__ uint64_t next() {
        s += kGolden;
        return mix64(s);
    }
    // uniform integer in [0, n): Lemire's multiply-and-reject
    __device__ uint64_t bounded(uint64_t n) {
        uint64_t x = next();
        uint64_t lo = x * n;
        uint64_t hi = __umul64hi(x, n);
        if (lo < n) {
            const uint64_t t = (0ull - n) % n;
            while (lo < t) {
                x = next();
                lo = x * n;
                hi = __umul64hi(x, n);
            }
        }
        return hi;
    }
    __device__ double uniform01() {
        return static_cast<double>(next() >> 11) * (1.0 / 9007199254740992.0);
    }
};

constexpr int kCdfLds = 64;    // entries of the cumulative table held in LDS

// weight of one shot; advances rng exactly as the host does.  cdf_lds holds
// the table's first min(n_cdf, kCdfLds) entries.
__device__ __forceinline__ int64_t draw_weight(DevRng& rng, int64_t i, const int32_t* weights,
                                               const double* cdf, const double* cdf_lds,
                                               int32_t n_cdf, int64_t M) {
    int64_t w;
    if (weights) {
        w = weights[i];
        if (w < 0) w = 0;
    } else {
        const double u = rng.uniform01();
        w = n_cdf - 1;
        for (int32_t k = 0; k < n_cdf; ++k) {
            if (u < (k < kCdfLds ? cdf_lds[k] : cdf[k])) {
                w = k;
                break;
            }
        }
    }
    return w < M ? w : M;
}

__device__ __forceinline__ void load_cdf(const int32_t* weights, const double* cdf, int32_t n_cdf,
                                         double* cdf_lds) {
    if (!weights)
        for (int k = threadIdx.x; k < kCdfLds && k < n_cdf; k += ST) cdf_lds[k] = cdf[k];
    __syncthreads();
}

// Inclusive scan of v over the block, and the block's total.
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t* s_wave, int64_t& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t u = __shfl_up(v, d);
        if (lane >= d) v += u;
    }
    if (lane == 63) s_wave[w] = v;
    __syncthreads();
    total = 0;
    for (int q = 0; q < ST / 64; ++q) {
        if (q < w) v += s_wave[q];
        total += s_wave[q];
    }
    return v;
}

__global__ __launch_bounds__(ST) void weight_kernel(int64_t n, uint64_t seed, uint64_t first,
                                                    const int32_t* __restrict__ weights,
                                                    const double* __restrict__ cdf, int32_t n_cdf,
                                                    int64_t M, int64_t* __restrict__ block_tot) {
    __shared__ int64_t s_wave[ST / 64];
    __shared__ double s_cdf[kCdfLds];
    const int64_t i = static_cast<int64_t>(blockIdx.x) * ST + threadIdx.x;
    load_cdf(weights, cdf, n_cdf, s_cdf);
    int64_t w = 0, total;
    if (i < n) {
        DevRng rng(seed, first + static_cast<uint64_t>(i));
        w = draw_weight(rng, i, weights, cdf, s_cdf, n_cdf, M);
    }
    block_scan(w, s_wave, total);
    if (threadIdx.x == 0) block_tot[blockIdx.x] = total;
}

// exclusive scan of the block totals within each superblock of kSup blocks,
// in place (one workgroup per superblock, coalesced), the superblock's
// total into sup[superblock]
__global__ __launch_bounds__(kSup) void local_scan_kernel(int64_t* cnt, int64_t nb,
                                                          int64_t* sup) {
    __shared__ int64_t sh[kSup];
    const int t = threadIdx.x;
    const int64_t j = static_cast<int64_t>(blockIdx.x) * kSup + t;
    const int64_t v = j < nb ? cnt[j] : 0;
    sh[t] = v;
    __syncthreads();
    for (int d = 1; d < kSup; d <<= 1) {
        const int64_t a = t >= d ? sh[t - d] : 0;
        __syncthreads();
        sh[t] += a;
        __syncthreads();
    }
    if (j < nb) cnt[j] = sh[t] - v;
    if (t == kSup - 1) sup[blockIdx.x] = sh[t];
}

// exclusive scan of the superblock totals in place (one block), grand total
// at [nb]
__global__ __launch_bounds__(kScanT) void total_scan_kernel(int64_t* cnt, int64_t nb) {
    __shared__ int64_t part[kScanT];
    const int tid = threadIdx.x;
    const int64_t per = (nb + kScanT - 1) / kScanT;
    const int64_t lo = tid * per, hi = (lo + per < nb) ? lo + per : nb;
    int64_t acc = 0;
    for (int64_t j = lo; j < hi; ++j) acc += cnt[j];
    part[tid] = acc;
    __syncthreads();
    for (int d = 1; d < kScanT; d <<= 1) {
        const int64_t v = tid >= d ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int64_t run = tid ? part[tid - 1] : 0;
    if (tid == kScanT - 1) cnt[nb] = part[kScanT - 1];
    for (int64_t j = lo; j < hi; ++j) {
        const int64_t v = cnt[j];
        cnt[j] = run;
        run += v;
    }
}

// One shot's channels (ascending) and Paulis at c and pa by its own lane, in
// the host's order of draws.
template <typename CP, typename PP>
__device__ void draw_shot(DevRng rng, int64_t w, int64_t M, const uint8_t* __restrict__ kind, CP c,
                          PP pa) {
    // Floyd: for j in [M-w, M) take t uniform in [0, j], or j if t is taken
    int64_t k = 0;
    for (int64_t j = M - w; j < M; ++j) {
        const int32_t t = static_cast<int32_t>(rng.bounded(static_cast<uint64_t>(j + 1)));
        bool have = false;
        for (int64_t q = 0; q < k; ++q) have |= c[q] == t;
        c[k++] = have ? static_cast<int32_t>(j) : t;
    }
    // ascending order (insertion sort)
    for (int64_t a = 1; a < w; ++a) {
        const int32_t v = c[a];
        int64_t b = a - 1;
        while (b >= 0 && c[b] > v) {
            c[b + 1] = c[b];
            --b;
        }
        c[b + 1] = v;
    }
    for (int64_t a = 0; a < w; ++a) {
        const int kd = kind[c[a]];
        uint8_t code;
        if (kd == CH_XERR) code = 1;
        else if (kd == CH_DEP1) code = static_cast<uint8_t>(1 + rng.bounded(3));
        else if (kd == CH_DEP2) code = static_cast<uint8_t>(1 + rng.bounded(15));
        else code = static_cast<uint8_t>(1 + rng.bounded(63));
        pa[a] = code;
    }
}

// The 64 x 32-bit product x n as (high 32 of the 96 bits, low 64).
__device__ __forceinline__ uint32_t mul96(uint64_t x, uint32_t n, uint64_t& lo) {
    const uint64_t p0 = static_cast<uint64_t>(static_cast<uint32_t>(x)) * n;
    const uint64_t p1 = static_cast<uint64_t>(static_cast<uint32_t>(x >> 32)) * n + (p0 >> 32);
    lo = (p1 << 32) | static_cast<uint32_t>(p0);
    return static_cast<uint32_t>(p1 >> 32);
}

// Offsets, channels and Paulis of the block's shots.  The generator is
// counter-based, so draw k of a shot is mix64(s0 + k golden) for any k, and
// the block's faults, dealt to the lanes one by one, take their draws
// independently: a wavefront no longer waits for its heaviest shot (of 64
// shots with 2.9 faults on average the worst has 8).  A fault's rank among
// its shot's raw channels is its place; the Paulis' draws follow in that
// order (an X flip takes none).  A shot whose raw channels repeat (Floyd's
// replacement) or one of whose draws Lemire's test would look at more closely
// (probability n 2^-64) is drawn again by its own lane in the host's order.
// The results leave through LDS in one contiguous run per block.  Blocks with
// more than kDrawCap faults draw shot by shot, straight to memory.
// 2^24 shots of the 81-qubit circuit (48 M faults), all three steps: one lane
// per shot with its channels in memory 0.89 ms (420 GB/s of output), now 0.52.
constexpr int kDrawCap = 1536;
constexpr int kKindShift = 28;     // the channel's kind above its index
__global__ __launch_bounds__(ST) void draw_kernel(int64_t n, uint64_t seed, uint64_t first,
                                                  const int32_t* __restrict__ weights,
                                                  const double* __restrict__ cdf, int32_t n_cdf,
                                                  int64_t M, const uint8_t* __restrict__ kind,
                                                  const int64_t* __restrict__ block_base,
                                                  const int64_t* __restrict__ sup_base,
                                                  int64_t nnz_cap, int64_t* __restrict__ shot_off,
                                                  int32_t* __restrict__ chan,
                                                  uint8_t* __restrict__ pauli) {
    __shared__ int64_t s_wave[ST / 64];
    __shared__ double s_cdf[kCdfLds];
    __shared__ uint64_t s_s0[ST];
    __shared__ int s_ofs[ST + 1];
    __shared__ uint8_t s_own[kDrawCap], s_pa[kDrawCap], s_redo[ST];
    __shared__ int32_t s_raw[kDrawCap], s_ch[kDrawCap];
    const int tid = threadIdx.x;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * ST + tid;
    load_cdf(weights, cdf, n_cdf, s_cdf);
    DevRng rng(seed, first + static_cast<uint64_t>(i));
    const uint64_t s0 = rng.s;
    const int64_t w = i < n ? draw_weight(rng, i, weights, cdf, s_cdf, n_cdf, M) : 0;
    int64_t total;
    const int64_t incl = block_scan(w, s_wave, total);
    const int64_t base = block_base[blockIdx.x] + sup_base[blockIdx.x / kSup];
    if (i == 0) shot_off[0] = 0;
    if (i < n) shot_off[i + 1] = base + incl;
    if (total > kDrawCap || M >= (int64_t(1) << kKindShift)) {
        if (w > 0 && base + incl <= nnz_cap)
            draw_shot(rng, w, M, kind, chan + base + incl - w, pauli + base + incl - w);
        return;
    }
    const int F = static_cast<int>(total), o0 = static_cast<int>(incl - w);
    s_s0[tid] = s0;
    s_ofs[tid + 1] = static_cast<int>(incl);
    if (tid == 0) s_ofs[0] = 0;
    s_redo[tid] = 0;
    for (int q = 0; q < static_cast<int>(w); ++q) s_own[o0 + q] = static_cast<uint8_t>(tid);
    __syncthreads();
    const uint32_t k0 = weights ? 0 : 1;       // draws taken by the weight
    for (int f = tid; f < F; f += ST) {
        const int own = s_own[f], b0 = s_ofs[own], wi = s_ofs[own + 1] - b0, j = f - b0;
        const uint32_t nn = static_cast<uint32_t>(M) - wi + j + 1;
        uint64_t lo;
        const uint32_t t = mul96(mix64(s_s0[own] + (k0 + j + 1) * kGolden), nn, lo);
        if (lo < nn) s_redo[own] = 1;
        s_raw[f] = static_cast<int32_t>(t | (static_cast<uint32_t>(kind[t]) << kKindShift));
    }
    __syncthreads();
    constexpr int32_t kMask = (1 << kKindShift) - 1;
    for (int f = tid; f < F; f += ST) {
        const int own = s_own[f], b0 = s_ofs[own], b1 = s_ofs[own + 1];
        const int32_t raw = s_raw[f], t = raw & kMask;
        int rank = 0, drawn = 0;               // smaller channels, those that take a draw
        bool dup = false;
        for (int q = b0; q < b1; ++q) {
            const int32_t r = s_raw[q];
            const bool less = (r & kMask) < t;
            rank += less;
            drawn += less && (r >> kKindShift) != CH_XERR;
            dup |= q != f && (r & kMask) == t;
        }
        if (dup) {
            s_redo[own] = 1;
            continue;
        }
        const int kd = raw >> kKindShift;
        int code = 1;
        if (kd != CH_XERR) {
            const uint32_t nn = kd == CH_DEP1 ? 3 : kd == CH_DEP2 ? 15 : 63;
            uint64_t lo;
            code += mul96(mix64(s_s0[own] + (k0 + (b1 - b0) + drawn + 1) * kGolden), nn, lo);
            if (lo < nn) s_redo[own] = 1;
        }
        s_ch[b0 + rank] = t;
        s_pa[b0 + rank] = static_cast<uint8_t>(code);
    }
    __syncthreads();
    if (s_redo[tid]) draw_shot(rng, w, M, kind, s_ch + o0, s_pa + o0);
    __syncthreads();
    const bool fits = base + total <= nnz_cap;
    for (int f = tid; f < F; f += ST) {
        if (!fits && base + s_ofs[s_own[f] + 1] > nnz_cap) continue;
        chan[base + f] = s_ch[f];
        pauli[base + f] = s_pa[f];
    }
}

}  // namespace

// the block totals, the superblock totals, the grand total
int64_t sampler_tmp_words(int64_t n) {
    const int64_t nb = (n + ST - 1) / ST;
    return nb + (nb + kSup - 1) / kSup + 1;
}

hipError_t launch_sampler(int64_t n, uint64_t seed, uint64_t first, const int32_t* weights,
                          const double* cdf, int32_t n_cdf, int64_t M, const uint8_t* kind,
                          int64_t nnz_cap, int64_t* shot_off, int32_t* chan, uint8_t* pauli,
                          int64_t* tmp, int64_t n_tmp, hipStream_t s) {
    const int64_t nb = (n + ST - 1) / ST;
    if (nb == 0) return hipSuccess;
    const int64_t ns = (nb + kSup - 1) / kSup;
    if (n_tmp < nb + ns + 1 || nb > 0x7fffffff) return hipErrorInvalidValue;
    int64_t* sup = tmp + nb;
    if (!weights && (!cdf || n_cdf < 1)) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(nb));
    hipLaunchKernelGGL(weight_kernel, grid, dim3(ST), 0, s, n, seed, first, weights, cdf, n_cdf, M,
                       tmp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(local_scan_kernel, dim3(static_cast<unsigned>(ns)), dim3(kSup), 0, s, tmp,
                       nb, sup);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(total_scan_kernel, dim3(1), dim3(kScanT), 0, s, sup, ns);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(draw_kernel, grid, dim3(ST), 0, s, n, seed, first, weights, cdf, n_cdf, M,
                       kind, tmp, sup, nnz_cap, shot_off, chan, pauli);
    return hipGetLastError();
}

}  // namespace msc
