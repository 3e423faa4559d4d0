// Offline-screening kernel (Section 4.2).
//
// A shot's signature over the decided measurements is the XOR of its
// faults' signatures; the shot must be simulated iff that signature is
// zero.  A fault's signature (the XOR of its basis components, X and Z on
// each of the channel's up to three qubits) is precombined per (channel,
// Pauli code) on the host, so each fault costs one lookup in an L2-resident
// table.  A block XORs its shots' lookups in LDS, and the wavefront's verdicts
// are packed with a 64-lane ballot into one uint64 of the survivor bitmap (bit
// j of word w <-> shot 64 w + j).  A second pass turns the bitmap into an
// ascending survivor index list: popcounts per 256 shots, one scan block, and
// a scatter with a per-wave prefix from the ballot mask.  Integer only.
//
// The CSR is checked on the way: a channel index outside [0, M), channels
// not strictly ascending within a shot, a Pauli code that is zero or names
// a qubit the channel does not have, or decreasing offsets set bits of a
// device flag word (CsrFlag), and the host turns a nonzero flag into
// MSC_E_INVALID.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "kernels.h"

namespace msc {
namespace {

// the one-workgroup scans use 256 threads: small enough to find room beside
// resident shot kernels of other streams
constexpr int kScanT = 256;

constexpr int PT = 256;   // threads per block (4 waves, 256 shots)
constexpr int kSup = 256; // blocks per superblock of the survivor scan

// tmp words of a screen of n shots: the per-block survivor counts (their
// scan in place), the superblock totals (their scan in place, plus one),
// the survivor total and the CSR flag word
constexpr int64_t screen_tmp_words(int64_t n) {
    return (n + PT - 1) / PT + ((n + PT - 1) / PT + kSup - 1) / kSup + 1 + 2;
}

// Largest Pauli code + 1 of each channel kind (ChanKind order): one qubit
// (x, z bits), two, the X flip (x of qubit 0 only), three.
__device__ __forceinline__ int code_limit(int kind) {
    return kind == CH_DEP1 ? 4 : kind == CH_DEP2 ? 16 : kind == CH_XERR ? 2 : 64;
}

// Checks of one fault against the previous one of its shot (CsrFlag bits).
__device__ __forceinline__ int fault_check(int64_t c, int64_t prev, int p, int32_t nch,
                                           const uint8_t* __restrict__ kind) {
    if (c < 0 || c >= nch) return CSR_BAD_CHANNEL;
    int bad = c <= prev ? CSR_NOT_ASCENDING : 0;
    if (p == 0 || p >= code_limit(kind[c])) bad |= CSR_BAD_PAULI;
    return bad;
}

// One fault's checks and its signature XORed into acc (W words; CsrFlag bits
// returned).  The channel's first table entry and its kind are one word.
template <int W, typename F>
__device__ __forceinline__ int screen_fault(int64_t c, int64_t prev, int p, int32_t nch,
                                            const uint64_t* __restrict__ sig,
                                            const int32_t* __restrict__ sig_off, F add) {
    if (c < 0 || c >= nch) return CSR_BAD_CHANNEL;
    const int32_t ek = sig_off[c];
    int bad = c <= prev ? CSR_NOT_ASCENDING : 0;
    // an invalid code has no entry (the call fails anyway)
    if (p == 0 || p >= code_limit(ek & 3)) return bad | CSR_BAD_PAULI;
    const uint64_t* s = sig + (static_cast<int64_t>(ek >> 2) + p) * W;
#pragma unroll
    for (int w = 0; w < W; ++w) add(w, s[w]);
    return bad;
}

// One shot by its own lane, fault after fault: its checks (CsrFlag bits into
// bad) and whether its signature is zero.
template <int W>
__device__ bool screen_shot(int64_t f0, int64_t f1, int32_t nch, const int32_t* __restrict__ chan,
                            const uint8_t* __restrict__ pauli, const uint64_t* __restrict__ sig,
                            const int32_t* __restrict__ sig_off, int& bad) {
    uint64_t acc[W];
#pragma unroll
    for (int w = 0; w < W; ++w) acc[w] = 0;
    if (f1 < f0 || f0 < 0) bad |= CSR_BAD_OFFSETS;
    int64_t prev = -1;
    for (int64_t f = f0; f < f1; ++f) {
        const int64_t c = chan[f];
        bad |= screen_fault<W>(c, prev, pauli[f], nch, sig, sig_off,
                               [&](int w, uint64_t x) { acc[w] ^= x; });
        prev = c;
    }
    uint64_t any = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) any |= acc[w];
    return any == 0;
}

// A block screens PT shots.  Their faults are one contiguous run of the CSR
// when the offsets rise: they are dealt to the lanes one by one, kScreenRun at
// a time (the screen is bound by the latency of offset, channel and table
// reads one behind the other, so by how many a wavefront has in flight).  A
// fault reads one word of the table, a linear hash of its signature, XORed into
// its shot's word in LDS: a shot whose hashes do not XOR to zero has a nonzero
// signature, which decides all but the survivors (and, once in 2^63, another).
// The survivors that have faults XOR their whole W-word signatures, fault by
// fault over the lanes, their faults packed (a walk by the shot's lane where
// the list runs out or the faults took several runs).  A whole signature and
// its entry's index are W + 1 gathers of 64 lines each.  Without a hash (tables
// above kMaxHashEntries), and in blocks whose offsets fall or are negative (the
// call fails), every shot is walked.
// 2^24 shots of the 81-qubit circuit, the call: one lane per shot walking its
// faults 571 us, now 345 (five times the fault rate: 2886 and 1186); 2^14
// shots 22 us both.  Four shots per lane take 377 us, and 33 for 2^14 shots.
constexpr int kScreenPer = 4;
constexpr int kScreenRun = PT * kScreenPer;
constexpr int kList = 2 * PT;
template <int W>
__global__ __launch_bounds__(PT) void screen_kernel(int32_t nch, int64_t n,
                                                    const int64_t* __restrict__ off,
                                                    const int32_t* __restrict__ chan,
                                                    const uint8_t* __restrict__ pauli,
                                                    const uint64_t* __restrict__ sig,
                                                    const int32_t* __restrict__ sig_off,
                                                    const uint64_t* __restrict__ hash, int shift,
                                                    uint64_t* __restrict__ bits,
                                                    int64_t* __restrict__ block_cnt,
                                                    int* __restrict__ flag) {
    __shared__ unsigned long long s_hash[PT];
    __shared__ int s_rel[PT + 1];                // offsets from the block's first
    __shared__ uint16_t s_own[kScreenRun];       // the shot of each fault of a run
    __shared__ unsigned long long s_acc[W][PT];
    __shared__ int s_cnt[PT / 64], s_nf;
    __shared__ int32_t s_lc[kList];              // the survivors' faults
    __shared__ uint16_t s_lp[kList];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * PT, i = i0 + tid;
    const int64_t first = off[i0], end = off[i + 1 < n ? i + 1 : n] - first;
    int bad = 0, odd = !hash || first < 0 || end < 0 || end >= (int64_t(1) << 31);
    s_rel[tid + 1] = static_cast<int>(end);
    s_hash[tid] = 0;
    if (tid == 0) {
        s_rel[0] = 0;
        s_nf = 0;
    }
    __syncthreads();
    const int my0 = s_rel[tid], my1 = s_rel[tid + 1];
    odd |= my1 < my0;
    bool alive;
    if (!__syncthreads_or(odd)) {
        const int total = s_rel[PT];
        int32_t c[kScreenPer];
        int p[kScreenPer];
        for (int r0 = 0; r0 < total; r0 += kScreenRun) {
            const int run = min(total - r0, kScreenRun);
#pragma unroll
            for (int u = 0; u < kScreenPer; ++u) {
                const int f = tid + PT * u;
                c[u] = -1;
                p[u] = 0;
                if (f < run) {
                    c[u] = chan[first + r0 + f];
                    p[u] = pauli[first + r0 + f];
                }
            }
            for (int f = max(my0 - r0, 0); f < min(my1 - r0, run); ++f)
                s_own[f] = static_cast<uint16_t>(tid);
            __syncthreads();
            uint64_t h[kScreenPer];
#pragma unroll
            for (int u = 0; u < kScreenPer; ++u) {
                const bool in = c[u] >= 0 && c[u] < nch && !(p[u] >> shift);
                h[u] = hash[in ? (static_cast<int64_t>(c[u]) << shift) + p[u] : 0];
                if (!in) h[u] = kHashInvalid;
            }
#pragma unroll
            for (int u = 0; u < kScreenPer; ++u) {
                const int f = tid + PT * u;
                // the channel before, from the lane below
                int32_t prev = __shfl_up(c[u], 1);
                if (f >= run) continue;
                if (lane == 0 && r0 + f > 0) prev = chan[first + r0 + f - 1];
                const int own = s_own[f];
                if (c[u] < 0 || c[u] >= nch) {
                    bad |= CSR_BAD_CHANNEL;
                    continue;
                }
                if (s_rel[own] < r0 + f && c[u] <= prev) bad |= CSR_NOT_ASCENDING;
                if (h[u] & kHashInvalid) bad |= CSR_BAD_PAULI;
                else if (h[u]) atomicXor(&s_hash[own], h[u]);
            }
            __syncthreads();
        }
#pragma unroll
        for (int w = 0; w < W; ++w) s_acc[w][tid] = 0;
        alive = i < n && s_hash[tid] == 0;
        const bool check = alive && my1 > my0;
        if (total <= kScreenRun) {
            if (__syncthreads_or(check)) {
                // the faults of the shots left, packed: the lanes that read
                // signatures are full
#pragma unroll
                for (int u = 0; u < kScreenPer; ++u) {
                    const int f = tid + PT * u;
                    if (f >= total) continue;
                    const int own = s_own[f];
                    if (s_hash[own] != 0) continue;
                    const int x = atomicAdd(&s_nf, 1);
                    if (x < kList) {
                        s_lc[x] = c[u];
                        s_lp[x] = static_cast<uint16_t>(p[u] | (own << 8));
                    }
                }
                __syncthreads();
                for (int x = tid; x < min(s_nf, kList); x += PT) {
                    const int own = s_lp[x] >> 8;
                    (void)screen_fault<W>(s_lc[x], -1, s_lp[x] & 255, nch, sig, sig_off,   // (checked above)
                                          [&](int w, uint64_t y) { atomicXor(&s_acc[w][own], y); });
                }
                __syncthreads();
            }
        }
        if (check && total <= kScreenRun && s_nf <= kList) {
            uint64_t any = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) any |= s_acc[w][tid];
            alive = any == 0;
        } else if (check) {
            int again = 0;                       // (the checks are done)
            alive = screen_shot<W>(first + my0, first + my1, nch, chan, pauli, sig, sig_off, again);
        }
    } else {
        alive = i < n && screen_shot<W>(off[i], off[i + 1], nch, chan, pauli, sig, sig_off, bad);
    }
    if (bad) atomicOr(flag, bad);
    const uint64_t mask = __ballot(alive);
    const int64_t word = (i0 + (tid & ~63)) >> 6;
    if (lane == 0) {
        if (word * 64 < n) bits[word] = mask;
        s_cnt[tid >> 6] = __popcll(mask);
    }
    __syncthreads();
    if (tid == 0 && block_cnt) {
        int64_t t = 0;
        for (int w = 0; w < PT / 64; ++w) t += s_cnt[w];
        block_cnt[blockIdx.x] = t;
    }
}

// The same checks alone, one shot per lane (for the entry points that
// take a caller's CSR without screening it).
__global__ __launch_bounds__(PT) void validate_kernel(int32_t nch, int64_t n,
                                                      const int64_t* __restrict__ off,
                                                      const int32_t* __restrict__ chan,
                                                      const uint8_t* __restrict__ pauli,
                                                      const uint8_t* __restrict__ kind,
                                                      int* __restrict__ flag) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * PT + threadIdx.x;
    if (i >= n) return;
    const int64_t f0 = off[i], f1 = off[i + 1];
    int bad = (f1 < f0 || f0 < 0) ? CSR_BAD_OFFSETS : 0;
    int64_t prev = -1;
    for (int64_t f = f0; f < f1; ++f) {
        const int64_t c = chan[f];
        bad |= fault_check(c, prev, pauli[f], nch, kind);
        prev = c;
    }
    if (bad) atomicOr(flag, bad);
}

// one word set to zero by a kernel (a fill node, not a memset, if captured)
__global__ void clear_flag_kernel(int* flag) { *flag = 0; }

// exclusive scan of the block counts within each superblock of kSup blocks,
// in place (one workgroup per superblock, coalesced), the superblock's total
// into sup[superblock]
__global__ __launch_bounds__(kSup) void scan_local_kernel(int64_t* cnt, int64_t nb,
                                                          int64_t* sup) {
    __shared__ int64_t s[kSup];
    const int t = threadIdx.x;
    const int64_t j = static_cast<int64_t>(blockIdx.x) * kSup + t;
    const int64_t v = j < nb ? cnt[j] : 0;
    s[t] = v;
    __syncthreads();
    // inclusive scan in LDS, log2(kSup) steps
    for (int d = 1; d < kSup; d <<= 1) {
        const int64_t a = t >= d ? s[t - d] : 0;
        __syncthreads();
        s[t] += a;
        __syncthreads();
    }
    if (j < nb) cnt[j] = s[t] - v;
    if (t == kSup - 1) sup[blockIdx.x] = s[t];
}

// exclusive scan of the superblock totals in place (one block), the total
// at *total
__global__ __launch_bounds__(kScanT) void scan_kernel(int64_t* cnt, int64_t nb, int64_t* total) {
    __shared__ int64_t part[kScanT];
    const int tid = threadIdx.x;
    const int64_t per = (nb + kScanT - 1) / kScanT;
    const int64_t lo = tid * per, hi = (lo + per < nb) ? lo + per : nb;
    int64_t s = 0;
    for (int64_t j = lo; j < hi; ++j) s += cnt[j];
    part[tid] = s;
    __syncthreads();
    if (tid == 0) {
        int64_t run = 0;
        for (int j = 0; j < kScanT; ++j) {
            int64_t v = part[j];
            part[j] = run;
            run += v;
        }
        *total = run;
    }
    __syncthreads();
    int64_t run = part[tid];
    for (int64_t j = lo; j < hi; ++j) {
        int64_t v = cnt[j];
        cnt[j] = run;
        run += v;
    }
}

__global__ __launch_bounds__(PT) void scatter_kernel(int64_t n, const uint64_t* __restrict__ bits,
                                                     const int64_t* __restrict__ block_off,
                                                     const int64_t* __restrict__ sup_off,
                                                     int64_t* __restrict__ idx) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * PT + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t word = (static_cast<int64_t>(blockIdx.x) * PT + (threadIdx.x & ~63)) >> 6;
    const uint64_t mask = (word * 64 < n) ? bits[word] : 0ull;
    __shared__ int s_pre[PT / 64];
    if (lane == 0) s_pre[wv] = __popcll(mask);
    __syncthreads();
    int64_t base = sup_off[blockIdx.x / kSup] + block_off[blockIdx.x];
    for (int w = 0; w < wv; ++w) base += s_pre[w];
    if (i < n && ((mask >> lane) & 1)) {
        const uint64_t below = lane ? (mask & ((1ull << lane) - 1)) : 0ull;
        idx[base + __popcll(below)] = i;
    }
}

}  // namespace

int64_t prescreen_tmp_words(int64_t n) { return screen_tmp_words(n); }

hipError_t launch_prescreen(int words, int32_t n_channels, int64_t n, const int64_t* off, const int32_t* chan,
                            const uint8_t* pauli, const uint64_t* sig, const int32_t* sig_off,
                            const uint64_t* hash, int hash_shift, uint64_t* bits,
                            int64_t* survivor_idx, int64_t* block_tmp, int64_t n_blocks_tmp,
                            int* flag, hipStream_t s) {
    const int64_t nb = (n + PT - 1) / PT;
    if (nb == 0) return hipSuccess;
    const int64_t ns = (nb + kSup - 1) / kSup;
    if (n_blocks_tmp < screen_tmp_words(n) || !flag) return hipErrorInvalidValue;
    int64_t* sup = block_tmp + nb;                    // ns + 1 words
    int64_t* total = block_tmp + n_blocks_tmp - 2;    // then the flag word
    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, s, flag);
    hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
    dim3 grid(static_cast<unsigned>(nb));
    switch (words) {
#define MSC_SCREEN_CASE(WW)                                                                   \
    case WW:                                                                                  \
        hipLaunchKernelGGL(screen_kernel<WW>, grid, dim3(PT), 0, s, n_channels, n, off, chan, \
                           pauli, sig, sig_off, hash, hash_shift, bits, block_tmp, flag);     \
        break;
        MSC_SCREEN_CASE(1)
        MSC_SCREEN_CASE(2)
        MSC_SCREEN_CASE(3)
        MSC_SCREEN_CASE(4)
        MSC_SCREEN_CASE(5)
        MSC_SCREEN_CASE(6)
        MSC_SCREEN_CASE(7)
        MSC_SCREEN_CASE(8)
#undef MSC_SCREEN_CASE
        default:
            return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(scan_local_kernel, dim3(static_cast<unsigned>(ns)), dim3(kSup), 0, s,
                       block_tmp, nb, sup);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(kScanT), 0, s, sup, ns, total);
    e = hipGetLastError();
    if (e != hipSuccess || !survivor_idx) return e;
    hipLaunchKernelGGL(scatter_kernel, grid, dim3(PT), 0, s, n, bits, block_tmp, sup,
                       survivor_idx);
    return hipGetLastError();
}

hipError_t launch_validate_csr(int32_t n_channels, int64_t n, const int64_t* off,
                               const int32_t* chan, const uint8_t* pauli, const uint8_t* kind,
                               int* flag, hipStream_t s) {
    if (!flag) return hipErrorInvalidValue;
    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, s, flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n <= 0) return e;
    const dim3 grid(static_cast<unsigned>((n + PT - 1) / PT));
    hipLaunchKernelGGL(validate_kernel, grid, dim3(PT), 0, s, n_channels, n, off, chan, pauli,
                       kind, flag);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fixed scratch of msc_prescreen_noalloc: the block counts and their scan
// (one word per 256 shots), the superblock totals, the survivor total and
// the CSR flag, for at most kNoAllocShots shots.  Each device holds its own copy until the process
// ends.  Host code never passes `scratch` itself to a kernel (on the host it
// is only a stand-in symbol): the device address is resolved once per device
// with hipGetSymbolAddress and that pointer is used everywhere.
namespace {
constexpr int64_t kNoAllocWords = screen_tmp_words(kNoAllocShots);
constexpr int kMaxDevices = 64;
}  // namespace

static __device__ __align__(256) int64_t scratch[kNoAllocWords];

static std::mutex g_scratch_mu;
static int64_t* g_scratch_ptr[kMaxDevices] = {};

hipError_t prescreen_noalloc_scratch(int device, int64_t** out) {
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = static_cast<int64_t*>(p);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

}  // namespace msc
