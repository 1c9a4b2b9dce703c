// ara_select.hip -- PML and TVaR from a Year Loss Table (section 2.3).
//
// PML(RP) is the k-th largest trial loss, k = max(1, floor(N / RP)); it is
// found by a most-significant-digit radix select over the bit patterns of the
// losses (non-negative IEEE floats order like their unsigned bit patterns;
// -0.0 is folded onto +0.0): 11-bit digits, a histogram pass per digit whose
// blocks first pick the digit before.  TVaR(RP) is the mean of the k largest
// losses: the sum of the losses strictly above the PML plus (k - their count)
// copies of the PML, accumulated in FP64 with a fixed reduction order
// (deterministic).
//
// The exceedance-probability curve (the return-period losses of the report
// the paper names) is the whole YLT in descending order: a stable
// least-significant-digit radix sort over the inverted key patterns (8-bit
// digits; per pass a block histogram, a scan per digit of its counts, and a
// scatter that ranks equal digits by wavefront ballots), followed by FP64
// running means of the sorted losses (the TVaR at every point).
//
// A YLT of up to 1M trials is a few megabytes: what these take is launches and
// the latency inside one, not bandwidth.  So there are as few passes as digits
// allow, and a YLT that one block holds takes one launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_device.h"
#include "ara_kernels.h"

namespace ara {

template <typename T>
struct KeyOf;
template <>
struct KeyOf<float> {
    using K = uint32_t;
    static constexpr int bits = 32;
    __device__ static K key(float v) {
        const uint32_t b = __float_as_uint(v);
        return b == 0x80000000u ? 0u : b;
    }
    __device__ static double value(uint64_t k) { return (double)__uint_as_float((uint32_t)k); }
};
template <>
struct KeyOf<double> {
    using K = uint64_t;
    static constexpr int bits = 64;
    __device__ static K key(double v) {
        const uint64_t b = (uint64_t)__double_as_longlong(v);
        return b == 0x8000000000000000ull ? 0ull : b;
    }
    __device__ static double value(uint64_t k) { return __longlong_as_double((long long)k); }
};

// Return periods are selected together, up to kSelGroup per pass over the YLT:
// periods whose selections still share their prefix share one histogram, so a
// group costs the same launches whatever its size.  Pass p's kernel starts with
// the picks of pass p - 1 (every block the same, a wavefront per period, 8 KB of
// counts each), which took launches of their own; launch boundaries order the
// passes (a last-block-done handshake would need a device-wide fence in every
// block, which costs more here).
constexpr int kSelGroup = 16;
constexpr int kSelBits = 11;
constexpr int kSelBins = 1 << kSelBits;
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelMaxPasses = (64 + kSelBits - 1) / kSelBits;
// Most blocks of a pass (a block flushes its histograms with device atomics, so
// few blocks of many losses each), and the losses that make another one worth it.  A
// pass over 1M FP32 losses and 9 periods takes 11 us, 10 of them the picks and one
// block's latency; 8-bit digits took 20 us and 8 us for the picks.
constexpr int kSelBlocks = 256;
constexpr int kSelLosses = 8192;

// A period's selection: the digits of the PML's key found so far, and the rank left
// among the keys that share them.
struct SelState {
    uint64_t prefix;
    int64_t krem;
};

struct SelGroup {
    int64_t k[kSelGroup];
};

// Scratch of one group.  Pass p counts in buffer p % 3, reads that of pass p - 1 and
// clears that of pass p + 1.
struct SelScratch {
    uint32_t *hist;                 // [3][kSelGroup][kSelBins]
    SelState *st;                   // [kSelMaxPasses + 1][kSelGroup]
    double *psum;                   // [kSelGroup][kSelBlocks]
};

__host__ __device__ constexpr int sel_passes(int bits) { return (bits + kSelBits - 1) / kSelBits; }
// lowest bit of digit p, of keys of bits bits
__host__ __device__ constexpr int sel_shift(int bits, int p) {
    return bits > kSelBits * (p + 1) ? bits - kSelBits * (p + 1) : 0;
}

// A group's selections in LDS.
struct SelLds {
    SelState st[kSelGroup];
    uint64_t pre[kSelGroup];        // the distinct prefixes
    int slot[kSelGroup];            // of each period: its prefix among them
    int n;                          // how many
};

// Distinct prefixes of the m periods, in order of their first period.
__device__ __forceinline__ void sel_slots(SelLds &S, int m) {
    __syncthreads();
    if (threadIdx.x < 64) {
        const int r = threadIdx.x;
        int first = r;
        if (r < m) {
            const uint64_t mine = S.st[r].prefix;
#pragma unroll
            for (int q = kSelGroup - 1; q >= 0; --q)
                if (S.st[q].prefix == mine && q < first) first = q;
        }
        const uint64_t heads = __ballot(r < m && first == r);
        if (r < m) {
            S.slot[r] = __popcll(heads & ((1ull << first) - 1ull));
            if (first == r) S.pre[S.slot[r]] = S.st[r].prefix;
        }
        if (r == 0) S.n = __popcll(heads);
    }
    __syncthreads();
}

// Inclusive sum over the lanes up to this one, laid out as wave_excl_scan.
__device__ __forceinline__ double wave_incl(double v) {
    v += dpp_f64<0x111, 0xf, true>(v);    // row_shr:1
    v += dpp_f64<0x112, 0xf, true>(v);    // row_shr:2
    v += dpp_f64<0x114, 0xf, true>(v);    // row_shr:4
    v += dpp_f64<0x118, 0xf, true>(v);    // row_shr:8
    v += dpp_f64<0x142, 0xa, false>(v);   // row_bcast:15
    v += dpp_f64<0x143, 0xc, false>(v);   // row_bcast:31
    return v;
}

// One wavefront: the digit that holds the krem-th largest key, from the counts of the
// digits; krem becomes its rank within the digit.  A lane adds up 32 bins, the top
// ones in lane 0, and the bins of the lane where the rank is reached are walked by 32
// lanes.  (Counts are whole numbers below 2^53: FP64 sums of them are exact, and
// their scan is DPP moves instead of the LDS permutes of a 64-bit integer one.)
template <bool LDS>
__device__ __forceinline__ uint32_t sel_digit(const uint32_t *h, int64_t *krem, int lane) {
    constexpr int kPer = kSelBins / 64;
    const uint32_t *mine = h + kSelBins - kPer * (lane + 1);
    uint64_t sum = 0;
    if (LDS) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) sum += mine[(j + lane) & (kPer - 1)];    // a bank each
    } else {
        uint4 v[kPer / 4];
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j) v[j] = reinterpret_cast<const uint4 *>(mine)[j];
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j)
            sum += (uint64_t)v[j].x + (uint64_t)v[j].y + (uint64_t)v[j].z + (uint64_t)v[j].w;
    }
    const double k = (double)*krem, s = (double)sum, upto = wave_incl(s);
    const int own = __builtin_ctzll(__ballot(upto >= k) | (1ull << 63));
    const double above = readlane_f64(upto - s, own);
    const int first = kSelBins - 1 - kPer * own;
    const double c = lane < kPer ? (double)h[first - lane] : 0.0;
    const double in = above + wave_incl(c);
    const int at = __builtin_ctzll(__ballot(in >= k) | (1ull << (kPer - 1)));
    *krem -= (int64_t)readlane_f64(in - c, at);
    return (uint32_t)(first - at);
}

// The selections before pass p: the picks of pass p - 1 from the counts it left.
__device__ __forceinline__ void sel_begin(const SelScratch &sc, const SelGroup &g, int m, int bits,
                                          int p, SelLds &S) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (p == 0) {
        if ((int)threadIdx.x < m) S.st[threadIdx.x] = {0, g.k[threadIdx.x]};
    } else {
        if ((int)threadIdx.x < m) S.st[threadIdx.x] = sc.st[(p - 1) * kSelGroup + threadIdx.x];
        sel_slots(S, m);
        const uint32_t *buf = sc.hist + (size_t)((p - 1) % 3) * kSelGroup * kSelBins;
        const int width = (p > 1 ? sel_shift(bits, p - 2) : bits) - sel_shift(bits, p - 1);
        if (w < m) {
            SelState s = S.st[w];
            const uint32_t *h = buf + S.slot[w] * kSelBins;
            const uint32_t d = sel_digit<false>(h, &s.krem, lane);
            s.prefix = (s.prefix << width) | d;
            if (lane == 0) S.st[w] = s;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && (int)threadIdx.x < m) sc.st[p * kSelGroup + threadIdx.x] = S.st[threadIdx.x];
}

// Digit p of losses [i0, n) in steps of step, counted in h by distinct prefix.
template <typename T>
__device__ __forceinline__ void sel_count(const T *__restrict__ y, int64_t i0, int64_t step, int64_t n,
                                          int p, const SelLds &S, uint32_t *h) {
    using K = typename KeyOf<T>::K;
    const int shift = sel_shift(KeyOf<T>::bits, p);
    const uint32_t mask = (1u << ((p ? sel_shift(KeyOf<T>::bits, p - 1) : KeyOf<T>::bits) - shift)) - 1u;
    const int nd = __builtin_amdgcn_readfirstlane(S.n);
    K pre[kSelGroup];
#pragma unroll
    for (int q = 0; q < kSelGroup; ++q) pre[q] = q < nd ? (K)S.pre[q] : (K)0;
    for (int i = threadIdx.x; i < nd * kSelBins; i += kSelThreads) h[i] = 0u;
    __syncthreads();
    for (int64_t i = i0; i < n; i += step) {
        const K k = KeyOf<T>::key(y[i]);
        const uint32_t d = (uint32_t)(k >> shift) & mask;
        if (p == 0) {
            atomicAdd(&h[d], 1u);
            continue;
        }
        const K up = k >> sel_shift(KeyOf<T>::bits, p - 1);
        int q = -1;
#pragma unroll
        for (int u = 0; u < kSelGroup; ++u)
            if (u < nd && up == pre[u]) q = u;
        if (q >= 0) atomicAdd(&h[q * kSelBins + (int)d], 1u);
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void k_sel_init(SelScratch sc) {
    sc.hist[blockIdx.x * 256 + threadIdx.x] = 0u;
}

template <typename T>
__global__ __launch_bounds__(kSelThreads) void k_sel_hist(const T *__restrict__ y, int64_t n,
                                                          SelScratch sc, SelGroup g, int m, int p) {
    __shared__ uint32_t h[kSelGroup * kSelBins];
    __shared__ SelLds S;
    const int64_t i0 = (int64_t)blockIdx.x * kSelThreads + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * kSelThreads;
    uint32_t *next = sc.hist + (size_t)((p + 1) % 3) * kSelGroup * kSelBins;
    for (int64_t i = i0; i < m * kSelBins; i += step) next[i] = 0u;
    sel_begin(sc, g, m, KeyOf<T>::bits, p, S);
    sel_slots(S, m);
    sel_count(y, i0, step, n, p, S, h);
    uint32_t *buf = sc.hist + (size_t)(p % 3) * kSelGroup * kSelBins;
    for (int i = threadIdx.x; i < S.n * kSelBins; i += kSelThreads)
        if (h[i]) atomicAdd(&buf[i], h[i]);
}

// The losses strictly above each period's PML, added in FP64 by this block (a fixed
// tree): sum r in the lanes of wavefront r.
template <typename T>
__device__ __forceinline__ double sel_sum(const T *__restrict__ y, int64_t i0, int64_t step, int64_t n,
                                          int m, const SelLds &S, double (*part)[kSelWaves]) {
    using K = typename KeyOf<T>::K;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    K thr[kSelGroup];
    double acc[kSelGroup];
#pragma unroll
    for (int r = 0; r < kSelGroup; ++r) {
        thr[r] = r < m ? (K)S.st[r].prefix : (K)0;
        acc[r] = 0.0;
    }
    for (int64_t i = i0; i < n; i += step) {
        const T v = y[i];
        const K k = KeyOf<T>::key(v);
#pragma unroll
        for (int r = 0; r < kSelGroup; ++r)
            if (r < m) acc[r] += k > thr[r] ? (double)v : 0.0;
    }
#pragma unroll
    for (int r = 0; r < kSelGroup; ++r) {
        if (r >= m) break;
        const double s = wave_incl(acc[r]);
        if (lane == 63) part[r][w] = s;
    }
    __syncthreads();
    return w < m ? readlane_f64(wave_incl(lane < kSelWaves ? part[w][lane] : 0.0), 63) : 0.0;
}

template <typename T>
__global__ __launch_bounds__(kSelThreads) void k_sel_sum(const T *__restrict__ y, int64_t n,
                                                         SelScratch sc, SelGroup g, int m) {
    __shared__ SelLds S;
    __shared__ double part[kSelGroup][kSelWaves];
    sel_begin(sc, g, m, KeyOf<T>::bits, sel_passes(KeyOf<T>::bits), S);
    const double s = sel_sum(y, (int64_t)blockIdx.x * kSelThreads + threadIdx.x,
                             (int64_t)gridDim.x * kSelThreads, n, m, S, part);
    const int w = threadIdx.x >> 6;
    if (w < m && (threadIdx.x & 63) == 0) sc.psum[w * kSelBlocks + blockIdx.x] = s;
}

// PML and TVaR of a period, from its selection (s.krem of its k largest losses are
// the PML itself) and the sum of the losses above.
template <typename T>
__device__ __forceinline__ void sel_write(const SelState &s, int64_t k, double sum, double *out, int at,
                                          int n_rp) {
    const double pml = KeyOf<T>::value(s.prefix);
    out[at] = pml;
    out[n_rp + at] = (sum + (double)s.krem * pml) / (double)k;
}

// A wavefront per period adds the nb blocks' sums.
template <typename T>
__global__ __launch_bounds__(64) void k_sel_finish(SelScratch sc, SelGroup g, int nb,
                                                   double *__restrict__ out, int r0, int n_rp) {
    const int r = blockIdx.x;
    double t = 0.0;
    for (int b = threadIdx.x; b < nb; b += 64) t += sc.psum[r * kSelBlocks + b];
    t = wave_incl(t);
    if (threadIdx.x == 63)
        sel_write<T>(sc.st[sel_passes(KeyOf<T>::bits) * kSelGroup + r], g.k[r], t, out, r0 + r, n_rp);
}

// All of it by one block, for a YLT of at most kSelSmall losses: 5,000 FP32 losses and 9
// periods 50 us with the copy of the results (178 us with 22 launches); at 16,384 one
// block takes 71 us (FP64 102) and six to nine launches 77 us (122), at 32,768 one
// block 103 us (156).
constexpr int64_t kSelSmall = 16384;

template <typename T>
__global__ __launch_bounds__(kSelThreads) void k_sel_small(const T *__restrict__ y, int64_t n,
                                                           SelGroup g, int m, double *__restrict__ out,
                                                           int r0, int n_rp) {
    __shared__ uint32_t h[kSelGroup * kSelBins];
    __shared__ SelLds S;
    __shared__ double part[kSelGroup][kSelWaves];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if ((int)threadIdx.x < m) S.st[threadIdx.x] = {0, g.k[threadIdx.x]};
    for (int p = 0; p < sel_passes(KeyOf<T>::bits); ++p) {
        sel_slots(S, m);
        sel_count(y, threadIdx.x, kSelThreads, n, p, S, h);
        if (w < m) {
            SelState s = S.st[w];
            const uint32_t *hw = h + S.slot[w] * kSelBins;
            const uint32_t d = sel_digit<true>(hw, &s.krem, lane);
            s.prefix = (s.prefix << ((p ? sel_shift(KeyOf<T>::bits, p - 1) : KeyOf<T>::bits) -
                                     sel_shift(KeyOf<T>::bits, p))) | d;
            if (lane == 0) S.st[w] = s;
        }
    }
    __syncthreads();
    const double s = sel_sum(y, threadIdx.x, kSelThreads, n, m, S, part);
    if (w < m && lane == 0) sel_write<T>(S.st[w], g.k[w], s, out, r0 + w, n_rp);
}

size_t pml_scratch_bytes(int64_t n) {
    (void)n;
    return 3 * kSelGroup * kSelBins * sizeof(uint32_t) +
           (kSelMaxPasses + 1) * kSelGroup * sizeof(SelState) +
           kSelGroup * kSelBlocks * sizeof(double);
}

template <typename T>
static hipError_t run_select(const T *y, int64_t n, const int64_t *ks, int32_t n_rp, void *scratch,
                             double *d_out, hipStream_t s) {
    SelScratch sc;
    sc.hist = (uint32_t *)scratch;
    sc.st = (SelState *)(sc.hist + 3 * kSelGroup * kSelBins);
    sc.psum = (double *)(sc.st + (kSelMaxPasses + 1) * kSelGroup);
    const int64_t want = (n + kSelLosses - 1) / kSelLosses;
    const dim3 g((unsigned)(want < kSelBlocks ? (want < 1 ? 1 : want) : kSelBlocks)), b(kSelThreads);
    for (int r0 = 0; r0 < n_rp; r0 += kSelGroup) {
        const int m = n_rp - r0 < kSelGroup ? n_rp - r0 : kSelGroup;
        SelGroup grp;
        for (int r = 0; r < kSelGroup; ++r) grp.k[r] = r < m ? ks[r0 + r] : 1;
        if (n <= kSelSmall) {
            hipLaunchKernelGGL(k_sel_small<T>, dim3(1), b, 0, s, y, n, grp, m, d_out, r0, n_rp);
            continue;
        }
        // (the first pass counts in one histogram)
        hipLaunchKernelGGL(k_sel_init, dim3(kSelBins / 256), dim3(256), 0, s, sc);
        for (int p = 0; p < sel_passes(KeyOf<T>::bits); ++p)
            hipLaunchKernelGGL(k_sel_hist<T>, g, b, 0, s, y, n, sc, grp, m, p);
        hipLaunchKernelGGL(k_sel_sum<T>, g, b, 0, s, y, n, sc, grp, m);
        hipLaunchKernelGGL(k_sel_finish<T>, dim3(m), dim3(64), 0, s, sc, grp, (int)g.x, d_out, r0, n_rp);
    }
    return hipGetLastError();
}

// ---- exceedance-probability curve ------------------------------------------
constexpr int kSortThreads = 512;
constexpr int kSortIpt = 8;
constexpr int kSortTile = kSortThreads * kSortIpt;   // keys per block and pass

// Key i of a pass: the first pass forms it from the loss (ascending inverted =
// descending losses).
template <typename T, bool FIRST>
__device__ __forceinline__ typename KeyOf<T>::K sort_key(const void *in, int64_t i) {
    if (FIRST) return ~KeyOf<T>::key(static_cast<const T *>(in)[i]);
    return static_cast<const typename KeyOf<T>::K *>(in)[i];
}

template <typename T, bool FIRST>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const void *__restrict__ in, int64_t n,
                                                            int shift, uint32_t *__restrict__ counts,
                                                            int nb) {
    __shared__ uint32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * kSortTile + threadIdx.x;
#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) {
        const int64_t i = t0 + r * kSortThreads;
        if (i < n) atomicAdd(&h[(uint32_t)(sort_key<T, FIRST>(in, i) >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256) counts[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// Block d: the counts of digit d become their inclusive sums over the blocks.
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t *__restrict__ counts, int nb) {
    __shared__ uint32_t sums[4];
    uint32_t *row = counts + (int64_t)blockIdx.x * nb;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 256) {
        const int b = b0 + threadIdx.x;
        const uint32_t v = b < nb ? row[b] : 0u;
        int tot;
        const uint32_t in = v + (uint32_t)wave_excl_scan((int)v, &tot);
        if (lane == 0) sums[w] = (uint32_t)tot;
        __syncthreads();
        uint32_t before = carry;
        for (int q = 0; q < 4; ++q) {
            if (q < w) before += sums[q];
            carry += sums[q];
        }
        if (b < nb) row[b] = before + in;
        __syncthreads();
    }
}

// The lanes of the wavefront whose digit is d, among the valid ones.
__device__ __forceinline__ uint64_t sort_peers(uint32_t d, bool valid) {
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        const bool on = (d >> bit) & 1u;
        const uint64_t b = __ballot(valid && on);
        m &= on ? b : ~b;
    }
    return m;
}

// Ranks of a block's keys within their digits, and the first local position of each
// digit.  A wavefront's keys are runs (up to R) of 64 in a row, ranked in turn (eight
// ballots find the lanes that share a digit) over the counts in its own wcnt, which
// needs no barrier; then the counts are summed over the wavefronts.  Afterwards key
// r of a lane belongs at wcnt[w][its digit] + rank[r].
template <typename K, int R, int W>
__device__ __forceinline__ void sort_rank(const K (&k)[R], int runs, int n_valid, int shift,
                                          uint32_t (*wcnt)[256], uint32_t *sums, uint32_t (&rank)[R]) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < W * 256; i += W * 64) wcnt[0][i] = 0u;
    __syncthreads();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        rank[r] = 0u;
        if (r >= runs || (w * runs + r) * 64 >= n_valid) break;
        const bool valid = (w * runs + r) * 64 + lane < n_valid;
        const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
        const uint64_t m = sort_peers(d, valid);
        const uint32_t at = (uint32_t)__popcll(m & below);
        rank[r] = wcnt[w][d] + at;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (valid && at == 0u) wcnt[w][d] += (uint32_t)__popcll(m);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t total = 0;
    int tot;
    if (threadIdx.x < 256) {
        uint32_t c[W];
#pragma unroll
        for (int q = 0; q < W; ++q) c[q] = wcnt[q][threadIdx.x];
#pragma unroll
        for (int q = 0; q < W; ++q) {
            wcnt[q][threadIdx.x] = total;
            total += c[q];
        }
    }
    uint32_t excl = (uint32_t)wave_excl_scan((int)total, &tot);
    if (threadIdx.x < 256 && lane == 0) sums[w] = (uint32_t)tot;
    __syncthreads();
    if (threadIdx.x < 256) {
        for (int q = 0; q < w; ++q) excl += sums[q];
#pragma unroll
        for (int q = 0; q < W; ++q) wcnt[q][threadIdx.x] += excl;
    }
    __syncthreads();
}

// Stable scatter of one digit: the block's keys are put in the digit's order in LDS
// and written from there, so that equal digits' keys leave in runs.  At 1M keys of 32
// bits a pass takes 18 us (this 9.5, the counts 5.7, their scan by 256 blocks 2.5: one
// block took 12), each a launch of one tile per CU and its latency; the whole curve
// 236 -> 83 us.
template <typename T, bool FIRST, bool LAST>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(const void *__restrict__ in,
                                                               void *__restrict__ out, int64_t n,
                                                               int shift,
                                                               const uint32_t *__restrict__ incl,
                                                               int nb) {
    using K = typename KeyOf<T>::K;
    constexpr int W = kSortThreads / 64;
    __shared__ uint32_t wcnt[W][256];
    __shared__ uint32_t sums[W], base[256];
    __shared__ K sorted[kSortTile];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int64_t t0 = (int64_t)blockIdx.x * kSortTile;
    const int n_valid = (int)(n - t0 < kSortTile ? n - t0 : kSortTile);
    K k[kSortIpt];
    uint32_t rank[kSortIpt];
#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) {
        const int i = w * kSortIpt * 64 + r * 64 + lane;
        k[r] = i < n_valid ? sort_key<T, FIRST>(in, t0 + i) : (K)0;
    }
    // the digit's keys in smaller digits, and in earlier blocks
    uint32_t total = 0, before = 0;
    if (tid < 256) {
        total = incl[(int64_t)tid * nb + nb - 1];
        before = blockIdx.x ? incl[(int64_t)tid * nb + blockIdx.x - 1] : 0u;
    }
    int tot;
    const uint32_t excl = (uint32_t)wave_excl_scan((int)total, &tot);
    if (lane == 0) sums[w] = (uint32_t)tot;
    __syncthreads();
    if (tid < 256) {
        before += excl;
        for (int q = 0; q < w; ++q) before += sums[q];
    }
    __syncthreads();
    sort_rank<K, kSortIpt, W>(k, kSortIpt, n_valid, shift, wcnt, sums, rank);
    if (tid < 256) base[tid] = before - wcnt[0][tid];
#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) {
        const int i = w * kSortIpt * 64 + r * 64 + lane;
        if (i < n_valid) sorted[wcnt[w][(uint32_t)(k[r] >> shift) & 255u] + rank[r]] = k[r];
    }
    __syncthreads();
    for (int i = tid; i < n_valid; i += kSortThreads) {
        const K v = sorted[i];
        const uint32_t at = base[(uint32_t)(v >> shift) & 255u] + (uint32_t)i;
        if (LAST) static_cast<T *>(out)[at] = (T)KeyOf<T>::value(~v);
        else static_cast<K *>(out)[at] = v;
    }
}

// The whole curve by one block, for a YLT of at most kSortSmall losses: the keys stay
// in LDS over the passes.  5,000 losses 26 us (104 us in 19 launches); at the limit,
// which the LDS sets, 68 us, as the passes of many blocks.
constexpr int kSmallThreads = 1024;
constexpr int kSmallIpt = 16;
constexpr int64_t kSortSmall = kSmallThreads * kSmallIpt;

template <typename T>
__global__ __launch_bounds__(kSmallThreads) void k_sort_small(const T *__restrict__ y, int64_t n,
                                                              T *__restrict__ out,
                                                              double *__restrict__ tm) {
    using K = typename KeyOf<T>::K;
    constexpr int W = kSmallThreads / 64;
    __shared__ K keys[kSortSmall];
    __shared__ uint32_t wcnt[W][256];
    __shared__ uint32_t sums[W];
    __shared__ double wsum[W];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = (int)n;
    const int runs = (m + kSmallThreads - 1) / kSmallThreads;    // of 64 keys, a wavefront's
    for (int i = tid; i < m; i += kSmallThreads) keys[i] = ~KeyOf<T>::key(y[i]);
    __syncthreads();
    for (int shift = 0; shift < KeyOf<T>::bits; shift += 8) {
        K k[kSmallIpt];
        uint32_t rank[kSmallIpt];
#pragma unroll
        for (int r = 0; r < kSmallIpt; ++r) {
            const int i = (w * runs + r) * 64 + lane;
            k[r] = r < runs && i < m ? keys[i] : (K)0;
        }
        sort_rank<K, kSmallIpt, W>(k, runs, m, shift, wcnt, sums, rank);
#pragma unroll
        for (int r = 0; r < kSmallIpt; ++r) {
            const int i = (w * runs + r) * 64 + lane;
            if (r < runs && i < m) keys[wcnt[w][(uint32_t)(k[r] >> shift) & 255u] + rank[r]] = k[r];
        }
        __syncthreads();
    }
    for (int i = tid; i < m; i += kSmallThreads) out[i] = (T)KeyOf<T>::value(~keys[i]);
    if (!tm) return;
    // running means: consecutive losses of a lane, then the lanes before, then the
    // wavefronts before
    const int i0 = tid * runs, i1 = min(i0 + runs, m);
    double run = 0.0;
    for (int i = i0; i < i1; ++i) run += KeyOf<T>::value(~keys[i]);
    const double in = wave_incl(run);
    if (lane == 63) wsum[w] = in;
    __syncthreads();
    double at = __shfl_up(in, 1, 64);
    if (lane == 0) at = 0.0;
    double before = 0.0;
    for (int q = 0; q < w; ++q) before += wsum[q];
    at += before;
    for (int i = i0; i < i1; ++i) {
        at += KeyOf<T>::value(~keys[i]);
        tm[i] = at / (double)(i + 1);
    }
}

// Running means of the sorted losses in FP64: block sums, a scan of them, and a
// block-local scan (a run of kSortIpt per thread).
template <typename T>
__global__ __launch_bounds__(kSortThreads) void k_tm_partial(const T *__restrict__ v, int64_t n,
                                                             double *__restrict__ part) {
    __shared__ double s[kSortThreads / 64];
    const int64_t b0 = (int64_t)blockIdx.x * kSortTile + threadIdx.x;
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < kSortIpt; ++j)
        if (b0 + j * kSortThreads < n) acc += (double)v[b0 + j * kSortThreads];
    acc = wave_incl(acc);
    if ((threadIdx.x & 63) == 63) s[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < kSortThreads / 64; ++q) t += s[q];
        part[blockIdx.x] = t;
    }
}

// Exclusive scan of the block sums: a serial run per thread, the runs' sums over the
// wavefronts, tile by tile.
__global__ __launch_bounds__(1024) void k_tm_scan(double *__restrict__ part, int nb) {
    constexpr int kPer = 8;
    __shared__ double wsum[16];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    double carry = 0.0;
    for (int b0 = 0; b0 < nb; b0 += 1024 * kPer) {
        // no more per thread than the tile needs
        const int per = min(kPer, (nb - b0 + 1023) / 1024);
        const int i0 = b0 + tid * per, i1 = min(i0 + per, nb);
        double run = 0.0;
        for (int i = i0; i < i1; ++i) run += part[i];
        const double in = wave_incl(run);
        if (lane == 63) wsum[w] = in;
        __syncthreads();
        double at = __shfl_up(in, 1, 64);
        if (lane == 0) at = 0.0;
        double before = carry;
        for (int q = 0; q < 16; ++q) {
            if (q < w) before += wsum[q];
            carry += wsum[q];
        }
        at += before;
        for (int i = i0; i < i1; ++i) {
            const double v = part[i];
            part[i] = at;
            at += v;
        }
        __syncthreads();
    }
}

template <typename T>
__global__ __launch_bounds__(kSortThreads) void k_tm_final(const T *__restrict__ v, int64_t n,
                                                           const double *__restrict__ part,
                                                           double *__restrict__ tm) {
    __shared__ double s[kSortThreads / 64];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int64_t b0 = (int64_t)blockIdx.x * kSortTile + (int64_t)tid * kSortIpt;
    double x[kSortIpt], acc = 0.0;
#pragma unroll
    for (int j = 0; j < kSortIpt; ++j) x[j] = b0 + j < n ? (double)v[b0 + j] : 0.0;
#pragma unroll
    for (int j = 0; j < kSortIpt; ++j) acc += x[j];
    const double in = wave_incl(acc);
    if (lane == 63) s[w] = in;
    __syncthreads();
    double run = __shfl_up(in, 1, 64);
    if (lane == 0) run = 0.0;
    double before = part[blockIdx.x];
    for (int q = 0; q < w; ++q) before += s[q];
    run += before;
#pragma unroll
    for (int j = 0; j < kSortIpt; ++j) {
        run += x[j];
        if (b0 + j < n) tm[b0 + j] = run / (double)(b0 + j + 1);
    }
}

static int sort_blocks(int64_t n) { return (int)((n + kSortTile - 1) / kSortTile); }

size_t ep_scratch_bytes(int64_t n, int32_t dtype) {
    const size_t ks = dtype == ARA_F64 ? 8 : 4;
    const size_t nb = (size_t)sort_blocks(n > 0 ? n : 1);
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    return up(ks * (size_t)(n > 0 ? n : 1)) + up(sizeof(uint32_t) * 256 * nb) + up(sizeof(double) * nb);
}

template <typename T>
static hipError_t run_ep(const T *y, int64_t n, T *sorted, double *tail_mean, void *scratch,
                         hipStream_t s) {
    using K = typename KeyOf<T>::K;
    if (n <= kSortSmall) {
        hipLaunchKernelGGL((k_sort_small<T>), dim3(1), dim3(kSmallThreads), 0, s, y, n, sorted, tail_mean);
        return hipGetLastError();
    }
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const int nb = sort_blocks(n);
    char *p = (char *)scratch;
    K *tmp = (K *)p;
    uint32_t *counts = (uint32_t *)(p + up(sizeof(K) * (size_t)n));
    double *part = (double *)((char *)counts + up(sizeof(uint32_t) * 256 * (size_t)nb));
    const dim3 g((unsigned)nb), b(kSortThreads);
    // an even number of passes, so the last one writes the losses to sorted
    const void *from = y;
    for (int shift = 0; shift < KeyOf<T>::bits; shift += 8) {
        const bool first = shift == 0, last = shift + 8 == KeyOf<T>::bits;
        void *to = from == (void *)tmp ? (void *)sorted : (void *)tmp;
        if (first) hipLaunchKernelGGL((k_sort_hist<T, true>), g, b, 0, s, from, n, shift, counts, nb);
        else hipLaunchKernelGGL((k_sort_hist<T, false>), g, b, 0, s, from, n, shift, counts, nb);
        hipLaunchKernelGGL(k_sort_scan, dim3(256), dim3(256), 0, s, counts, nb);
        if (first)
            hipLaunchKernelGGL((k_sort_scatter<T, true, false>), g, b, 0, s, from, to, n, shift, counts, nb);
        else if (last)
            hipLaunchKernelGGL((k_sort_scatter<T, false, true>), g, b, 0, s, from, to, n, shift, counts, nb);
        else
            hipLaunchKernelGGL((k_sort_scatter<T, false, false>), g, b, 0, s, from, to, n, shift, counts, nb);
        from = to;
    }
    if (tail_mean) {
        hipLaunchKernelGGL((k_tm_partial<T>), g, b, 0, s, sorted, n, part);
        hipLaunchKernelGGL(k_tm_scan, dim3(1), dim3(1024), 0, s, part, nb);
        hipLaunchKernelGGL((k_tm_final<T>), g, b, 0, s, sorted, n, part, tail_mean);
    }
    return hipGetLastError();
}

hipError_t launch_ep_curve(const void *ylt, int32_t dtype, int64_t n, void *sorted,
                           double *tail_mean, void *scratch, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (dtype == ARA_F64)
        return run_ep<double>((const double *)ylt, n, (double *)sorted, tail_mean, scratch, s);
    return run_ep<float>((const float *)ylt, n, (float *)sorted, tail_mean, scratch, s);
}

hipError_t launch_pml_tvar(const void *ylt, int32_t dtype, int64_t n, const int64_t *ks, int32_t n_rp,
                           void *scratch, double *d_out, hipStream_t s) {
    if (dtype == ARA_F64) return run_select<double>((const double *)ylt, n, ks, n_rp, scratch, d_out, s);
    return run_select<float>((const float *)ylt, n, ks, n_rp, scratch, d_out, s);
}

}  // namespace ara
