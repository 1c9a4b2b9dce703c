// ara_su.hip -- the analysis of one portfolio with secondary uncertainty.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ara_su.h"

namespace ara {

// Lean pass: one wavefront (block) per trial.  ITER: with the FP32 quantile of shapes
// without a slot.  DIAG: every row visited, hit
// counts and checksums (and the occurrence view when asked for); OCC: the
// lean pass that also writes the occurrence view (its per-occurrence sums
// are those of the DIAG pass: the rows it skips add +0).
template <int MODE, bool F64OUT, bool DIAG, bool OCC, bool ITER>
__global__ __launch_bounds__(64) ARA_SU_OCCUPANCY(ITER ? 6 : DIAG || OCC ? 7 : 8) void k_ara_su(SuArgs A, PhiloxKeys keys) {
    __shared__ float X[kSeg];
    __shared__ uint2 Q[kQCap];
    __shared__ EltDev El[kEltLds];
    const SuLds S = {X, Q, El, nullptr, nullptr};
    const int64_t t = blockIdx.x;
    if (t >= A.trial_count) return;
    const bool gone = su_trial<MODE, F64OUT, DIAG, ITER ? SU_ITER : SU_LEAN, OCC>(A, keys, t, S);
    if (threadIdx.x == 0) A.redo[t] = gone;
}

// Full pass, either over every trial (one block each, for portfolios with rows
// that the lean pass cannot take) or over the trials the lean pass flagged, so no
// host round trip is needed between the passes.  (Every trial writes its flag: a list
// with a counter needs a launch that clears it, 2 us of a small run's 19.)
template <int MODE, bool F64OUT, bool DIAG, bool OCC>
__global__ __launch_bounds__(64) ARA_FULL_OCCUPANCY void k_ara_full(SuArgs A, PhiloxKeys keys) {
    __shared__ float X[kSeg], XH[kSeg];
    __shared__ uint2 Q[kQCap], QH[kHCap];
    __shared__ EltDev El[kEltLds];
    const SuLds S = {X, Q, El, XH, QH};
    const uint32_t n = (uint32_t)A.trial_count, step = A.redo_step ? A.redo_step : 1u;
    for (uint32_t r0 = blockIdx.x * step; r0 < n; r0 += gridDim.x * step) {
        uint64_t m = 1;
        if (A.redo_step)
            m = __ballot(threadIdx.x < step && r0 + threadIdx.x < n && A.redo[r0 + threadIdx.x] != 0);
        for (; m; m &= m - 1)
            su_trial<MODE, F64OUT, DIAG, SU_FULL, OCC>(A, keys, (int64_t)(r0 + (uint32_t)__builtin_ctzll(m)), S);
    }
}

// Lean pass of one layer with its event table, or its filter, in LDS: one block of 16
// wavefronts per CU holds it, and each wavefront takes a trial at a time in turn.  The layers of a portfolio are launches of their own, the portfolio
// sum accumulated in their order, so one layer's records at a time (2 MB of 16
// ELTs x 20,000 rows) have the L2s.  A trial that a layer abandons is flagged and
// the full pass runs all its layers again.
//
// The one-wavefront form is bound by its divergent gathers: per 64 occurrences,
// 64 lines of (first record, rows) pairs, 123 cycles of the CU's address unit,
// which was busy 83 % of the time.  Here they are LDS reads (address unit 40 %)
// and the vector units are the bound, busy 80 % of the time with four wavefronts
// per SIMD: the table leaves no LDS for more, so the draws are pipelined
// (su_layer_tab).  1M trials x 16 ELTs 9.83 -> 7.95 ms; 4 portfolios of 5 layers x
// 25,000 trials 6.87 -> 3.68 ms.  With the filter, events without rows gather
// nothing: 100,000 trials x 1,000 over 250,007 events of 0.6 rows 693 -> 463 us, over 1M
// events of 0.3 rows, whose pairs are twice an L2, 1150 -> 463 us.
template <int MODE, bool F64OUT, bool OCC, typename TAB>
__global__ __launch_bounds__(64 * kTabWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_ara_su_tab(
    SuArgs A, PhiloxKeys keys, LayerDev L, int32_t l, const uint32_t *__restrict__ tab,
    int32_t words, int32_t shape) {
    __shared__ __align__(16) uint32_t T[3 * kTabGroups];
    __shared__ __align__(16) float LP[kTabWaves][kLp + kLpPad];
    __shared__ uint16_t ST[kTabWaves][kSeg + 8];
    __shared__ EltDev El[kEltLds];
    for (int i = threadIdx.x; i < words; i += blockDim.x) T[i] = tab[i];
    if (L.n_elts <= kEltLds && (int)threadIdx.x < L.n_elts)
        El[threadIdx.x] = A.elts[L.elt_begin + threadIdx.x];
    __syncthreads();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const LeanLds S = {LP[w], ST[w], El};
    TAB E;
    if constexpr (std::is_same_v<TAB, EvTab>)
        E = {reinterpret_cast<const uint2 *>(T), T + 2 * shape};
    else
        E = {T, reinterpret_cast<const uint2 *>(A.evoff + L.live_base), shape};
    // the next trial's offsets and first ids are on the way while one runs
    const int64_t step = (int64_t)gridDim.x * kTabWaves;
    const int64_t *off = A.off + A.trial_begin;
    int64_t t = (int64_t)blockIdx.x * kTabWaves + w;
    if (t >= A.trial_count) return;
    int64_t o0 = off[t], o1 = off[t + 1];
    SegIds I;
    load_ids(I, A.ev + o0, 0, o1 - o0, L.chunk);
    for (; t < A.trial_count; t += step) {
        const int64_t tn = t + step < A.trial_count ? t + step : t;
        const int64_t p0 = off[tn], p1 = off[tn + 1];
        double Y;
        const bool gone = su_layer_tab<MODE, F64OUT, OCC, TAB>(A, keys, L, l, t, o0, o1 - o0, I,
                                                          A.ev + p0, p1 - p0, S, E, &Y);
        // an abandoned trial, or one of no occurrences, has loaded no ids
        if (gone || o1 == o0) load_ids(I, A.ev + p0, 0, p1 - p0, L.chunk);
        o0 = p0, o1 = p1;
        // the first layer's launch clears the flags of the trials that it finishes
        if (lane == 0 && (gone || l == 0)) A.redo[t] = gone;
        if (gone) continue;
        if (lane == 0 && A.ylt_pf) {
            if (F64OUT) {
                double *p = (double *)A.ylt_pf + t;
                *p = l ? *p + Y : Y;
            } else {
                float *p = (float *)A.ylt_pf + t;
                *p = l ? *p + (float)Y : (float)Y;
            }
        }
    }
}

template <int MODE, bool F64OUT>
static hipError_t su_dispatch2(const SuLaunch &p, hipStream_t s) {
    SuArgs A;
    A.off = p.off; A.ev = p.ev; A.trial_begin = p.trial_begin; A.trial_count = p.trial_count;
    A.layers = p.layers; A.n_layers = p.n_layers; A.elts = p.elts; A.evoff = p.evoff;
    A.rowq = p.rowq; A.rowf = p.rowf; A.row_mean = p.row_mean; A.row_cfrac = p.row_cfrac;
    A.row_meta = p.row_meta;
    A.row_lnb = p.row_lnb;
    A.tail_band = p.tail_band; A.dev_band = p.dev_band; A.ylt_layers = p.ylt_layers; A.ylt_pf = p.ylt_pf;
    A.hits = p.hits; A.hit_chk = p.hit_chk; A.status = p.status;
    A.redo = p.redo; A.f64_iters = p.f64_iters;
    A.shape_tab = p.shape_tab; A.row_shape = p.row_shape;
    A.occ_view = p.occ_view; A.occ_stride = p.occ_stride;
    const PhiloxKeys keys = philox_keys(p.seed);
    const dim3 g((unsigned)p.trial_count), gr((unsigned)p.redo_grid);
    // DIAG first: its occurrence view is written by either instantiation
    const bool diag = p.hits || p.hit_chk, occ = !diag && p.occ_view;
    auto full = [&](const dim3 &grid) {
        if (diag) hipLaunchKernelGGL((k_ara_full<MODE, F64OUT, true, false>), grid, dim3(64), 0, s, A, keys);
        else if (occ) hipLaunchKernelGGL((k_ara_full<MODE, F64OUT, false, true>), grid, dim3(64), 0, s, A, keys);
        else hipLaunchKernelGGL((k_ara_full<MODE, F64OUT, false, false>), grid, dim3(64), 0, s, A, keys);
    };
    A.redo_step = (uint32_t)((p.trial_count + p.redo_grid - 1) / p.redo_grid);
    if (A.redo_step > (uint32_t)kWave) A.redo_step = (uint32_t)kWave;
    if (p.form == SU_FULL) {
        A.redo_step = 0;
        full(g);
        return hipGetLastError();
    }
    if (p.form == SU_TABLE) {
        const bool filter = ev_filter(p.n_cat);
        const int32_t words = (int32_t)evtab_words(p.n_cat);
        const int32_t shape = filter ? filter_shift(p.n_cat) : words / 3;
        const int64_t blocks = (p.trial_count + kTabWaves - 1) / kTabWaves;
        const dim3 gt((unsigned)(blocks < p.n_cu ? blocks : p.n_cu)), bt(64 * kTabWaves);
        auto tab_pass = [&](auto kernel, int32_t l) {
            hipLaunchKernelGGL(kernel, gt, bt, 0, s, A, keys, p.h_layers[l], l,
                               p.evtab + (size_t)l * words, words, shape);
        };
        for (int32_t l = 0; l < p.n_layers; ++l) {
            if (filter && occ) tab_pass(k_ara_su_tab<MODE, F64OUT, true, EvFilter>, l);
            else if (filter) tab_pass(k_ara_su_tab<MODE, F64OUT, false, EvFilter>, l);
            else if (occ) tab_pass(k_ara_su_tab<MODE, F64OUT, true, EvTab>, l);
            else tab_pass(k_ara_su_tab<MODE, F64OUT, false, EvTab>, l);
        }
        full(gr);
        return hipGetLastError();
    }
    auto lean = [&](auto iter) {
        constexpr bool I = decltype(iter)::value;
        if (diag) hipLaunchKernelGGL((k_ara_su<MODE, F64OUT, true, false, I>), g, dim3(64), p.lds, s, A, keys);
        else if (occ) hipLaunchKernelGGL((k_ara_su<MODE, F64OUT, false, true, I>), g, dim3(64), p.lds, s, A, keys);
        else hipLaunchKernelGGL((k_ara_su<MODE, F64OUT, false, false, I>), g, dim3(64), p.lds, s, A, keys);
    };
    if (p.form == SU_ITER) lean(std::true_type());
    else lean(std::false_type());
    full(gr);
    return hipGetLastError();
}

hipError_t launch_su(const SuLaunch &p, int mode, bool f64out, hipStream_t s) {
    if (p.trial_count <= 0) return hipSuccess;
    if (mode == ARA_SUM_NAIVE32) return f64out ? su_dispatch2<ARA_SUM_NAIVE32, true>(p, s)
                                               : su_dispatch2<ARA_SUM_NAIVE32, false>(p, s);
    if (mode == ARA_SUM_KAHAN32) return f64out ? su_dispatch2<ARA_SUM_KAHAN32, true>(p, s)
                                               : su_dispatch2<ARA_SUM_KAHAN32, false>(p, s);
    return f64out ? su_dispatch2<ARA_SUM_F64, true>(p, s) : su_dispatch2<ARA_SUM_F64, false>(p, s);
}

}  // namespace ara
