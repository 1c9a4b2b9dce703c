// ara_su.hip -- the analysis of one portfolio with secondary uncertainty.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_su.h"

namespace ara {

// Lean pass: one wavefront (block) per trial.  DIAG: every row visited, hit
// counts and checksums (and the occurrence view when asked for); OCC: the
// lean pass that also writes the occurrence view (its per-occurrence sums
// are those of the DIAG pass: the rows it skips add +0).
template <int MODE, bool F64OUT, bool DIAG, bool OCC = false>
__global__ __launch_bounds__(64) ARA_SU_OCCUPANCY void k_ara_su(SuArgs A, PhiloxKeys keys) {
    __shared__ float X[kSeg];
    __shared__ uint2 Q[kQCap];
    __shared__ EltDev El[kEltLds];
    const SuLds S = {X, Q, El, nullptr, nullptr};
    const int64_t t = blockIdx.x;
    if (t >= A.trial_count) return;
    if (su_trial<MODE, F64OUT, DIAG, false, OCC>(A, keys, t, S) && threadIdx.x == 0)
        A.redo[atomicAdd(A.redo_count, 1u)] = (int32_t)t;
}

// Full pass, either over every trial (redo null: one block per trial, for
// portfolios with rows that the lean pass cannot take) or over the trials the
// lean pass handed over; that count is read on the device, so no host round
// trip is needed between the passes.
template <int MODE, bool F64OUT, bool DIAG, bool OCC>
__global__ __launch_bounds__(64) ARA_FULL_OCCUPANCY void k_ara_full(SuArgs A, PhiloxKeys keys) {
    __shared__ float X[kSeg], XH[kSeg];
    __shared__ uint2 Q[kQCap], QH[kHCap];
    __shared__ EltDev El[kEltLds];
    const SuLds S = {X, Q, El, XH, QH};
    // the list holds at most one entry per trial of the run; an entry outside
    // the run (scratch shared by runs that overlapped, against the contract)
    // is reported instead of followed
    uint32_t n = (uint32_t)A.trial_count;
    if (A.redo) n = min(n, *A.redo_count);
    for (uint32_t r = blockIdx.x; r < n; r += gridDim.x) {
        const int32_t t = A.redo ? A.redo[r] : (int32_t)r;
        if (t < 0 || (int64_t)t >= A.trial_count) {
            if (threadIdx.x == 0) report(A.status, ARA_E_INVALID_ARG, r, t, A.trial_count);
            continue;
        }
        su_trial<MODE, F64OUT, DIAG, true, OCC>(A, keys, (int64_t)t, S);
    }
}

__global__ void k_reset_u32(uint32_t *p) { *p = 0u; }

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
    A.redo = p.redo; A.redo_count = p.redo_count; A.f64_iters = p.f64_iters;
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
    if (p.full) {
        A.redo = nullptr;
        full(g);
        return hipGetLastError();
    }
    // a kernel, not hipMemsetAsync, so the sequence can be captured in a graph
    hipLaunchKernelGGL(k_reset_u32, dim3(1), dim3(1), 0, s, p.redo_count);
    if (diag) hipLaunchKernelGGL((k_ara_su<MODE, F64OUT, true>), g, dim3(64), 0, s, A, keys);
    else if (occ) hipLaunchKernelGGL((k_ara_su<MODE, F64OUT, false, true>), g, dim3(64), 0, s, A, keys);
    else hipLaunchKernelGGL((k_ara_su<MODE, F64OUT, false>), g, dim3(64), 0, s, A, keys);
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
