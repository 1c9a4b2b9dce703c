// ara_batch.hip -- many portfolios with secondary uncertainty over one YET.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_su.h"

namespace ara {

// ---------------------------------------------------------------------------
// batched portfolios: one persistent launch over (trial tile, portfolio)
// work items, trial-major so the portfolios of one tile run close together
// and share that tile's event ids from cache; an atomic counter hands out the
// items (load balance across portfolios of very different cost)
// ---------------------------------------------------------------------------
__global__ void k_batch_reset(unsigned long long *counter, uint32_t *redo_count) {
    *counter = 0ull;
    *redo_count = 0u;
}

__device__ __forceinline__ void batch_view(const BatchArgs &B, int p, SuArgs &A, PhiloxKeys &keys) {
    const BatchPf &P = B.pfs[p];
    A.off = B.off;
    A.ev = B.ev;
    A.trial_begin = P.trial_begin;
    A.trial_count = P.trial_count;
    A.layers = P.layers;
    A.n_layers = P.n_layers;
    A.elts = P.elts;
    A.evoff = P.evoff;
    A.rowq = P.rowq;
    A.rowf = P.rowf;
    A.row_mean = P.row_mean;
    A.row_cfrac = P.row_cfrac;
    A.row_meta = P.row_meta;
    A.row_lnb = P.row_lnb;
    A.tail_band = B.tail_band;
    A.dev_band = B.dev_band;
    A.ylt_layers = P.ylt_layers;
    A.ylt_pf = P.ylt_pf;
    A.hits = nullptr;
    A.hit_chk = nullptr;
    A.status = B.status;
    A.redo = nullptr;
    A.redo_step = 0;
    A.f64_iters = kF64QuantileIters;
    A.shape_tab = P.shape_tab;
    A.row_shape = nullptr;
    A.occ_view = nullptr;
    A.occ_stride = 0;
    keys.k0 = P.k0;
    keys.k1 = P.k1;
}

// One work item of a batch: a tile of B.tile trials of one portfolio.  The
// item index is wave-uniform; the portfolio and tile are derived from it
// (trial-major: tile-then-portfolio; portfolio-major: each portfolio's block
// of items in turn).
template <int MODE, bool F64OUT, int ROWS>
__device__ __forceinline__ void batch_item(const BatchArgs &B, unsigned long long item,
                                           const SuLds &S) {
    int64_t tile;
    int p;
    if (B.trial_major) {
        tile = (int64_t)(item / (unsigned long long)B.n_pf);
        p = (int)(item % (unsigned long long)B.n_pf);
    } else {
        // the portfolio whose block of work items holds this item
        int lo_p = 0, hi_p = B.n_pf - 1;
        while (lo_p < hi_p) {
            const int mid = (lo_p + hi_p + 1) >> 1;
            if ((unsigned long long)B.pfs[mid].tile_base <= item) lo_p = mid; else hi_p = mid - 1;
        }
        p = lo_p;
        tile = (int64_t)item - B.pfs[p].tile_base;
    }
    // wave-uniform by construction; said explicitly so the portfolio's
    // pointers are read with scalar loads into scalar registers
    p = __builtin_amdgcn_readfirstlane(p);
    tile = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(tile >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)tile));
    SuArgs A;
    PhiloxKeys keys;
    batch_view(B, p, A, keys);
    const int64_t t0 = tile * B.tile;
    const int64_t t1 = (t0 + B.tile) < A.trial_count ? (t0 + B.tile) : A.trial_count;
    for (int64_t t = t0; t < t1; ++t)
        if (su_trial<MODE, F64OUT, false, ROWS>(A, keys, t, S) && threadIdx.x == 0)
            B.redo[atomicAdd(B.redo_count, 1u)] = ((unsigned long long)p << 32) | (uint64_t)t;
}

// Persistent form: grid-wide loop over work items taken from an atomic
// counter (waves_per_cu wavefronts per CU stay resident).
template <int MODE, bool F64OUT, int ROWS>
__device__ __forceinline__ void batch_loop(const BatchArgs &B, const SuLds &S) {
    const unsigned long long n_items = (unsigned long long)B.n_items;
    while (true) {
        unsigned long long item = 0;
        if (threadIdx.x == 0) item = atomicAdd(B.counter, 1ull);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)item);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(item >> 32));
        item = ((unsigned long long)hi << 32) | lo;
        if (item >= n_items) break;
        batch_item<MODE, F64OUT, ROWS>(B, item, S);
    }
}

template <int MODE, bool F64OUT, int ROWS>
__global__ __launch_bounds__(64) void k_ara_batch(BatchArgs B) {
    __shared__ float X[kSeg];
    __shared__ uint2 Q[kQCap];
    __shared__ EltDev El[kEltLds];
    batch_loop<MODE, F64OUT, ROWS>(B, {X, Q, El, nullptr, nullptr});
}

// One workgroup per work item: the dispatcher hands the items out in index
// order as wavefronts retire, and a wavefront keeps no state across items,
// so the kernel runs at the single-portfolio kernel's occupancy.
template <int MODE, bool F64OUT, int ROWS>
__global__ __launch_bounds__(64) ARA_SU_OCCUPANCY(ROWS == SU_ITER ? 6 : 8) void k_ara_batch_items(BatchArgs B) {
    __shared__ float X[kSeg];
    __shared__ uint2 Q[kQCap];
    __shared__ EltDev El[kEltLds];
    const unsigned long long item = blockIdx.x;
    if (item >= (unsigned long long)B.n_items) return;
    batch_item<MODE, F64OUT, ROWS>(B, item, {X, Q, El, nullptr, nullptr});
}

// The full pass: the work items of portfolios with rows that the lean pass
// cannot take (items: one workgroup each, else the persistent form), or the
// trials that the lean pass handed over (redo).
enum { FULL_ITEMS, FULL_LOOP, FULL_REDO };

template <int MODE, bool F64OUT, int FORM>
__global__ __launch_bounds__(64) ARA_FULL_OCCUPANCY void k_ara_batch_full(BatchArgs B) {
    __shared__ float X[kSeg], XH[kSeg];
    __shared__ uint2 Q[kQCap], QH[kHCap];
    __shared__ EltDev El[kEltLds];
    const SuLds S = {X, Q, El, XH, QH};
    if (FORM == FULL_ITEMS) {
        if ((int64_t)blockIdx.x < B.n_items)
            batch_item<MODE, F64OUT, SU_FULL>(B, (unsigned long long)blockIdx.x, S);
    } else if (FORM == FULL_LOOP) {
        batch_loop<MODE, F64OUT, SU_FULL>(B, S);
    } else {
        const uint32_t n = *B.redo_count;
        for (uint32_t r = blockIdx.x; r < n; r += gridDim.x) {
            const unsigned long long e = B.redo[r];
            const int p = (int)(e >> 32);
            const int64_t t = (int64_t)(e & 0xffffffffull);
            // (an entry that no lean pass of this batch wrote: scratch shared with another)
            if (p >= B.n_pf || t >= B.pfs[p].trial_count) {
                if (threadIdx.x == 0) report(B.status, ARA_E_INVALID_ARG, r, p, t);
                continue;
            }
            SuArgs A;
            PhiloxKeys keys;
            batch_view(B, p, A, keys);
            su_trial<MODE, F64OUT, false, SU_FULL>(A, keys, t, S);
        }
    }
}

// grid <= 0: one workgroup per work item (of the lean pass with so much dynamic LDS);
// otherwise the persistent form with that many workgroups.
template <int MODE, bool F64OUT>
static void batch_dispatch(const BatchArgs &B, int grid, int redo_grid, SuForm form, size_t lds, hipStream_t s) {
    const dim3 items((unsigned)B.n_items), loop((unsigned)(grid > 0 ? grid : 1)), b(64);
    hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(1), 0, s, B.counter, B.redo_count);
    if (form == SU_FULL) {
        if (grid <= 0) hipLaunchKernelGGL((k_ara_batch_full<MODE, F64OUT, FULL_ITEMS>), items, b, 0, s, B);
        else hipLaunchKernelGGL((k_ara_batch_full<MODE, F64OUT, FULL_LOOP>), loop, b, 0, s, B);
        return;
    }
    if (form == SU_ITER) {
        if (grid <= 0) hipLaunchKernelGGL((k_ara_batch_items<MODE, F64OUT, SU_ITER>), items, b, lds, s, B);
        else hipLaunchKernelGGL((k_ara_batch<MODE, F64OUT, SU_ITER>), loop, b, 0, s, B);
    } else {
        if (grid <= 0) hipLaunchKernelGGL((k_ara_batch_items<MODE, F64OUT, SU_LEAN>), items, b, lds, s, B);
        else hipLaunchKernelGGL((k_ara_batch<MODE, F64OUT, SU_LEAN>), loop, b, 0, s, B);
    }
    hipLaunchKernelGGL((k_ara_batch_full<MODE, F64OUT, FULL_REDO>), dim3(redo_grid), b, 0, s, B);
}

hipError_t launch_batch(const BatchArgs &B, int mode, bool f64out, int grid, int redo_grid,
                        SuForm form, size_t lds, hipStream_t s) {
    if (B.n_items <= 0 || B.n_pf <= 0) return hipSuccess;
    if (mode == ARA_SUM_NAIVE32) {
        if (f64out) batch_dispatch<ARA_SUM_NAIVE32, true>(B, grid, redo_grid, form, lds, s);
        else batch_dispatch<ARA_SUM_NAIVE32, false>(B, grid, redo_grid, form, lds, s);
    } else if (mode == ARA_SUM_KAHAN32) {
        if (f64out) batch_dispatch<ARA_SUM_KAHAN32, true>(B, grid, redo_grid, form, lds, s);
        else batch_dispatch<ARA_SUM_KAHAN32, false>(B, grid, redo_grid, form, lds, s);
    } else {
        if (f64out) batch_dispatch<ARA_SUM_F64, true>(B, grid, redo_grid, form, lds, s);
        else batch_dispatch<ARA_SUM_F64, false>(B, grid, redo_grid, form, lds, s);
    }
    return hipGetLastError();
}

}  // namespace ara
