// ara_kernels.hip -- gfx950 kernels of Aggregate Risk Analysis.
//
//  * YET validation (section 2.1 (i)).
//  * Portfolio build (sections 3.3 and 4.2): per-ELT direct-access tables over
//    the catalogue, the per-layer event-major row lists, the per-row Beta
//    moment fit, and (without secondary uncertainty) the per-event
//    occurrence-loss table.
//  * The analysis (Algorithm 1 with secondary uncertainty):
//      - k_ara_pu (ara_pu.hip): primary uncertainty only.  The loss of an occurrence is
//        then a function of its event id alone, so the layer's per-event
//        occurrence losses are tabulated once (lookup, ELT terms, cross-ELT
//        sum and occurrence terms for every catalogue event) and a trial is a
//        gather-sum over its event ids followed by the aggregate terms.
//      - k_ara_su (ara_su.hip): secondary uncertainty, the lean pass.  One
//        wavefront per trial; lanes read consecutive occurrences, look each up
//        in the layer's event-major rows, and append the hits to an LDS queue
//        (only the rows that can pay: the others add exactly 0); the queue is
//        drained 64 hits at a time so every lane of a batch draws, reads the
//        quantile of its row's shape slot and applies the ELT terms on real
//        work (the paper's "convergence switching" idea applied to SIMD lanes).
//        With rows of shapes without a slot, an instantiation iterates those in
//        the FP32 domain.
//      - k_ara_su_tab (ara_su.hip): the same for large runs of slotted rows, a
//        layer at a time, with the layer's event table or filter in LDS.
//      - k_ara_full (ara_su.hip): the same trial code with a second queue for
//        the FP64 quantile; it takes the trials that the lean pass hands over
//        (a hit outside the FP32 domain, a draw in the caller's tail band), or
//        every trial where most have such a hit.
//      - k_ara_batch* (ara_batch.hip): the same trial code over (portfolio,
//        trial tile) work items of many portfolios at once.
//      - the occurrence view (per-occurrence increments of the aggregate
//        terms): the OCC instantiations of k_ara_su and k_ara_su_tab, or the
//        VIEW ones of k_ara_pu, through a wavefront's FP64 scan.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_device.h"

namespace ara {

// ---------------------------------------------------------------------------
// YET validation: one wavefront per trial
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_validate_yet(const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ ev,
                                                      const float *__restrict__ times,
                                                      int64_t n_trials, int32_t n_cat,
                                                      Status *st, unsigned long long *max_len) {
    const int lane = threadIdx.x & 63;
    const int64_t wid = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x / 64);
    if (wid == 0 && lane == 0 && off[0] != 0) report(st, ARA_E_OFFSETS_NOT_MONOTONE, 0, off[0], 0);
    const int64_t n_occ = off[n_trials];
    unsigned long long longest = 0;   // this wavefront's longest trial (one atomic per wavefront)
    for (int64_t t = wid; t < n_trials; t += nw) {
        const int64_t a = off[t], b = off[t + 1];
        // a trial is read only when it lies inside [0, offsets[n_trials])
        if (a < 0 || b < a || b > n_occ) {
            if (lane == 0) report(st, ARA_E_OFFSETS_NOT_MONOTONE, t, a, b);
            continue;
        }
        if ((unsigned long long)(b - a) > longest) longest = (unsigned long long)(b - a);
        // four ids (and time pairs) in flight per lane: every load takes an
        // index inside the trial (a lane past its end reads its first
        // element) so they issue together; the checks use the real index
        for (int64_t j0 = a + lane; j0 < b; j0 += 4 * 64) {
            int32_t e[4];
            float t0[4], t1[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t j = j0 + 64 * u;
                const int64_t jj = j < b ? j : a;
                e[u] = ev[jj];
                if (times) {
                    t0[u] = times[jj];
                    t1[u] = times[jj + 1 < b ? jj + 1 : jj];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t j = j0 + 64 * u;
                if (j < b && (e[u] < 0 || e[u] >= n_cat))
                    report(st, ARA_E_EVENT_ID_RANGE, t, j - a, e[u]);
                if (times && j + 1 < b && !(t0[u] <= t1[u]))
                    report(st, ARA_E_TIMES_UNSORTED, t, j - a, 0);
            }
        }
    }
    if (lane == 0 && longest > 0) atomicMax(max_len, longest);
}

// ---------------------------------------------------------------------------
// portfolio build
// ---------------------------------------------------------------------------
__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Row checks that need no other row: finite, non-negative, mean < max_loss
// where the row has secondary uncertainty, event id in range.
__global__ void k_check_rows(const RawRow *__restrict__ raw, int64_t n, int32_t n_cat,
                             int32_t su, Status *st) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const RawRow r = raw[i];
        bool bad = !(r.mean >= 0.0f && r.sigma_i >= 0.0f && r.sigma_c >= 0.0f) ||
                   !isfinite(r.mean) || !isfinite(r.sigma_i) || !isfinite(r.sigma_c);
        if (su && (r.sigma_i + r.sigma_c) > 0.0f)
            bad = bad || !(r.max_loss > r.mean) || !isfinite(r.max_loss);
        if (r.event < 0 || r.event >= n_cat) report(st, ARA_E_EVENT_ID_RANGE, -1, i, r.event);
        else if (bad) report(st, ARA_E_BAD_ELT_ROW, -1, i, 0);
    }
}

// Direct-access tables of one layer: dat[j * n_cat + event] = raw row index
// for the layer's ELT j (section 4.2).  A second row for the same event in
// one ELT is a duplicate.
__global__ void k_dat_scatter(const RawRow *__restrict__ raw, const int64_t *__restrict__ elt_row_off,
                              int32_t elt_begin, int32_t n_elts, int32_t n_cat,
                              int32_t *__restrict__ dat, uint32_t *__restrict__ rank, Status *st) {
    const int64_t r0 = elt_row_off[elt_begin], r1 = elt_row_off[elt_begin + n_elts];
    for (int64_t r = r0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < r1;
         r += (int64_t)gridDim.x * blockDim.x) {
        int lo = 0, hi = n_elts - 1;   // ELT of row r
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (elt_row_off[elt_begin + mid] <= r) lo = mid; else hi = mid - 1;
        }
        const int32_t e = raw[r].event;
        rank[r] = ~0u;                 // until k_ev_count finds the row
        if (e < 0 || e >= n_cat) continue;
        const int32_t old = atomicCAS(&dat[(int64_t)lo * n_cat + e], -1, (int32_t)(r - r0));
        if (old != -1) report(st, ARA_E_BAD_ELT_ROW, -2, r, e);
    }
}

// A row whose ELT terms give 0 for every draw: a loss never exceeds its
// scale (max_l, or the mean when there is no draw), so scale <= retention,
// a zero limit or a zero share make share * min(max(loss - R, 0), L)
// exactly 0.
__device__ __forceinline__ bool row_cannot_pay(const RawRow &rr, const EltDev &ed, int32_t su) {
    const bool det = !su || (double)rr.sigma_i + (double)rr.sigma_c == 0.0;
    const float scale = det ? rr.mean : rr.max_loss;
    return scale <= ed.retention || ed.limit == 0.0f || ed.share == 0.0f;
}

// The rows of each catalogue event of a layer, an event a thread: their number (evoff)
// and that of the rows that can pay (liveoff), both also summed per tile of kEvTile
// events (parts, a row of tiles for each); for each row its ELT and its rank among the
// event's rows that can, or cannot, pay; and the event's occurrence loss when
// secondary uncertainty is off.
__global__ __launch_bounds__(kEvTile) void k_ev_count(
    const int32_t *__restrict__ dat, const RawRow *__restrict__ raw, const EltDev *__restrict__ elts,
    const LayerDev *__restrict__ layer, int32_t n_cat, int32_t su, int32_t tiles,
    uint32_t *__restrict__ evoff, uint32_t *__restrict__ liveoff, uint32_t *__restrict__ parts,
    uint32_t *__restrict__ rank, float *__restrict__ otab) {
    __shared__ uint32_t sums[2][kEvTile / 64];
    const LayerDev L = *layer;
    raw += L.row_base;
    rank += L.row_base;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int32_t e = tile * kEvTile + (int32_t)threadIdx.x;
        uint32_t dead = 0, live = 0;
        float X = 0.0f;
        if (e < n_cat) {
#pragma unroll 4
            for (int j = 0; j < L.n_elts; ++j) {
                const int32_t r = dat[(int64_t)j * n_cat + e];
                if (r < 0) continue;
                const RawRow rr = raw[r];
                const EltDev ed = elts[L.elt_begin + j];
                uint32_t &n = row_cannot_pay(rr, ed, su) ? dead : live;
                rank[r] = (n++ << 16) | (uint32_t)j;
                // (a row that cannot pay adds exactly 0)
                X += ed.share * clampf_terms(rr.mean, ed.retention, ed.limit);
            }
            if (otab) otab[L.otab_base + e] = clampf_terms(X, L.occ_r, L.occ_l);
        }
        if (e <= n_cat) {
            evoff[e] = dead + live;
            liveoff[e] = live;
        }
        const uint32_t c = wave_sum(dead + live), cl = wave_sum(live);
        if (lane == 0) {
            sums[0][w] = c;
            sums[1][w] = cl;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            uint32_t t = 0;
            for (int q = 0; q < kEvTile / 64; ++q) t += sums[threadIdx.x][q];
            parts[(int64_t)threadIdx.x * tiles + tile] = t;
        }
        __syncthreads();
    }
}

// In-place exclusive scan of n values with one 1024-thread block (block b those at
// p + b n): rounds of
// 8 tiles of 1024 values, loaded together (coalesced) and scanned tile by
// tile in order with a wavefront scan and the 16 wavefront totals in LDS.
__global__ __launch_bounds__(1024) void k_scan_excl_u32(uint32_t *p, int64_t n) {
    constexpr int kTiles = 8;
    __shared__ uint32_t wsum[16];
    p += (int64_t)blockIdx.x * n;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t carry = 0;                          // sum of everything before the round
    for (int64_t base = 0; base < n; base += (int64_t)kTiles * 1024) {
        uint32_t v[kTiles];
#pragma unroll
        for (int k = 0; k < kTiles; ++k) {
            const int64_t i = base + (int64_t)k * 1024 + tid;
            v[k] = i < n ? p[i] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kTiles; ++k) {
            int wt;
            // the bits of a uint32 sum are those of the int32 sum
            const uint32_t ex = (uint32_t)wave_excl_scan((int)v[k], &wt);
            if (lane == 0) wsum[w] = (uint32_t)wt;
            __syncthreads();
            uint32_t before = 0, tile = 0;
            for (int q = 0; q < 16; ++q) {
                const uint32_t t = wsum[q];
                before += q < w ? t : 0u;
                tile += t;
            }
            const int64_t i = base + (int64_t)k * 1024 + tid;
            if (i < n) p[i] = carry + before + ex;
            carry += tile;
            __syncthreads();
        }
    }
}

// Beta moment fit of section 3.3 in FP64, then rounded shape parameters.
__device__ void fit_row(const RawRow &r, int32_t su, RowQ *q, uint32_t *flags, float *cfrac,
                        double *lnb64) {
    const double mu = r.mean, si = r.sigma_i, sc = r.sigma_c, mx = r.max_loss;
    const double sigma = si + sc;
    *cfrac = 0.0f;
    if (!su || sigma == 0.0) {
        *flags = ROW_DET;
        q->scale = r.mean;
        q->a = q->b = q->lnb = 0.0f;
        *lnb64 = 0.0;
        return;
    }
    const double mu_b = mu / mx;
    double s_b = sigma / mx;
    const double s_max = sqrt(mu_b * (1.0 - mu_b));
    bool capped = false;
    if (s_b >= s_max) {
        s_b = (1.0 - 1e-6) * s_max;
        capped = true;
    }
    const double rr = s_max / s_b;
    const double kappa = rr * rr - 1.0;
    const float a = (float)(mu_b * kappa), b = (float)((1.0 - mu_b) * kappa);
    const double lnb = lgamma((double)a) + lgamma((double)b) - lgamma((double)a + (double)b);
    q->scale = r.max_loss;
    q->a = a;
    q->b = b;
    q->lnb = (float)(lnb * 1.4426950408889634);   // log2 B(a, b)
    *lnb64 = lnb;
    uint32_t f = 0;
    if (capped || !(a >= kF32MinShape && b >= kF32MinShape && a <= kF32MaxShape &&
                    b <= kF32MaxShape)) {
        f |= ROW_F64;
    } else {
        const int na = cf_terms((double)a, (double)b), nb = cf_terms((double)b, (double)a);
        if (na == 0 || nb == 0) f |= ROW_F64;
        else f |= ((uint32_t)na << 20) | ((uint32_t)nb << 26);
    }
    if (f & ROW_F64)       // pairs for the FP64 fraction (0: adaptive)
        f |= ((uint32_t)cf_pairs((double)a, (double)b, 1e-11, 63) << 20) |
             ((uint32_t)cf_pairs((double)b, (double)a, 1e-11, 63) << 26);
    if (si > 0.0 && sc > 0.0) {
        f |= ROW_CORR;
        *cfrac = (float)(sc / sigma);
    } else if (si == 0.0) {
        f |= ROW_CONLY;
    }
    *flags = f;
}

// The Beta fit of every raw row of the portfolio, one thread per row: the
// fit (FP64 moment fit, ln B and the continued-fraction term counts) is the
// costly part of the build and does not depend on where the row lands.
__global__ void k_fit_rows(const RawRow *__restrict__ raw, int64_t n, int32_t su,
                           RowFit *__restrict__ fit) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        RowFit f;
        fit_row(raw[i], su, &f.q, &f.flags, &f.cfrac, &f.lnb);
        fit[i] = f;
    }
}

// The counts of k_ev_count become offsets: each tile's scan on top of the tiles before
// it; and the (first record, paying rows) pair of each event.
__global__ __launch_bounds__(kEvTile) void k_ev_offsets(uint32_t *__restrict__ evoff,
                                                        uint32_t *__restrict__ liveoff, int32_t n_cat,
                                                        int32_t tiles, const uint32_t *__restrict__ parts,
                                                        uint2 *__restrict__ pairs) {
    __shared__ uint32_t sums[2][kEvTile / 64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int32_t e = tile * kEvTile + (int32_t)threadIdx.x;
        const uint32_t c = e <= n_cat ? evoff[e] : 0u, live = e <= n_cat ? liveoff[e] : 0u;
        int tc, tl;
        uint32_t oc = (uint32_t)wave_excl_scan((int)c, &tc) + parts[tile];
        uint32_t ol = (uint32_t)wave_excl_scan((int)live, &tl) + parts[tiles + tile];
        if (lane == 0) {
            sums[0][w] = (uint32_t)tc;
            sums[1][w] = (uint32_t)tl;
        }
        __syncthreads();
        for (int q = 0; q < w; ++q) {
            oc += sums[0][q];
            ol += sums[1][q];
        }
        if (e <= n_cat) {
            evoff[e] = oc;
            liveoff[e] = ol;
        }
        if (e < n_cat) pairs[e] = make_uint2(ol, live);
        __syncthreads();
    }
}

// Event-major rows of one layer, a raw row a thread: for every catalogue event its
// rows that can pay and then those that cannot, each in the layer's ELT order, with the
// fitted Beta constants; the rows that can pay also as compact records.  With a thread
// per event (and its rows in a loop) the scattered row took its turn behind the 15
// others': 12,000 rows x 16 ELTs over 100,000 events 40 us, now 14.5; with the offsets
// from two launches of one block each (49 us each) a layer's load took 245 us, now 68.
__global__ void k_row_place(const RawRow *__restrict__ raw, const RowFit *__restrict__ fit,
                            const uint32_t *__restrict__ rank, const EltDev *__restrict__ elts,
                            LayerDev *__restrict__ layer, int32_t su,
                            const uint32_t *__restrict__ evoff, const uint2 *__restrict__ pairs,
                            RowQ *__restrict__ rowq, RowF *__restrict__ rowf,
                            float *__restrict__ row_mean, float *__restrict__ row_cfrac,
                            uint32_t *__restrict__ row_meta, double *__restrict__ row_lnb) {
    const LayerDev L = *layer;
    uint32_t fl_or = 0;
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < L.n_rows; i += gridDim.x * blockDim.x) {
        const uint32_t at = rank[L.row_base + i];
        if (at == ~0u) continue;               // a duplicate, already reported
        const RawRow rr = raw[L.row_base + i];
        const RowFit rf = fit[L.row_base + i];
        const uint32_t j = at & 0xffffu, k = at >> 16;
        const bool dead = row_cannot_pay(rr, elts[L.elt_begin + (int32_t)j], su);
        const uint2 own = pairs[rr.event];
        const int64_t pos = (int64_t)evoff[rr.event] + (dead ? own.y + k : k);
        const int64_t row = L.row_base + pos;
        row_lnb[row] = rf.lnb;
        rowq[row] = rf.q;
        row_mean[row] = rr.mean;
        row_cfrac[row] = rf.cfrac;
        row_meta[row] = rf.flags | j;
        fl_or |= rf.flags & ROW_FLAGS;
        if (!dead) {
            RowF F;
            F.scale = rf.q.scale;
            F.meta = rf.flags | j;
            F.rs = (uint32_t)pos << 5;         // shape set by k_shape_assign
            F.cfrac = rf.cfrac;
            rowf[L.row_base + own.x + k] = F;
        }
    }
    // one atomic per wavefront and flag at most
    for (uint32_t f = ROW_DET; f <= ROW_CONLY; f <<= 1)
        if (__any(fl_or & f) && (threadIdx.x & 63) == 0) atomicOr(&layer->flags, f);
}

// ---------------------------------------------------------------------------
// primary uncertainty: per-event occurrence-loss table, gather-sum per trial
// ---------------------------------------------------------------------------
// Sparse form of a layer's otab: bit w*32+i of bits[] set when otab is
// non-zero, rank[w] = set bits before word w (exclusive scan), vals[] the
// non-zero values in event order.  Lookup of event E: one LDS word, and for
// the (rare) non-zero events the rank and the value.
__global__ void k_sp_bits(const float *__restrict__ otab, int32_t n_cat, uint32_t *__restrict__ bits,
                          uint32_t *__restrict__ rank) {
    const int32_t nw = (n_cat + 31) >> 5;
    for (int32_t w = blockIdx.x * blockDim.x + threadIdx.x; w <= nw; w += gridDim.x * blockDim.x) {
        uint32_t b = 0;
        if (w < nw)
            for (int i = 0; i < 32; ++i) {
                const int32_t e = w * 32 + i;
                if (e < n_cat && otab[e] != 0.0f) b |= 1u << i;
            }
        if (w < nw) bits[w] = b;
        rank[w] = __popc(b);
    }
}

__global__ void k_sp_vals(const float *__restrict__ otab, int32_t n_cat,
                          const uint32_t *__restrict__ bits, const uint32_t *__restrict__ rank,
                          float *__restrict__ vals, LayerDev *layer) {
    const int32_t nw = (n_cat + 31) >> 5;
    for (int32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < nw; w += gridDim.x * blockDim.x) {
        uint32_t b = bits[w], r = rank[w];
        while (b) {
            const int i = __ffs(b) - 1;
            vals[r++] = otab[w * 32 + i];
            b &= b - 1;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) layer->nnz = (int32_t)rank[nw];
}

// ---------------------------------------------------------------------------
// diagnostics
// ---------------------------------------------------------------------------
__global__ void k_debug_philox(int64_t n, const uint32_t *__restrict__ ctr, PhiloxKeys keys,
                               uint32_t *__restrict__ out) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x) {
        const uint4 c = make_uint4(ctr[4 * j], ctr[4 * j + 1], ctr[4 * j + 2], ctr[4 * j + 3]);
        const uint4 r = philox10(c, keys);
        out[4 * j] = r.x;
        out[4 * j + 1] = r.y;
        out[4 * j + 2] = r.z;
        out[4 * j + 3] = r.w;
        if (philox10_x0(c, keys) != r.x) out[4 * j] = ~r.x;   // both forms must agree
    }
}

// tab: a shape table built for every entry's (a, b) (one shape), or null
__global__ __launch_bounds__(64) void k_debug_quantile(int64_t n, const float *__restrict__ a,
                                                       const float *__restrict__ b,
                                                       const double *__restrict__ z,
                                                       const double *__restrict__ zc, float tail,
                                                       const float *__restrict__ tab,
                                                       float *__restrict__ x,
                                                       int32_t *__restrict__ path) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const float A = a[j], B = b[j];
    const float zf = (float)z[j], zcf = (float)zc[j];
    const bool shape_ok = A >= kF32MinShape && B >= kF32MinShape && A <= kF32MaxShape &&
                          B <= kF32MaxShape;
    bool use64 = !shape_ok || fminf(zf, zcf) < tail;
    const double lnb = lgamma((double)A) + lgamma((double)B) - lgamma((double)A + (double)B);
    float r = 0.0f;
    if (!use64) {
        const int na = cf_terms((double)A, (double)B), nb = cf_terms((double)B, (double)A);
        if (na == 0 || nb == 0) use64 = true;
        else {
            bool ok;
            if (tab) {
                r = slot_quantile(tab, min((uint32_t)(z[j] * 16777216.0) | 1u, 16777215u));
                ok = true;
            } else {
                r = beta_quantile32(A, B, (float)(lnb * 1.4426950408889634), na, nb, zf, zcf, &ok);
            }
            if (!ok) use64 = true;
        }
    }
    if (use64) {
        bool ok;
        r = (float)beta_quantile64((double)A, (double)B, lnb, cf_pairs((double)A, (double)B, 1e-11, 63),
                                   cf_pairs((double)B, (double)A, 1e-11, 63), z[j], zc[j],
                                   kF64QuantileIters, &ok);
        if (!ok) r = __builtin_nanf("");
    }
    x[j] = r;
    if (path) path[j] = use64 ? 1 : 0;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline int grid_for(int64_t n, int block, int cap = 65536) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

hipError_t launch_validate_yet(const int64_t *off, const int32_t *ev, const float *times,
                               int64_t n_trials, int32_t n_cat, Status *st,
                               unsigned long long *max_len, hipStream_t s) {
    // a resident grid (8 blocks of 4 wavefronts per CU of the largest part)
    // that strides over the trials: one atomic per wavefront for the longest
    // trial, not one per trial on a single address
    const int g = grid_for(n_trials, 4, 2048);
    hipLaunchKernelGGL(k_validate_yet, dim3(g), dim3(256), 0, s, off, ev, times, n_trials, n_cat,
                       st, max_len);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_check_rows(const RawRow *raw, int64_t n, int32_t n_cat, int32_t su, Status *st,
                             hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_rows, dim3(grid_for(n, 256)), dim3(256), 0, s, raw, n, n_cat, su, st);
    return hipGetLastError();
}

hipError_t launch_fit_rows(const RawRow *raw, int64_t n, int32_t su, RowFit *fit, hipStream_t s) {
    if (n > 0)
        hipLaunchKernelGGL(k_fit_rows, dim3(grid_for(n, 256)), dim3(256), 0, s, raw, n, su, fit);
    return hipGetLastError();
}

hipError_t launch_build_layer(const RawRow *raw, const RowFit *fit, const int64_t *elt_row_off,
                              const EltDev *elts,
                              LayerDev *d_layer, const LayerDev &h_layer, int32_t n_cat, int32_t su,
                              int32_t *dat, uint32_t *evoff, uint32_t *liveoff, uint32_t *rank,
                              uint32_t *parts, RowQ *rowq, RowF *rowf, float *row_mean,
                              float *row_cfrac, uint32_t *row_meta, double *row_lnb, float *otab,
                              Status *st, hipStream_t s) {
    const int64_t nd = (int64_t)h_layer.n_elts * n_cat;
    const int32_t tiles = ev_tiles(n_cat);
    hipError_t e = launch_fill_i32(dat, nd > 0 ? nd : 1, -1, s);
    if (e != hipSuccess) return e;
    if (h_layer.n_rows > 0)
        hipLaunchKernelGGL(k_dat_scatter, dim3(grid_for(h_layer.n_rows, 256)), dim3(256), 0, s,
                           raw, elt_row_off, h_layer.elt_begin, h_layer.n_elts, n_cat, dat, rank, st);
    uint32_t *eo = evoff + h_layer.evoff_base;
    uint2 *pairs = reinterpret_cast<uint2 *>(evoff + h_layer.live_base);
    const dim3 g((unsigned)(tiles < 65536 ? tiles : 65536)), b(kEvTile);
    hipLaunchKernelGGL(k_ev_count, g, b, 0, s, dat, raw, elts, d_layer, n_cat, su, tiles, eo, liveoff,
                       parts, rank, otab);
    hipLaunchKernelGGL(k_scan_excl_u32, dim3(2), dim3(1024), 0, s, parts, (int64_t)tiles);
    hipLaunchKernelGGL(k_ev_offsets, g, b, 0, s, eo, liveoff, n_cat, tiles, parts, pairs);
    if (h_layer.n_rows > 0)
        hipLaunchKernelGGL(k_row_place, dim3(grid_for(h_layer.n_rows, 256)), dim3(256), 0, s, raw, fit,
                           rank, elts, d_layer, su, eo, pairs, rowq, rowf, row_mean, row_cfrac,
                           row_meta, row_lnb);
    return hipGetLastError();
}

// The event table of one layer from its (first record, paying rows) pairs.
__global__ void k_ev_table(const uint2 *__restrict__ pairs, int32_t n_cat, int32_t groups,
                           uint32_t *__restrict__ tab, LayerDev *__restrict__ layer) {
    uint32_t top = 0;
    for (int32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < groups; g += gridDim.x * blockDim.x) {
        uint64_t w = 0;
        uint32_t most = 0;
        for (int i = 0; i < kTabGroup; ++i) {
            const int32_t e = g * kTabGroup + i;
            const uint32_t c = e < n_cat ? pairs[e].y : 0u;
            most = max(most, c);
            w |= (uint64_t)(c & 15u) << (4 * i);
        }
        tab[2 * g] = (uint32_t)w;
        tab[2 * g + 1] = (uint32_t)(w >> 32);
        tab[2 * groups + g] = pairs[g * kTabGroup].x;
        top = max(top, most);
    }
    if (top > 15u || layer->n_rows >= (1 << kMarkRow)) atomicOr(&layer->flags, LAYER_DENSE);
    // a chunk of the table form: as many occurrences as surely fit a segment's hits
    if (top > (uint32_t)(kLp / kWave)) atomicMin(&layer->chunk, (int32_t)((uint32_t)kLp / top));
}

// The event filter of one layer, a thread per bit.
__global__ void k_ev_filter(const uint2 *__restrict__ pairs, int32_t n_cat, int32_t shift, int32_t words,
                            uint32_t *__restrict__ tab, LayerDev *__restrict__ layer) {
    uint32_t top = 0;
    const int64_t bits = (int64_t)words * 32;
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < ((bits + 63) & ~(int64_t)63);
         b += (int64_t)gridDim.x * blockDim.x) {
        uint32_t most = 0;
        for (int64_t e = b << shift; e < min((b + 1) << shift, (int64_t)n_cat); ++e)
            most = max(most, pairs[e].y);
        const uint64_t m = __ballot(most != 0u);
        if ((b & 31) == 0 && b < bits) tab[b >> 5] = (uint32_t)(b & 32 ? m >> 32 : m);
        top = max(top, most);
    }
    if (top > 15u || layer->n_rows >= (1 << kMarkRow)) atomicOr(&layer->flags, LAYER_DENSE);
    if (top > (uint32_t)(kLp / kWave)) atomicMin(&layer->chunk, (int32_t)((uint32_t)kLp / top));
}

hipError_t launch_event_table(const uint32_t *pairs, int32_t n_cat, uint32_t *tab, LayerDev *d_layer,
                              hipStream_t s) {
    if (ev_filter(n_cat)) {
        const int32_t words = (int32_t)evtab_words(n_cat);
        hipLaunchKernelGGL(k_ev_filter, dim3(grid_for((int64_t)words * 32, 256, 4096)), dim3(256), 0, s,
                           reinterpret_cast<const uint2 *>(pairs), n_cat, filter_shift(n_cat), words,
                           tab, d_layer);
        return hipGetLastError();
    }
    const int32_t groups = (n_cat - 1) / kTabGroup + 1;
    hipLaunchKernelGGL(k_ev_table, dim3(grid_for(groups, 256)), dim3(256), 0, s,
                       reinterpret_cast<const uint2 *>(pairs), n_cat, groups, tab, d_layer);
    return hipGetLastError();
}

hipError_t launch_build_sparse(const float *otab, int32_t n_cat, uint32_t *bits, uint32_t *rank,
                               float *vals, LayerDev *d_layer, hipStream_t s) {
    const int32_t nw = (n_cat + 31) >> 5;
    hipLaunchKernelGGL(k_sp_bits, dim3(grid_for((int64_t)nw + 1, 256)), dim3(256), 0, s, otab, n_cat,
                       bits, rank);
    hipLaunchKernelGGL(k_scan_excl_u32, dim3(1), dim3(1024), 0, s, rank, (int64_t)nw + 1);
    hipLaunchKernelGGL(k_sp_vals, dim3(grid_for(nw, 256)), dim3(256), 0, s, otab, n_cat, bits, rank,
                       vals, d_layer);
    return hipGetLastError();
}

hipError_t launch_debug_philox(int64_t n, const uint32_t *ctr, uint64_t key, uint32_t *out,
                               hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_debug_philox, dim3(grid_for(n, 256)), dim3(256), 0, s, n, ctr,
                       philox_keys(key), out);
    return hipGetLastError();
}

hipError_t launch_debug_quantile(int64_t n, const float *a, const float *b, const double *z,
                                 const double *zc, float tail, const float *tab, float *x,
                                 int32_t *path, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_debug_quantile, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, n, a, b,
                       z, zc, tail, tab, x, path);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// shape tables
// ---------------------------------------------------------------------------
// The distinct Beta shapes of one layer's paying rows on the FP32 quantile
// path into kShapeSlots slots, by a rule that depends on the rows alone (so
// every load of a portfolio gives every row the same path): the first distinct
// ones, in row order, among the layer's first kShapeScan paying rows, found one
// after the other as the first row whose shape has no slot yet (one block per
// layer, its keys in registers, 6 us; lists per thread merged by one thread
// took 72; keys [kShapeSlots] receives the slots, 0 = unused).  k_shape_assign then gives
// every paying row 1 + its slot, or 0, in its compact record and in the
// per-row array.
constexpr uint32_t kShapeScan = 4096;

__device__ __forceinline__ bool shape_eligible(const RowF &F) {
    return !(F.meta & (ROW_DET | ROW_F64));
}
__device__ __forceinline__ unsigned long long shape_key(const RowQ &q) {
    return ((unsigned long long)__float_as_uint(q.a) << 32) | __float_as_uint(q.b);
}

__global__ __launch_bounds__(1024) void k_shape_collect(const RowF *__restrict__ rowf,
                                                        const RowQ *__restrict__ rowq,
                                                        int64_t row_base,
                                                        const uint32_t *__restrict__ liveoff,
                                                        int32_t n_cat,
                                                        unsigned long long *__restrict__ keys) {
    constexpr int kPer = kShapeScan / 1024;
    __shared__ uint32_t first[16];
    __shared__ unsigned long long slot[kShapeSlots];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const uint32_t n = min(liveoff[n_cat], kShapeScan);
    unsigned long long key[kPer];          // of row q * 1024 + tid, 0: none, or in a slot
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const uint32_t i = (uint32_t)(q * 1024 + tid);
        key[q] = 0ull;
        if (i < n) {
            const RowF F = rowf[row_base + i];
            if (shape_eligible(F)) key[q] = shape_key(rowq[row_base + rowf_row(F)]);
        }
    }
    if (tid < kShapeSlots) slot[tid] = 0ull;
    for (int k = 0; k < kShapeSlots; ++k) {
        uint32_t f = ~0u;
#pragma unroll
        for (int q = kPer - 1; q >= 0; --q) {
            const uint64_t m = __ballot(key[q] != 0ull);
            if (m) f = (uint32_t)(q * 1024 + w * 64 + __builtin_ctzll(m));
        }
        if (lane == 0) first[w] = f;
        __syncthreads();
        f = first[0];
#pragma unroll
        for (int q = 1; q < 16; ++q) f = min(f, first[q]);
        if (f == ~0u) break;
#pragma unroll
        for (int q = 0; q < kPer; ++q)
            if (f == (uint32_t)(q * 1024 + tid)) slot[k] = key[q];
        __syncthreads();
        const unsigned long long mine = slot[k];
#pragma unroll
        for (int q = 0; q < kPer; ++q)
            if (key[q] == mine) key[q] = 0ull;
    }
    __syncthreads();
    if (tid < kShapeSlots) keys[tid] = slot[tid];
}

__global__ __launch_bounds__(256) void k_shape_assign(RowF *__restrict__ rowf,
                                                      const RowQ *__restrict__ rowq, int64_t row_base,
                                                      const uint32_t *__restrict__ liveoff,
                                                      int32_t n_cat,
                                                      const unsigned long long *__restrict__ keys,
                                                      uint32_t *__restrict__ row_shape,
                                                      LayerDev *__restrict__ layer) {
    __shared__ unsigned long long slot[kShapeSlots];
    if (threadIdx.x < kShapeSlots) slot[threadIdx.x] = keys[threadIdx.x];
    __syncthreads();
    const uint32_t n = liveoff[n_cat];
    bool slow = false, iter = false;       // rows without a slot; for the FP32 iteration
    int32_t n_f64 = 0, n_mix = 0;          // for the FP64 quantile; mixed, with a slot
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        RowF &F = rowf[row_base + i];
        uint32_t sh = 0;
        if (shape_eligible(F)) {
            const unsigned long long key = shape_key(rowq[row_base + rowf_row(F)]);
            for (int k = 0; k < kShapeSlots; ++k)
                if (slot[k] == key) {
                    sh = (uint32_t)k + 1u;
                    break;
                }
        }
        F.rs = (F.rs & ~31u) | sh;
        row_shape[row_base + rowf_row(F)] = sh;
        if (sh == 0u && !(F.meta & ROW_DET)) {
            slow = true;
            if (F.meta & (ROW_F64 | ROW_CORR)) ++n_f64;
            else iter = true;
        }
        if (sh != 0u && (F.meta & ROW_CORR)) ++n_mix;
    }
    const uint32_t fl = (__any(slow) ? LAYER_SLOW : 0u) | (__any(iter) ? LAYER_ITER : 0u);
    n_f64 = wave_sum(n_f64);
    n_mix = wave_sum(n_mix);
    if ((threadIdx.x & 63) != 0) return;
    if (fl) atomicOr(&layer->flags, fl);
    if (n_f64) atomicAdd(&layer->n_f64, n_f64);
    if (n_mix) atomicAdd(&layer->n_mix, n_mix);
}

// The segments of the used slots, and after them the normal segments: one
// block per slot, one thread per interpolation point, then one per segment.
constexpr int kSlotSegs = 2 * kOctaves + kDevSegs;

__global__ __launch_bounds__(kSlotSegs *kSegCoefs) void k_shape_tables(
    const unsigned long long *__restrict__ keys, int32_t n_slots, float *__restrict__ tab) {
    __shared__ double y[kSlotSegs * kSegCoefs];
    const int seg = threadIdx.x / kSegCoefs, q = threadIdx.x % kSegCoefs;
    float *slot = tab + (size_t)blockIdx.x * kShapeStride;
    if ((int)blockIdx.x == n_slots) {
        // Phi^-1 on the lower half: -sqrt(2) erfcinv(2 z)
        if (seg < kOctaves)
            y[threadIdx.x] = -1.4142135623730951 * erfcinv(ldexp(1.5 + seg_node(q), seg - 23));
        __syncthreads();
        if ((int)threadIdx.x < kOctaves)
            seg_fit(y + threadIdx.x * kSegCoefs, slot + threadIdx.x * kSegCoefs);
        return;
    }
    const unsigned long long key = keys[blockIdx.x];
    if (key == 0ull) return;
    const double a = (double)__uint_as_float((uint32_t)(key >> 32));
    const double b = (double)__uint_as_float((uint32_t)key);
    const double lnb = lgamma(a) + lgamma(b) - lgamma(a + b);
    y[threadIdx.x] = slot_point(a, b, lnb, seg, q);
    __syncthreads();
    const int s = threadIdx.x;
    if (s < kSlotSegs) {
        const int at = s < kOctaves ? s : s < 2 * kOctaves ? kSegUpper + s - kOctaves
                                                           : kSegDev + s - 2 * kOctaves;
        seg_fit(y + s * kSegCoefs, slot + at * kSegCoefs);
    }
}

hipError_t launch_shape_collect(RowF *rowf, const RowQ *rowq, int64_t row_base, int64_t n_rows,
                                const uint32_t *liveoff, int32_t n_cat, uint32_t *row_shape,
                                unsigned long long *keys, LayerDev *d_layer, hipStream_t s) {
    hipLaunchKernelGGL(k_shape_collect, dim3(1), dim3(1024), 0, s, rowf, rowq, row_base, liveoff,
                       n_cat, keys);
    // a grid over the layer's rows (the paying ones are a prefix of them)
    hipLaunchKernelGGL(k_shape_assign, dim3(grid_for(n_rows > 0 ? n_rows : 1, 256, 1024)),
                       dim3(256), 0, s, rowf, rowq, row_base, liveoff, n_cat, keys, row_shape, d_layer);
    return hipGetLastError();
}

hipError_t launch_shape_tables(const unsigned long long *keys, int64_t n_slots, float *tab,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_shape_tables, dim3((unsigned)n_slots + 1), dim3(kSlotSegs * kSegCoefs), 0,
                       s, keys, (int32_t)n_slots, tab);
    return hipGetLastError();
}

}  // namespace ara
