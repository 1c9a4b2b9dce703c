// ara_su.h -- one trial of the analysis with secondary uncertainty, for the run
// kernels (ara_su.hip) and the batched ones (ara_batch.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_internal.h"
#include "ara_math.h"
#include "ara_device.h"

namespace ara {

// ---------------------------------------------------------------------------
// secondary uncertainty
// ---------------------------------------------------------------------------
// LDS per wavefront: X[kSeg] floats + Q[kQCap] pairs = 4 KB, so LDS allows 40
// waves per CU and the register budget sets the occupancy (7 per SIMD,
// measured best on the full-shape workload against 5, 6 and 8)
constexpr int kSeg = 512;         // occurrences per LDS segment
constexpr int kQCap = 256;        // hit queue (power of two)
#define ARA_SU_OCCUPANCY __attribute__((amdgpu_waves_per_eu(7, 7)))
#define ARA_FULL_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4, 4)))
// A layer's ELT records are staged in LDS when it has at most this many ELTs
// (1 KB more per wavefront, still within the occupancy above); the draw then
// needs one global load (the row) before its Philox key is known.
constexpr int kEltLds = 64;
constexpr int kQMask = kQCap - 1;
// The full pass's own LDS: the occurrence sums of hits from its second queue
// and that queue (a light batch adds at most 64 entries to fewer than 64).
constexpr int kHCap = 128;
constexpr int kHMask = kHCap - 1;
constexpr int kPerLane = (kQCap - kWave) / kWave;   // hits a lane appends per sub-step

struct SuArgs {
    const int64_t *off;
    const int32_t *ev;
    int64_t trial_begin, trial_count;
    const LayerDev *layers;
    int32_t n_layers;
    const EltDev *elts;
    const uint32_t *evoff;
    const RowQ *rowq;
    const RowF *rowf;
    const float *row_mean;
    const float *row_cfrac;
    const uint32_t *row_meta;
    const double *row_lnb;
    float tail_band;
    float dev_band;           // |Phi^-1(z)| from which a mixed draw takes the FP64 quantile
    void *ylt_layers;
    void *ylt_pf;
    int64_t *hits;
    uint64_t *hit_chk;
    Status *status;
    int32_t *redo;            // trials (relative index) handed to the FP64-capable pass
    uint32_t *redo_count;
    int32_t f64_iters;        // step limit of the FP64 quantile
    const float *shape_tab;   // the portfolio's shape tables ([layer][kShapeSlots][kShapeStride],
                              // then the normal segments)
    const uint32_t *row_shape;   // per row: 1 + its shape slot, or 0 (the diagnostic pass)
    void *occ_view;           // occurrence view, written by the DIAG and OCC instantiations
    int64_t occ_stride;
};

// The two uniforms of a hit on the 2^-24 grid (j such that u = j 2^-24):
// jI for the independent part, jC for the correlated part, drawn only when
// the row needs them.  Occurrence keying: (k, i, elt_id, 0) and (k, i, 0, 1);
// paper keying (section 3.1's z_(Prog,E) and z_(E)): (k, i, program, 2) and
// (E, 0, 0, 3).
__device__ __forceinline__ void draw_j(uint32_t flags, int32_t keying, uint32_t k, uint32_t i,
                                       uint32_t elt_id, uint32_t program, uint32_t event,
                                       const PhiloxKeys &keys, uint32_t *jI, uint32_t *jC) {
    const bool paper = keying == ARA_KEYING_PAPER;
    const uint4 cI = paper ? make_uint4(k, i, program, 2u) : make_uint4(k, i, elt_id, 0u);
    const uint4 cC = paper ? make_uint4(event, 0u, 0u, 3u) : make_uint4(k, i, 0u, 1u);
    *jI = (flags & ROW_CONLY) ? 0u : u24(philox10_x0(cI, keys));
    *jC = (flags & (ROW_CONLY | ROW_CORR)) ? u24(philox10_x0(cC, keys)) : 0u;
}

// z and 1 - z of a hit in FP64 (section 3.2).  A pure independent or
// correlated draw is an exact grid value u = j 2^-24 (and 1 - u is exact too);
// the mixed case maps both uniforms through Phi^-1, mixes, and maps back with
// the smaller of Phi(v), Phi(-v).  Phi^-1 is one Halley step in FP64 from the
// FP32 segments (5e-7 -> 1e-18), on the side of the smaller tail: erfcinv spills
// 1.2 KB a lane here.
__device__ __attribute__((noinline)) inline void hit_z(uint32_t meta, uint32_t jI, uint32_t jC,
                                                       double cfrac, const float *norm, double *z,
                                                       double *zc) {
    const double s24 = 5.9604644775390625e-08;
    if (!(meta & ROW_CORR)) {
        const uint32_t j = (meta & ROW_CONLY) ? jC : jI;
        *z = (double)j * s24;
        *zc = (double)(16777216u - j) * s24;
        return;
    }
    double v = 0.0, w = 1.0 - cfrac;
    const double n2 = w * w + cfrac * cfrac;
    uint32_t j = jI;
    double t = 0.0;
#pragma unroll 1
    for (int q = 0; q < 3; ++q) {        // one copy of erfc: the two draws, then their mix
        const bool low = j < 8388608u;
        const double d = q < 2 ? -fabs((double)norm_dev(norm, j)) : -fabs(v);
        t = 0.5 * erfc(-d * 0.70710678118654752);
        if (q < 2) {
            const double p = (double)(low ? j : 16777216u - j) * s24;
            const double u = (t - p) * 2.5066282746310002 * exp(0.5 * d * d);
            const double x = d - u / (1.0 + 0.5 * d * u);
            v += (low ? x : -x) * w;
            j = jC;
            w = cfrac;
            if (q == 1) v /= sqrt(n2);
        }
    }
    *z = v < 0.0 ? t : 1.0 - t;
    *zc = v < 0.0 ? 1.0 - t : t;
}

// LDS of one wavefront.
struct SuLds {
    float *X;        // [kSeg] occurrence sums
    uint2 *Q;        // [kQCap] hit queue: (occurrence in the segment, row)
    EltDev *El;      // [kEltLds]
    float *XH;       // full pass: [kSeg] sums of the second queue's hits
    uint2 *QH;       // full pass: [kHCap]
};

// One trial of the analysis, all layers (Algorithm 1 from the layer loop
// down).
//
// FULL = false is the lean pass: rows without a draw and rows whose shape has
// a slot.  A draw outside the slot's range (the caller's tail band) abandons
// the trial, which is then queued for the full pass.  Returns true when
// abandoned.
//
// FULL = true takes every row.  What a light batch cannot finish in FP32
// (shapes outside the FP32 domain, the tail band, the mix of shapes without a
// slot, FP32 non-convergence) goes to a second queue and is drained 64 at a
// time by the FP64 quantile, so that neither kind of hit waits with idle lanes
// for the other.  The hits of the second queue are summed apart (XH) and the
// two sums added per occurrence: each is in (occurrence, row) order and a
// hit's queue depends on its row and draw alone, so the result does not depend
// on how the batches fell.  It is bound by the FP64 arithmetic and latency of
// the second queue: 20,011 trials x 16 ELTs with every row its own shape take
// 1.89 ms (27.4 ms when the lean pass ran first, handed every trial over, and
// each wavefront ran both kinds of hit in one batch until its last FP64 lane
// converged), with 30 % capped rows 0.77 ms (36.6 ms).  Four wavefronts per SIMD
// (128 VGPRs): the FP64 quantile is a call of its own, since inlined its
// hoisted constants spill 450 registers; as a call 42.
template <int MODE, bool F64OUT, bool DIAG, bool FULL, bool OCC = false>
__device__ __forceinline__ bool su_trial(const SuArgs &A, const PhiloxKeys &keys, int64_t t,
                                         const SuLds &S) {
    float *X = S.X;
    uint2 *Q = S.Q;
    EltDev *El = S.El;
    const int lane = threadIdx.x;
    const int64_t ti = A.trial_begin + t;
    const uint32_t i_abs = (uint32_t)ti;
    const int64_t o0 = A.off[ti];
    const int64_t n = A.off[ti + 1] - o0;
    double pf_sum = 0.0;
    const float *norm = A.shape_tab + (size_t)A.n_layers * kShapeSlots * kShapeStride;

    for (int l = 0; l < A.n_layers; ++l) {
        const LayerDev L = A.layers[l];
        const uint32_t *eo = A.evoff + L.evoff_base;
        const int64_t rb0 = L.row_base;
        const bool elt_lds = L.n_elts <= kEltLds;
        if (elt_lds) {
            __syncthreads();
            for (int i = lane; i < L.n_elts; i += kWave) El[i] = A.elts[L.elt_begin + i];
            __syncthreads();
        }
        Acc<MODE> acc;
        uint64_t chk = 0;
        int64_t nh = 0;
        double occ_s = 0.0, occ_a = 0.0;      // occurrence-view carries
        (void)occ_s;
        (void)occ_a;

        // the layer's ELT record: an LDS read when the layer's records are
        // staged (the global read is a different instruction, so the two are
        // not merged into one flat load)
        auto elt_of = [&](uint32_t ei) {
            EltDev ed;
            if (elt_lds) {
                ed = El[ei];
            } else {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                const u32x4 g = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x4 *>(A.elts + L.elt_begin + ei));
                ed.elt_id = g.x;
                ed.retention = __uint_as_float(g.y);
                ed.limit = __uint_as_float(g.z);
                ed.share = __uint_as_float(g.w);
            }
            return ed;
        };

        for (int64_t seg = 0; seg < n; seg += kSeg) {
            const int segn = (int)((n - seg) < kSeg ? (n - seg) : kSeg);
            for (int i = lane; i < segn; i += kWave) {
                X[i] = 0.0f;
                if (FULL) S.XH[i] = 0.0f;
            }
            uint32_t qh = 0, qt = 0;   // queue head / tail (wave-uniform)
            uint32_t hh = 0, ht = 0;   // the second queue's
            (void)hh;
            (void)ht;
            bool abandon = false;
            __syncthreads();

            auto draws_of = [&](uint32_t kl, uint32_t meta, const EltDev &ed, uint32_t *jI,
                                uint32_t *jC) {
                const uint32_t ev =
                    L.keying == ARA_KEYING_PAPER ? (uint32_t)A.ev[o0 + seg + kl] : 0u;
                draw_j(meta, L.keying, (uint32_t)(seg + kl), i_abs, ed.elt_id, L.program_id, ev,
                       keys, jI, jC);
            };

            // Drain cnt entries of the second queue from head h: the FP64
            // quantile.
            auto run_heavy = [&](uint32_t h, int cnt) {
                __syncthreads();
                if (lane < cnt) {
                    const uint2 e = S.QH[(h + lane) & kHMask];
                    const uint32_t kl = e.x, row = e.y;
                    uint32_t meta, orow;
                    float scale, cfrac;
                    if (DIAG) {
                        meta = A.row_meta[row];
                        scale = A.rowq[row].scale;
                        cfrac = A.row_cfrac[row];
                        orow = row;
                    } else {
                        const RowF F = A.rowf[row];
                        meta = F.meta;
                        scale = F.scale;
                        orow = (uint32_t)rb0 + rowf_row(F);
                        cfrac = F.cfrac;
                    }
                    const RowQ q = A.rowq[orow];
                    const EltDev ed = elt_of(meta & 0xffffu);
                    uint32_t jI, jC;
                    draws_of(kl, meta, ed, &jI, &jC);
                    double z, zc;
                    hit_z(meta, jI, jC, (double)cfrac, norm, &z, &zc);
                    // the row's pair counts serve the FP64 quantile for the rows
                    // that always take it
                    const bool f64 = (meta & ROW_F64) != 0;
                    bool ok;
                    const double x = beta_quantile64((double)q.a, (double)q.b, A.row_lnb[orow],
                                                     f64 ? meta_na(meta) : 0,
                                                     f64 ? meta_nb(meta) : 0, z, zc, A.f64_iters,
                                                     &ok);
                    if (!ok) report(A.status, ARA_E_NUMERIC, ti, seg + kl, ed.elt_id);
                    const float loss = (float)((double)scale * x);
                    atomicAdd(&S.XH[kl], ed.share * clampf_terms(loss, ed.retention, ed.limit));
                }
                __syncthreads();
            };

            // Drain cnt queue entries from head h, one hit per lane: draw,
            // invert the Beta CDF, ELT terms, accumulate into X[k].
            auto run_batch = [&](uint32_t h, int cnt) {
                __syncthreads();
                bool defer = false;
                uint2 e = make_uint2(0u, 0u);
                if (lane < cnt) {
                    e = Q[(h + lane) & kQMask];
                    const uint32_t kl = e.x, row = e.y;
                    // the row's flags: one compact record in the fast passes
                    // (row indexes the paying rows), the per-row arrays in the
                    // diagnostic pass (row indexes all rows)
                    uint32_t meta, orow, shape;
                    float scale, cfrac;
                    if (DIAG) {
                        meta = A.row_meta[row];
                        scale = A.rowq[row].scale;
                        cfrac = A.row_cfrac[row];
                        orow = row;
                        shape = A.row_shape[row];
                    } else {
                        const RowF F = A.rowf[row];
                        meta = F.meta;
                        scale = F.scale;
                        orow = (uint32_t)rb0 + rowf_row(F);
                        shape = rowf_shape(F);
                        cfrac = F.cfrac;
                    }
                    (void)orow;
                    const EltDev ed = elt_of(meta & 0xffffu);
                    float loss = 0.0f;
                    if (meta & ROW_DET) {
                        loss = scale;
                    } else if (DIAG && (scale <= ed.retention || ed.limit == 0.0f ||
                                        ed.share == 0.0f)) {
                        // a row that cannot pay (row_cannot_pay) adds exactly 0
                        // whatever it draws
                    } else if (shape) {
                        // the slot's segments; a mixed draw goes from the two
                        // normal deviates to the quantile without forming z.
                        // About 25 instructions where a Halley step and its
                        // continued fraction took 120: 12.75 -> 10.98 ms for
                        // 1.24e9 draws (1M trials, 16 ELTs), which the walk over
                        // the occurrences now sets; mixed rows, once redone
                        // whole in the second pass, 3.93 -> 0.62 ms for 40,003
                        // trials.
                        const float *tab =
                            A.shape_tab + ((size_t)l * kShapeSlots + (shape - 1u)) * kShapeStride;
                        uint32_t jI, jC;
                        draws_of(kl, meta, ed, &jI, &jC);
                        float x;
                        if (meta & ROW_CORR) {
                            const float wi = 1.0f - cfrac;
                            const float n2 = fmaf(wi, wi, cfrac * cfrac);
                            const float v = fmaf(norm_dev(norm, jI), wi,
                                                 norm_dev(norm, jC) * cfrac) * rsqrtf(n2);
                            defer = !(fabsf(v) < A.dev_band);
                            x = slot_quantile_dev(tab, v);
                        } else {
                            const uint32_t j = (meta & ROW_CONLY) ? jC : jI;
                            defer = (float)min(j, 16777216u - j) * 5.9604644775390625e-08f <
                                    A.tail_band;
                            x = slot_quantile(tab, j);
                        }
                        loss = scale * x;
                    } else if (!FULL || (meta & (ROW_F64 | ROW_CORR))) {
                        defer = true;
                    } else {
                        uint32_t jI, jC;
                        draws_of(kl, meta, ed, &jI, &jC);
                        const uint32_t j = (meta & ROW_CONLY) ? jC : jI;
                        const float z = (float)j * 5.9604644775390625e-08f;
                        const float zc = (float)(16777216u - j) * 5.9604644775390625e-08f;
                        const RowQ q = A.rowq[orow];
                        bool ok;
                        const float x = beta_quantile32(q.a, q.b, q.lnb, meta_na(meta),
                                                        meta_nb(meta), z, zc, &ok);
                        defer = !ok || fminf(z, zc) < A.tail_band;
                        loss = scale * x;
                    }
                    if (DIAG) {
                        nh += 1;
                        chk += (uint64_t)(seg + kl + 1) * 2654435761ull + (uint64_t)ed.elt_id;
                    }
                    if (!defer) {
                        const float lp = ed.share * clampf_terms(loss, ed.retention, ed.limit);
                        atomicAdd(&X[kl], lp);
                    }
                }
                if (!FULL) {
                    if (__any(defer)) abandon = true;
                } else {
                    const uint64_t m = __ballot(defer);
                    if (defer) {
                        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                        S.QH[(ht + below) & kHMask] = e;
                    }
                    ht += (uint32_t)__popcll(m);
                    if (ht - hh >= (uint32_t)kWave) {
                        run_heavy(hh, kWave);
                        hh += kWave;
                    }
                }
                __syncthreads();
            };

            // The fast pass enqueues only the rows that can pay, from the
            // per-event (first record, count) pairs; the diagnostic pass
            // visits every row so it counts every non-zero lookup.  The fast
            // pass keeps its loads one chunk ahead: the next chunk's pairs
            // and the event ids of the chunk after that are in flight while
            // this chunk's hits are drawn.
            const int32_t *evs = A.ev + o0 + seg;
            const uint2 *lpairs = reinterpret_cast<const uint2 *>(A.evoff + L.live_base);
            uint2 pr_next = make_uint2(0u, 0u);
            int32_t e_after = -1;
            if (!DIAG) {
                if (lane < segn) pr_next = lpairs[evs[lane]];
                if (kWave + lane < segn) e_after = evs[kWave + lane];
            }
            for (int c = 0; c < segn && !abandon; c += kWave) {
                const int kl = c + lane;
                const bool valid = kl < segn;
                uint32_t rb = 0, cnt = 0;
                if (DIAG) {
                    if (valid) {
                        const int32_t E = evs[kl];
                        rb = eo[E];
                        cnt = eo[E + 1] - rb;
                    }
                } else {
                    rb = pr_next.x;
                    cnt = pr_next.y;                  // zero past the segment's end
                    pr_next = e_after >= 0 ? lpairs[e_after] : make_uint2(0u, 0u);
                    e_after = (c + 2 * kWave + lane < segn) ? evs[c + 2 * kWave + lane] : -1;
                }
                uint32_t done = 0;
                while (!abandon) {
                    const int take = (int)min(cnt - done, (uint32_t)kPerLane);
                    int tot;
                    const int excl = wave_excl_scan(take, &tot);
                    for (int j = 0; j < take; ++j)
                        Q[(qt + excl + j) & kQMask] =
                            make_uint2((uint32_t)kl, (uint32_t)(rb0 + rb + done + j));
                    qt += tot;
                    done += take;
                    while (qt - qh >= (uint32_t)kWave && !abandon) {
                        run_batch(qh, kWave);
                        qh += kWave;
                    }
                    if (!__any(done < cnt)) break;
                }
            }
            if (!abandon && qt != qh) run_batch(qh, (int)(qt - qh));
            if (abandon) return true;
            if (FULL) {
                if (ht != hh) run_heavy(hh, (int)(ht - hh));
                __syncthreads();
                for (int i = lane; i < segn; i += kWave) X[i] += S.XH[i];
            }
            __syncthreads();
            for (int i = lane; i < segn; i += kWave)
                acc.add(clampf_terms(X[i], L.occ_r, L.occ_l));
            if ((DIAG || OCC) && A.occ_view) {
                const int64_t pos0 = o0 - A.off[A.trial_begin] + seg;
                for (int c = 0; c < segn; c += kWave) {
                    const int i = c + lane;
                    const bool valid = i < segn;
                    const double o = valid ? (double)clampf_terms(X[i], L.occ_r, L.occ_l) : 0.0;
                    occ_chunk<F64OUT>(o, valid, pos0 + i, l, A.occ_view, A.occ_stride, L.agg_r,
                                      L.agg_l, &occ_s, &occ_a, A.status, ti);
                }
            }
            __syncthreads();
        }

        const double total = acc.total();
        double Y;
        if (MODE == ARA_SUM_F64) Y = clampd_terms(total, (double)L.agg_r, (double)L.agg_l);
        else Y = (double)clampf_terms((float)total, L.agg_r, L.agg_l);
        if (DIAG) {
            nh = wave_sum(nh);
            chk = wave_sum(chk);
        }
        if (lane == 0) {
            if (F64OUT) {
                if (A.ylt_layers) ((double *)A.ylt_layers)[(int64_t)l * A.trial_count + t] = Y;
            } else {
                if (A.ylt_layers) ((float *)A.ylt_layers)[(int64_t)l * A.trial_count + t] = (float)Y;
            }
            if (DIAG) {
                if (A.hits) A.hits[(int64_t)l * A.trial_count + t] = nh;
                if (A.hit_chk) A.hit_chk[(int64_t)l * A.trial_count + t] = chk;
            }
        }
        if (F64OUT) pf_sum += Y;
        else pf_sum = (double)((float)pf_sum + (float)Y);
    }
    if (lane == 0 && A.ylt_pf) {
        if (F64OUT) ((double *)A.ylt_pf)[t] = pf_sum;
        else ((float *)A.ylt_pf)[t] = (float)pf_sum;
    }
    return false;
}

}  // namespace ara
