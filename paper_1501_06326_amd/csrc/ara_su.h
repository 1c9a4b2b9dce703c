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
// LDS per wavefront: X[kSeg] floats + Q[kQCap] pairs + El[kEltLds] records =
// 5 KB, so LDS allows the 32 waves per CU that the lean pass's registers do
// (1M trials, 16 ELTs: 9.92 ms at 8 per SIMD, 10.04 ms at 7).  With the FP32 iteration
// 6: at 7 it spills 8 registers (65,536 trials x 1,000 occurrences, one row in 10,000
// iterated: 0.61 against 0.67 ms; all: 1.50 and 1.51), with a view or diagnostics 7 (at 8 up
// to 14: 20,000 x 200 over 2 layers of 250,000 events 104 against 128 us with a view).
constexpr int kQCap = 256;        // hit queue (power of two)
#define ARA_SU_OCCUPANCY(N) __attribute__((amdgpu_waves_per_eu(N, N)))
#define ARA_FULL_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4, 4)))
// A layer's ELT records are staged in LDS when it has at most this many ELTs
// (1 KB per wavefront, within the occupancy above); the draw then
// needs one global load (the row) before its Philox key is known.
constexpr int kEltLds = 64;
constexpr int kQMask = kQCap - 1;
// The full pass's own LDS: the occurrence sums of hits from its second queue
// and that queue (a light batch adds at most 64 entries to fewer than 64).
constexpr int kHCap = 128;
constexpr int kHMask = kHCap - 1;

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
    int32_t *redo;            // a flag for each trial of the run: handed to the full pass
    uint32_t redo_step;       // flags a block of the full pass reads at a time (at most a
                              // lane each); 0: it runs every trial
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

// The normal deviate of a mixed draw (section 3.2): the two uniforms' deviates,
// mixed, without forming z.
__device__ __forceinline__ float mixed_deviate(const float *norm, uint32_t jI, uint32_t jC,
                                               float cfrac) {
    const float wi = 1.0f - cfrac;
    const float n2 = fmaf(wi, wi, mul_rn(cfrac, cfrac));
    return mul_rn(fmaf(norm_dev(norm, jI), wi, mul_rn(norm_dev(norm, jC), cfrac)), rsqrtf(n2));
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

// X[k] += v for the lanes with a hit, k non-descending over the lanes: the sum of
// each occurrence's hits in lane order, as 64 LDS float atomics would give it
// bit for bit.  Those take 190 LDS cycles per batch (3 a lane, measured), which
// kept the LDS busy two thirds of the time; here each lane takes its left
// neighbour's sum when its turn in the occurrence comes (dist), at three
// vector instructions per hit of the longest occurrence (10.9 -> 10.0 ms for 1M
// trials x 16 ELTs).  Only the first occurrence of a batch can hold a sum already.
__device__ __forceinline__ void seq_add(float *X, uint32_t k, float v, bool hit, int lane) {
    // lanes without a hit lie behind the last hit: a run of their own
    const int key = hit ? (int)k : -1;
    const int left = __builtin_amdgcn_update_dpp(-2, key, 0x138, 0xf, 0xf, false);    // wave_shr:1
    const uint64_t heads = __ballot(left != key);
    const uint64_t upto = heads & (~0ull >> (63 - lane));
    const int dist = lane - (63 - __builtin_clzll(upto));
    const int right = __builtin_amdgcn_update_dpp(-2, key, 0x130, 0xf, 0xf, false);   // wave_shl:1
    float s = v;
    if (lane == 0 && hit) s += X[k];
    for (int d = 1; __any(hit && dist >= d); ++d) {
        const float t = __int_as_float(
            __builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x138, 0xf, 0xf, true));
        s = dist == d ? t + v : s;
    }
    if (hit && right != key) X[k] = s;
}

// LDS traffic of one wavefront is in order; only the compiler must not move it.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A layer's event table (kTabGroup events a group): the paying rows of each
// event as a nibble, and the first record of the group.
struct EvTab {
    static constexpr bool kInLds = true;
    const uint2 *nib;
    const uint32_t *base;
};

// (first record, rows) of event E; 16 events are 64 bits of nibbles, and the
// rows before E in its group are a masked dot product with ones.
__device__ __forceinline__ uint2 tab_pair(const EvTab &T, int32_t E) {
    const int g = E >> 4, sh = 4 * (E & 15);
    const uint2 w = T.nib[g];
    const uint64_t W = ((uint64_t)w.y << 32) | w.x, m = W & ((1ull << sh) - 1ull);
    uint32_t r = T.base[g];
    r = __builtin_amdgcn_udot8((uint32_t)m, 0x11111111u, r, false);
    r = __builtin_amdgcn_udot8((uint32_t)(m >> 32), 0x11111111u, r, false);
    return make_uint2(r, (uint32_t)(W >> sh) & 15u);
}

// A layer's event filter, of catalogues too large for the table: a bit per 2^shift
// events says whether any has rows; only those look up their pair in memory.
struct EvFilter {
    static constexpr bool kInLds = false;
    const uint32_t *bits;
    const uint2 *pairs;
    int shift;
};
__device__ __forceinline__ uint2 tab_pair(const EvFilter &T, int32_t E) {
    const uint32_t b = (uint32_t)E >> T.shift;
    uint2 r = make_uint2(0u, 0u);
    if ((T.bits[b >> 5] >> (b & 31u)) & 1u) r = T.pairs[E];
    return r;
}

// The lean pass' LDS of one wavefront: positions of a segment's hits, and where
// each occurrence's begin.
constexpr int kSumChunks = 4;
constexpr int kLpPad = 8;         // reads past an occurrence's last hit, added as 0
struct LeanLds {
    float *LP;       // [kLp + kLpPad] mark of a first position, then the hit's loss
    uint16_t *ST;    // [kSeg + 8] first position of each occurrence
    EltDev *El;      // [kEltLds]
};

// LDS of one wavefront.
struct SuLds {
    float *X;        // [kSeg] occurrence sums
    uint2 *Q;        // [kQCap] hit queue: (occurrence in the segment, row)
    EltDev *El;      // [kEltLds]
    float *XH;       // full pass: [kSeg] sums of the second queue's hits
    uint2 *QH;       // full pass: [kHCap]
};

// One trial of one layer (Algorithm 1 inside the layer loop).
//
// ROWS = SU_LEAN is the lean pass: rows without a draw and rows whose shape has
// a slot; SU_ITER also iterates the FP32 quantile of shapes without one.  Any other
// hit, and a draw in the caller's tail band, abandons the trial, which is then handed
// to the full pass.  Returns true when abandoned.
//
// ROWS = SU_FULL takes every row.  What a light batch cannot finish in FP32
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
template <int MODE, bool F64OUT, bool DIAG, int ROWS, bool OCC>
__device__ __forceinline__ bool su_layer(const SuArgs &A, const PhiloxKeys &keys, const LayerDev &L,
                                         int l, int64_t t, int64_t o0, int64_t n, const SuLds &S,
                                         double *Y_out) {
    constexpr bool FULL = ROWS == SU_FULL;
    float *X = S.X;
    uint2 *Q = S.Q;
    EltDev *El = S.El;
    const int lane = threadIdx.x & 63;
    const int64_t ti = A.trial_begin + t;
    const uint32_t i_abs = (uint32_t)ti;
    const float *norm = A.shape_tab + (size_t)A.n_layers * kShapeSlots * kShapeStride;
    const uint32_t *eo = A.evoff + L.evoff_base;
    const int64_t rb0 = L.row_base;
    const bool elt_lds = L.n_elts <= kEltLds;
    if (elt_lds) {
        wave_sync();
        for (int i = lane; i < L.n_elts; i += kWave) El[i] = A.elts[L.elt_begin + i];
        wave_sync();
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
        wave_sync();

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
            wave_sync();
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
            wave_sync();
        };

        // Drain cnt queue entries from head h, one hit per lane: draw,
        // invert the Beta CDF, ELT terms, accumulate into X[k].
        auto run_batch = [&](uint32_t h, int cnt) {
            wave_sync();
            bool defer = false;
            uint2 e = make_uint2(0u, 0u);
            float lp = 0.0f;
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
                    // whole in a pass of their own, 3.93 -> 0.62 ms for 40,003
                    // trials.
                    const float *tab =
                        A.shape_tab + ((size_t)l * kShapeSlots + (shape - 1u)) * kShapeStride;
                    uint32_t jI, jC;
                    draws_of(kl, meta, ed, &jI, &jC);
                    float x;
                    if (meta & ROW_CORR) {
                        const float v = mixed_deviate(norm, jI, jC, cfrac);
                        defer = !(fabsf(v) < A.dev_band);
                        x = slot_quantile_dev(tab, v);
                    } else {
                        const uint32_t j = (meta & ROW_CONLY) ? jC : jI;
                        defer = (float)min(j, 16777216u - j) * 5.9604644775390625e-08f <
                                A.tail_band;
                        x = slot_quantile(tab, j);
                    }
                    loss = mul_rn(scale, x);
                } else if (ROWS == SU_LEAN || (meta & (ROW_F64 | ROW_CORR))) {
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
                    loss = mul_rn(scale, x);
                }
                if (DIAG) {
                    nh += 1;
                    chk += (uint64_t)(seg + kl + 1) * 2654435761ull + (uint64_t)ed.elt_id;
                }
                if (!defer) lp = ed.share * clampf_terms(loss, ed.retention, ed.limit);
            }
            seq_add(X, e.x, lp, lane < cnt, lane);
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
            wave_sync();
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
            // append the chunk's hits in (occurrence, row) order, as many as
            // the queue takes beside the fewer than 64 left in it (the whole
            // chunk unless its events hold more than three rows each on average)
            int tot;
            const int excl = wave_excl_scan((int)cnt, &tot);
            for (int w0 = 0; w0 < tot && !abandon; w0 += (kQCap - kWave)) {
                const int w1 = min(tot, w0 + (kQCap - kWave));
                const int j1 = min((int)cnt, w1 - excl);
                for (int j = max(0, w0 - excl); j < j1; ++j)
                    Q[(qt + (uint32_t)(excl + j - w0)) & kQMask] =
                        make_uint2((uint32_t)kl, (uint32_t)(rb0 + rb + j));
                qt += (uint32_t)(w1 - w0);
                while (qt - qh >= (uint32_t)kWave && !abandon) {
                    run_batch(qh, kWave);
                    qh += kWave;
                }
            }
        }
        if (!abandon && qt != qh) run_batch(qh, (int)(qt - qh));
        if (abandon) return true;
        if (FULL) {
            if (ht != hh) run_heavy(hh, (int)(ht - hh));
            wave_sync();
            for (int i = lane; i < segn; i += kWave) X[i] += S.XH[i];
        }
        wave_sync();
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
        wave_sync();
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
    *Y_out = Y;
    return false;
}

// The ELT record of a row: an LDS read when the layer's records are staged
// (the global read is a different instruction, so the two are not merged into
// one flat load).
__device__ __forceinline__ EltDev elt_record(const EltDev *El, bool staged, const EltDev *elts,
                                             uint32_t ei) {
    if (staged) return El[ei];
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 g = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(elts + ei));
    return {g.x, __uint_as_float(g.y), __uint_as_float(g.z), __uint_as_float(g.w)};
}

// Lane i receives the value of lane src (any lane of the wavefront).
__device__ __forceinline__ uint32_t lane_get(uint32_t v, int src) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)v);
}

// The event ids of the kChunks chunks of cw occurrences from k on, of a trial of
// n at evs: a lane each, -1 past its end.
constexpr int kChunks = kSeg / kWave;
struct SegIds {
    int32_t e[kChunks];
};
__device__ __forceinline__ void load_ids(SegIds &I, const int32_t *evs, int64_t k, int64_t n, int cw) {
    const int lane = threadIdx.x & 63;
    const int left = (int)min((int64_t)(kChunks * cw), n - k);
    const int32_t *p = evs + k;
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
        I.e[c] = lane < min(cw, left - c * cw) ? p[c * cw + lane] : -1;
}

// One trial of one layer, the lean pass: rows without a draw and slotted rows.
//
// A segment is up to kChunks chunks of L.chunk occurrences (one a lane; so many
// that the hits of any chunk fit kLp) whose hits fit kLp.
//  * Their hits take consecutive positions, in (occurrence, row) order, by a scan
//    of their counts; only each occurrence's first position is marked (LP:
//    occurrence + 1 and first record).
//  * The positions are drawn 64 at a time in a pipeline of three turns (start:
//    a lane finds its occurrence as the last mark up to its position, the highest
//    bit of a ballot up to its own, and loads its record; draw; finish), and
//    each hit's loss net of the ELT terms is left at its position.
//  * Each lane adds up the hits of its occurrences in order, and the trial's sum takes
//    them in the order in which su_layer does: occurrence k is lane k mod 64's, also
//    where a segment begins at another multiple of L.chunk.
// I holds the ids of the trial's first segment; the next segment's, and at the
// end those of the next trial (evs_next, n_next), are loaded before the sums,
// which wait for nothing but LDS.  Ids loaded a chunk ahead inside the turns
// were waited for by the next turn's record: loads return in order, and the wait
// counts merge at the loop.
template <int MODE, bool F64OUT, bool OCC, typename TAB>
__device__ __forceinline__ bool su_layer_tab(const SuArgs &A, const PhiloxKeys &keys,
                                             const LayerDev &L, int l, int64_t t, int64_t o0,
                                             int64_t n, SegIds &I, const int32_t *evs_next,
                                             int64_t n_next, const LeanLds &S, const TAB &T,
                                             double *Y_out) {
    float *LP = S.LP;
    uint32_t *MK = reinterpret_cast<uint32_t *>(S.LP);
    const int lane = threadIdx.x & 63;
    const int64_t ti = A.trial_begin + t;
    const uint32_t i_abs = (uint32_t)ti;
    const float *slots = A.shape_tab + (size_t)l * kShapeSlots * kShapeStride;
    const RowF *rows = A.rowf + L.row_base;
    const bool elt_lds = L.n_elts <= kEltLds;
    const int cw = L.chunk;
    const bool check_tail = A.tail_band > 5.9604644775390625e-08f;
    Acc<MODE> acc;
    double occ_s = 0.0, occ_a = 0.0;      // occurrence-view carries
    (void)occ_s;
    (void)occ_a;

    const int32_t *evs = A.ev + o0;
    const uint64_t upto = ~0ull >> (63 - lane);
    // occurrence keying and independent draws only: the usual rows
    const bool plain = L.keying == ARA_KEYING_OCCURRENCE && !(L.flags & ROW_CONLY);

    // the pipeline's registers: the batch whose records are on the way (n_start
    // hits, from position p_start) and the one whose segments are
    RowF F;
    uint32_t kl = 0, p_start = 0, p_draw = 0;
    int n_start = 0, n_draw = 0;
    float4 lo, hi;
    float d, scale, ret, lim, share;
    bool det = false;

    for (int64_t seg = 0; seg < n;) {
        bool abandon = false;
        wave_sync();
        for (int i = lane; i < kLp / 4; i += kWave)
            reinterpret_cast<uint4 *>(MK)[i] = make_uint4(0u, 0u, 0u, 0u);
        wave_sync();
        uint32_t hh = 0, ht = 0;           // positions started, placed (wave-uniform)
        uint32_t c_mark = 0, c_pos = 0;    // last mark started and its position

        // One turn of the pipeline: cnt new positions from hh start (their
        // records are loaded), the batch started in the turn before draws (its
        // polynomial segments are loaded), the one drawn before that is
        // finished.  Each load has a turn's arithmetic to arrive in.
        auto turn = [&](int cnt) {
            wave_sync();
            // start: the mark at the position
            const uint32_t p = hh + (uint32_t)lane;
            const bool hit = lane < cnt;
            const uint32_t mk = hit ? MK[p] : 0u;
            // finish
            if (n_draw > 0) {
                float x = fmaf(hi.w, d, hi.z);
                x = fmaf(x, d, hi.y);
                x = fmaf(x, d, hi.x);
                x = fmaf(x, d, lo.w);
                x = fmaf(x, d, lo.z);
                x = fmaf(x, d, lo.y);
                x = fmaf(x, d, lo.x);
                const float loss = det ? scale : mul_rn(scale, x);
                const float lp = share * clampf_terms(loss, ret, lim);
                if (lane < n_draw) LP[p_draw + (uint32_t)lane] = lp;
            }
            // start: its occurrence's mark, the last one up to it
            const uint64_t marks = __ballot(mk != 0u), mine = marks & upto;
            const int own = 63 - __builtin_clzll(mine | 1ull);
            const uint32_t got = lane_get(mk, own);
            // draw
            n_draw = n_start;
            if (n_start > 0) {
                p_draw = p_start;
                const EltDev ed = elt_record(S.El, elt_lds, A.elts + L.elt_begin, F.meta & 0xffffu);
                const bool on = lane < n_start;
                const uint32_t k = (uint32_t)seg + kl;
                det = (F.meta & ROW_DET) != 0;
                scale = F.scale;
                ret = ed.retention;
                lim = ed.limit;
                share = ed.share;
                uint32_t at = (uint32_t)max((int)rowf_shape(F) - 1, 0) * (uint32_t)kShapeStride;
                // (a draw in the tail band abandons the trial; no draw is in the default one)
                auto tail = [&](uint32_t j) {
                    if (__any(grid_tail(j) < A.tail_band && on && !det)) abandon = true;
                };
                if (plain) {
                    const uint32_t j =
                        u24(philox10_x0(make_uint4(k, i_abs, ed.elt_id, 0u), keys));
                    at += slot_segment(j, &d);
                    if (check_tail) tail(j);
                } else {
                    const uint32_t ev = L.keying == ARA_KEYING_PAPER && on ? (uint32_t)evs[k] : 0u;
                    uint32_t jI, jC;
                    draw_j(F.meta, L.keying, k, i_abs, ed.elt_id, L.program_id, ev, keys, &jI, &jC);
                    const uint32_t j = max(max(jI, jC), 1u);     // a row without a mix draws one
                    at += slot_segment(j, &d);
                    if (check_tail) tail(j);
                }
                lo = *reinterpret_cast<const float4 *>(slots + at);
                hi = *reinterpret_cast<const float4 *>(slots + at + 4);
            }
            // start: its record
            n_start = cnt;
            if (cnt > 0) {
                p_start = hh;
                const uint32_t mark = mine ? got : c_mark;
                const uint32_t step = mine ? (uint32_t)(lane - own) : p - c_pos;
                if (marks) {
                    const int last = 63 - __builtin_clzll(marks);
                    c_mark = (uint32_t)__builtin_amdgcn_readlane((int)mk, last);
                    c_pos = hh + (uint32_t)last;
                }
                kl = (mark >> kMarkRow) - 1u;
                F = rows[hit ? (mark & ((1u << kMarkRow) - 1u)) + step : 0u];
                hh += (uint32_t)cnt;
            }
        };

        const int room = (int)min((int64_t)(kChunks * cw), n - seg);
        int taken = 0;                     // occurrences of the segment
        uint2 pr[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            pr[c] = I.e[c] < 0 ? make_uint2(0u, 0u) : tab_pair(T, I.e[c]);
        // counts from LDS are scanned three chunks at a time, ten bits each (at most 15 rows
        // an event; 8.06 -> 7.95 ms for 1M trials x 16 ELTs); those from memory as they arrive
        // (496 us for 100,000 trials x 1,000 over 1M events, three at a time; 463 one by one)
        uint32_t before[(kChunks + 2) / 3];
        int tots[(kChunks + 2) / 3];
        if (TAB::kInLds) {
#pragma unroll
            for (int g = 0; g < (kChunks + 2) / 3; ++g) {
                uint32_t v = pr[3 * g].y;
                if (3 * g + 1 < kChunks) v |= pr[3 * g + 1].y << 10;
                if (3 * g + 2 < kChunks) v |= pr[3 * g + 2].y << 20;
                before[g] = (uint32_t)wave_excl_scan((int)v, &tots[g]);
            }
        }
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            if (taken != c * cw || taken >= room) continue;
            uint32_t excl, tot;
            if (TAB::kInLds) {
                excl = (before[c / 3] >> (10 * (c % 3))) & 1023u;
                tot = ((uint32_t)tots[c / 3] >> (10 * (c % 3))) & 1023u;
            } else {
                int n_c;
                excl = (uint32_t)wave_excl_scan((int)pr[c].y, &n_c);
                tot = (uint32_t)n_c;
            }
            if (ht + tot > (uint32_t)kLp) continue;
            const uint32_t start = ht + excl;
            if (lane < cw) S.ST[taken + lane] = (uint16_t)start;
            if (pr[c].y) MK[start] = ((uint32_t)(taken + lane + 1) << kMarkRow) | pr[c].x;
            ht += tot;
            taken += cw;
        }
        taken = min(taken, room);
        while (ht - hh >= 64u && !abandon) turn(kWave);
        while ((hh != ht || n_start + n_draw > 0) && !abandon) turn((int)(ht - hh));
        // (a chunk always fits an empty segment: L.chunk sees to it)
        if (abandon || taken == 0) return true;
        if (lane == 0) S.ST[taken] = (uint16_t)ht;
        wave_sync();
        if (seg + taken < n) load_ids(I, evs, seg + taken, n, cw);
        else load_ids(I, evs_next, 0, n_next, cw);
        const int64_t pos0 = OCC ? o0 - A.off[A.trial_begin] + seg : 0;
        // the lane of the segment's first occurrence (the view has segments of whole chunks of 64)
        const int lane0 = OCC ? 0 : (int)(seg & 63);
        // kSumChunks occurrences a lane at a time, four hits of each in flight
        // (an occurrence's hits are added in order whatever the grouping)
        for (int c = -lane0; c < taken; c += kSumChunks * kWave) {
            float x[kSumChunks];
            const float *q[kSumChunks];
            int cnt[kSumChunks], most = 0;
#pragma unroll
            for (int u = 0; u < kSumChunks; ++u) {
                // (before the first occurrence, as past the last: no hits)
                const uint32_t i = (uint32_t)(c + u * kWave + lane), end = (uint32_t)taken;
                const int s0 = S.ST[min(i, end)], s1 = S.ST[min(i + 1u, end)];
                q[u] = LP + s0;
                cnt[u] = s1 - s0;
                most = max(most, cnt[u]);
            }
#pragma unroll
            for (int u = 0; u < kSumChunks; ++u) {
                const float v0 = q[u][0], v1 = q[u][1], v2 = q[u][2], v3 = q[u][3];
                x[u] = 0 < cnt[u] ? v0 : 0.0f;       // (a loss is never -0)
                x[u] += 1 < cnt[u] ? v1 : 0.0f;
                x[u] += 2 < cnt[u] ? v2 : 0.0f;
                x[u] += 3 < cnt[u] ? v3 : 0.0f;
            }
            for (int j = 4; __any(j < most); j += 2) {
#pragma unroll
                for (int u = 0; u < kSumChunks; ++u) {
                    q[u] += j < cnt[u] ? (j == 4 ? 4 : 2) : 0;
                    const float v0 = q[u][0], v1 = q[u][1];
                    x[u] += j < cnt[u] ? v0 : 0.0f;
                    x[u] += j + 1 < cnt[u] ? v1 : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < kSumChunks; ++u) {
                const int i = c + u * kWave + lane;
                const bool valid = (uint32_t)i < (uint32_t)taken;
                const float o = clampf_terms(x[u], L.occ_r, L.occ_l);
                if (valid) acc.add(o);
                if (OCC && A.occ_view && c + u * kWave < taken)
                    occ_chunk<F64OUT>(valid ? (double)o : 0.0, valid, pos0 + i, l, A.occ_view,
                                      A.occ_stride, L.agg_r, L.agg_l, &occ_s, &occ_a, A.status, ti);
            }
        }
        seg += taken;
    }

    const double total = acc.total();
    double Y;
    if (MODE == ARA_SUM_F64) Y = clampd_terms(total, (double)L.agg_r, (double)L.agg_l);
    else Y = (double)clampf_terms((float)total, L.agg_r, L.agg_l);
    if (lane == 0 && A.ylt_layers) {
        if (F64OUT) ((double *)A.ylt_layers)[(int64_t)l * A.trial_count + t] = Y;
        else ((float *)A.ylt_layers)[(int64_t)l * A.trial_count + t] = (float)Y;
    }
    *Y_out = Y;
    return false;
}

// All layers of one trial, one wavefront.
template <int MODE, bool F64OUT, bool DIAG, int ROWS, bool OCC = false>
__device__ __forceinline__ bool su_trial(const SuArgs &A, const PhiloxKeys &keys, int64_t t,
                                         const SuLds &S) {
    const int64_t o0 = A.off[A.trial_begin + t];
    const int64_t n = A.off[A.trial_begin + t + 1] - o0;
    double pf_sum = 0.0;
    for (int l = 0; l < A.n_layers; ++l) {
        const LayerDev L = A.layers[l];
        double Y;
        if (su_layer<MODE, F64OUT, DIAG, ROWS, OCC>(A, keys, L, l, t, o0, n, S, &Y))
            return true;
        if (F64OUT) pf_sum += Y;
        else pf_sum = (double)((float)pf_sum + (float)Y);
    }
    if ((threadIdx.x & 63) == 0 && A.ylt_pf) {
        if (F64OUT) ((double *)A.ylt_pf)[t] = pf_sum;
        else ((float *)A.ylt_pf)[t] = (float)pf_sum;
    }
    return false;
}

}  // namespace ara
