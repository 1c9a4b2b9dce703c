// ara_pu.hip -- the analysis without secondary uncertainty: a trial is a
// gather-sum of per-event occurrence losses followed by the aggregate terms.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_device.h"

namespace ara {

// Where a layer's per-event occurrence losses are read from:
//  * LDS, dense (small catalogues) or sparse: a bit per event, the rank of each
//    32-event word and the non-zero values, for one layer or several;
//  * a bit per event in LDS and the non-zero values from the dense table in
//    global memory;
//  * the dense table in global memory.
enum { TAB_GLOBAL = 0, TAB_LDS_DENSE = 1, TAB_LDS_SPARSE = 2, TAB_LDS_BITS = 3 };

// How the occurrence view is made: not, by quads of occurrences a lane from the lookups of
// the sums, or of short trials by single ones, looked up once more.
enum { VIEW_NONE = 0, VIEW_QUADS, VIEW_SINGLES };

template <int NL>
struct PuArgs {
    const int64_t *off;
    const int32_t *ev;
    int64_t trial_begin, trial_count;
    int32_t n_cat;
    int32_t accumulate_pf;
    void *ylt_layers, *ylt_pf;
    void *occ_view;
    int64_t occ_stride;
    Status *status;
    PuTable tab[NL];
};

// The layers' tables staged by the whole block (none for TAB_GLOBAL).
template <int TAB, int NL>
__device__ __forceinline__ void pu_stage(const PuArgs<NL> &P, uint32_t *sm) {
    const int32_t nw = (P.n_cat + 31) >> 5;
    auto copy = [&](uint32_t *to, const uint32_t *from, int n) {
        for (int i = threadIdx.x; i < n; i += blockDim.x) to[i] = from[i];
    };
    if (TAB == TAB_LDS_DENSE) copy(sm, (const uint32_t *)P.tab[0].otab, P.n_cat);
    if (TAB == TAB_LDS_BITS) copy(sm, P.tab[0].bits, nw);
    if (TAB == TAB_LDS_SPARSE) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            copy(sm, P.tab[u].bits, nw);
            copy(sm + nw, P.tab[u].rank, nw + 1);
            copy(sm + 2 * nw + 1, (const uint32_t *)P.tab[u].vals, P.tab[u].nnz);
            sm += 2 * nw + 1 + P.tab[u].nnz;
        }
    }
    if (TAB != TAB_GLOBAL) __syncthreads();
}

// The occurrence loss of event E in layer T (its table at sm).
template <int TAB>
__device__ __forceinline__ float pu_look(int32_t n_cat, const PuTable &T, const uint32_t *sm,
                                         int32_t E) {
    if (TAB == TAB_LDS_DENSE) return ((const float *)sm)[E];
    if (TAB == TAB_LDS_BITS) return (sm[E >> 5] >> (E & 31)) & 1u ? T.otab[E] : 0.0f;
    if (TAB == TAB_GLOBAL) return T.otab[E];
    const int32_t nw = (n_cat + 31) >> 5;
    const uint32_t w = sm[E >> 5];
    const uint32_t m = 1u << (E & 31);
    return (w & m) ? ((const float *)(sm + 2 * nw + 1))[sm[nw + (E >> 5)] + __popc(w & (m - 1u))]
                   : 0.0f;
}

// Those of four events.
template <int TAB>
__device__ __forceinline__ float4 pu_look4(int32_t n_cat, const PuTable &T, const uint32_t *sm,
                                           int4 q) {
    if (TAB == TAB_LDS_BITS) {
        const int32_t E[4] = {q.x, q.y, q.z, q.w};
        bool on[4];
        float v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            on[c] = (sm[E[c] >> 5] >> (E[c] & 31)) & 1u;
            v[c] = 0.0f;
        }
        // lanes without a value share one line (event 0's), and the loads of a
        // wavefront with none are skipped
        if (__any(on[0] || on[1] || on[2] || on[3])) {
            float g[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) g[c] = T.otab[on[c] ? E[c] : 0];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = on[c] ? g[c] : 0.0f;
        }
        return make_float4(v[0], v[1], v[2], v[3]);
    }
    return make_float4(pu_look<TAB>(n_cat, T, sm, q.x), pu_look<TAB>(n_cat, T, sm, q.y),
                       pu_look<TAB>(n_cat, T, sm, q.z), pu_look<TAB>(n_cat, T, sm, q.w));
}

// A 16-byte load of the event-id stream, marked non-temporal: every id is read
// once, so it should not displace the cached tables (11 % faster for the
// primary-uncertainty pass, 0.76 -> 0.67 ms at the full shape).
__device__ __forceinline__ int4 ld_stream(const int4 *p) {
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const i32x4 g = __builtin_nontemporal_load(reinterpret_cast<const i32x4 *>(p));
    return make_int4(g.x, g.y, g.z, g.w);
}

// The occurrence view of four consecutive occurrences a lane, in stored order
// over the wavefront (see occ_chunk); pos the first one's place in the view.
template <bool F64OUT>
__device__ __forceinline__ void occ_quads(float4 o, bool valid, int64_t pos, const PuArgs<1> &P,
                                          const PuTable &T, double *cs, double *ca, int64_t trial) {
    const double s1 = (double)o.x, s2 = s1 + (double)o.y, s3 = s2 + (double)o.z,
                 s4 = s3 + (double)o.w;
    double s = valid ? s4 : 0.0;
    s += dpp_f64<0x111, 0xf, true>(s);    // row_shr:1
    s += dpp_f64<0x112, 0xf, true>(s);
    s += dpp_f64<0x114, 0xf, true>(s);
    s += dpp_f64<0x118, 0xf, true>(s);
    s += dpp_f64<0x142, 0xa, false>(s);   // row_bcast:15
    s += dpp_f64<0x143, 0xc, false>(s);   // row_bcast:31
    const double S = *cs + s;                          // after the lane's last
    double before = __shfl_up(S, 1, 64);
    if ((threadIdx.x & 63) == 0) before = *cs;
    const double r = (double)T.agg_r, l = (double)T.agg_l;
    const double A0 = clampd_terms(before, r, l), A1 = clampd_terms(before + s1, r, l),
                 A2 = clampd_terms(before + s2, r, l), A3 = clampd_terms(before + s3, r, l),
                 A4 = clampd_terms(S, r, l);
    if (valid) {
        const int64_t at = (int64_t)T.layer * P.occ_stride + pos;
        const double d[4] = {A1 - A0, A2 - A1, A3 - A2, A4 - A3};
        if (!F64OUT && pos + 3 < P.occ_stride && (at & 3) == 0 &&
            ((uintptr_t)P.occ_view & 15) == 0) {
            *reinterpret_cast<float4 *>((float *)P.occ_view + at) =
                make_float4((float)d[0], (float)d[1], (float)d[2], (float)d[3]);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (pos + c >= P.occ_stride) {
                    report(P.status, ARA_E_WORKSPACE_TOO_SMALL, trial, pos + c, P.occ_stride);
                    break;
                }
                if (F64OUT) ((double *)P.occ_view)[at + c] = d[c];
                else ((float *)P.occ_view)[at + c] = (float)d[c];
            }
        }
    }
    *cs = readlane_f64(S, 63);
    *ca = readlane_f64(A4, 63);
}

// One wavefront per trial (persistent grid-stride over trials), NL layers at
// once.  With the tables in LDS a block is 16 wavefronts sharing one copy, two
// blocks per CU while two copies fit, else one; with a table in global memory
// blocks are 4 wavefronts.  Event ids are streamed with 16-byte loads (after a
// scalar head that reaches 16-byte alignment), four loads in flight per lane.
// Bound, at 1M trials x 1,000 occurrences (4 GB of ids): one table of up to 78 KB
// by the id stream (671 us, 5.9 TB/s).  Tables beyond that by the LDS lookups and
// the one block per CU, which is still far ahead of a scattered load of a line
// per occurrence (300,007 trials x 1,000 occurrences, 1M events: 289 us against
// 1.60 ms).  Layers taken together read the ids once and pay for the staging
// once: 8 layers, 100,003 trials x 1,000, FP64 sums, 490 - 680 us by the draw of
// their tables, one by one 650 - 770 us, by scattered loads where a table passed
// 60 KB 1.07 - 2.20 ms.  VIEW: the layer's occurrence view is written from the same
// ids and lookups (NL = 1), quads of occurrences scanned at a time: 655 us for
// 250,000 x 1,000 where a pass of its own over single occurrences made it 970 us; of
// short trials from single occurrences (kPuViewLds), 1M x 60 0.52 ms where quads took 0.81
// and that pass 0.60.
template <int MODE, bool F64OUT, int TAB, int NL, int VIEWS>
__device__ __forceinline__ void pu_trials(const PuArgs<NL> &P) {
    constexpr bool VIEW = VIEWS == VIEW_QUADS;
    extern __shared__ uint32_t sm[];
    pu_stage<TAB, NL>(P, sm);
    const uint32_t *tabs[NL];
    tabs[0] = sm;
#pragma unroll
    for (int u = 1; u < NL; ++u)
        tabs[u] = tabs[u - 1] + 2 * ((P.n_cat + 31) >> 5) + 1 + P.tab[u - 1].nnz;
    const int lane = threadIdx.x & 63;
    // (with a view the trial and what follows from it are kept in scalar registers)
    const uint32_t w = VIEWS ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
    const int64_t wid = (int64_t)blockIdx.x * (blockDim.x / 64) + w;
    const int64_t nwv = (int64_t)gridDim.x * (blockDim.x / 64);
    const int64_t base = VIEWS ? P.off[P.trial_begin] : 0;
    for (int64_t t = wid; t < P.trial_count; t += nwv) {
        const int64_t a = P.off[P.trial_begin + t], b = P.off[P.trial_begin + t + 1];
        const int64_t n = b - a;
        Acc<MODE> acc[NL];
        double cs = 0.0, ca = 0.0;        // occurrence-view carries
        (void)cs;
        (void)ca;
        auto add1 = [&](int64_t k, int count) {     // up to 64 single occurrences from k
            const bool on = lane < count;
            const int32_t E = !VIEW || on ? P.ev[a + k + lane] : 0;
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                const float o = pu_look<TAB>(P.n_cat, P.tab[u], tabs[u], E);
                if (!VIEW || on) acc[u].add(o);
                if (VIEW)
                    occ_chunk<F64OUT>(on ? (double)o : 0.0, on, a - base + k + lane, P.tab[u].layer,
                                      P.occ_view, P.occ_stride, P.tab[u].agg_r, P.tab[u].agg_l, &cs,
                                      &ca, P.status, P.trial_begin + t);
            }
        };
        // the four losses of one 16-byte load: compensated summation adds
        // their pairwise sum (error within 2 ulp of the group, so the trial's
        // error stays a few ulp of its total whatever its length) at a
        // quarter of the per-element cost; the other modes add them one by one
        // (for a table of one layer the lookups stay inside the sums: taken
        // together first, they spill at 64 registers and lose 10 %)
        auto add4 = [&](const int4 q, bool on, int64_t k) {
            if (!VIEW && NL == 1 && TAB != TAB_LDS_BITS) {
                auto look = [&](int32_t E) { return pu_look<TAB>(P.n_cat, P.tab[0], sm, E); };
                if (MODE == ARA_SUM_KAHAN32) {
                    acc[0].add((look(q.x) + look(q.y)) + (look(q.z) + look(q.w)));
                } else {
                    acc[0].add(look(q.x)); acc[0].add(look(q.y));
                    acc[0].add(look(q.z)); acc[0].add(look(q.w));
                }
                return;
            }
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                const float4 v = pu_look4<TAB>(P.n_cat, P.tab[u], tabs[u], q);
                if (!VIEW || on) {
                    if (MODE == ARA_SUM_KAHAN32) {
                        acc[u].add((v.x + v.y) + (v.z + v.w));
                    } else {
                        acc[u].add(v.x); acc[u].add(v.y); acc[u].add(v.z); acc[u].add(v.w);
                    }
                }
                if constexpr (VIEW)
                    occ_quads<F64OUT>(v, on, a - base + k, P, P.tab[u], &cs, &ca, P.trial_begin + t);
            }
        };
        // int32 elements up to the next 16-byte boundary of the event-id stream
        int64_t head = (int64_t)(((16u - ((uint32_t)(uintptr_t)(P.ev + a) & 15u)) & 15u) >> 2);
        if (head > n) head = n;
        if (VIEW ? head > 0 : lane < head) add1(0, (int)head);
        const int4 *v4 = (const int4 *)(P.ev + a + head);
        const int64_t n4 = (n - head) >> 2;
        if (VIEW) {
            // every lane takes part in the view's scans
            for (int64_t i0 = 0; i0 < n4; i0 += 4 * 64) {
                const int64_t i = i0 + lane;
                int4 q[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    q[c] = make_int4(0, 0, 0, 0);
                    if (i + 64 * c < n4) q[c] = ld_stream(v4 + i + 64 * c);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (i0 + 64 * c < n4) add4(q[c], i + 64 * c < n4, head + 4 * (i + 64 * c));
            }
        } else {
            for (int64_t i = lane; i < n4; i += 4 * 64) {
                const bool h1 = i + 64 < n4, h2 = i + 128 < n4, h3 = i + 192 < n4;
                const int4 q0 = ld_stream(v4 + i);
                int4 q1 = make_int4(0, 0, 0, 0), q2 = q1, q3 = q1;
                if (h1) q1 = ld_stream(v4 + i + 64);
                if (h2) q2 = ld_stream(v4 + i + 128);
                if (h3) q3 = ld_stream(v4 + i + 192);
                add4(q0, true, 0);
                if (h1) add4(q1, true, 0);
                if (h2) add4(q2, true, 0);
                if (h3) add4(q3, true, 0);
            }
        }
        const int64_t done = head + 4 * n4;
        if (VIEW ? done < n : lane < n - done) add1(done, (int)(n - done));
        if constexpr (VIEWS == VIEW_SINGLES) {
            for (int64_t k = lane; k - lane < n; k += 64) {
                const bool on = k < n;
                const float o = on ? pu_look<TAB>(P.n_cat, P.tab[0], tabs[0], P.ev[a + k]) : 0.0f;
                occ_chunk<F64OUT>((double)o, on, a - base + k, P.tab[0].layer, P.occ_view, P.occ_stride,
                                  P.tab[0].agg_r, P.tab[0].agg_l, &cs, &ca, P.status,
                                  P.trial_begin + t);
            }
        }
        double sum64 = 0.0;               // the portfolio's sum, in layer order
        float sum32 = 0.0f;
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const double S = acc[u].total();
            if (lane > 0) continue;
            const PuTable &T = P.tab[u];
            double Y;
            if (MODE == ARA_SUM_F64) Y = clampd_terms(S, (double)T.agg_r, (double)T.agg_l);
            else Y = (double)clampf_terms((float)S, T.agg_r, T.agg_l);
            if (F64OUT) {
                if (P.ylt_layers) ((double *)P.ylt_layers)[(int64_t)T.layer * P.trial_count + t] = Y;
                if (P.ylt_pf) {
                    double *p = (double *)P.ylt_pf + t;
                    if (u > 0) sum64 += Y;
                    else sum64 = P.accumulate_pf ? *p + Y : Y;
                    if (u == NL - 1) *p = sum64;
                }
            } else {
                if (P.ylt_layers)
                    ((float *)P.ylt_layers)[(int64_t)T.layer * P.trial_count + t] = (float)Y;
                if (P.ylt_pf) {
                    float *p = (float *)P.ylt_pf + t;
                    if (u > 0) sum32 += (float)Y;
                    else sum32 = P.accumulate_pf ? *p + (float)Y : (float)Y;
                    if (u == NL - 1) *p = sum32;
                }
            }
        }
    }
}

// Tables in LDS: 16 wavefronts per block.
template <int MODE, bool F64OUT, int TAB, int NL, int VIEWS>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(VIEWS == VIEW_QUADS || NL > 1 ? 4 : 8, 8))) void k_ara_pu(
    PuArgs<NL> P) {
    pu_trials<MODE, F64OUT, TAB, NL, VIEWS>(P);
}

// Table in global memory: 4 wavefronts per block.
template <int MODE, bool F64OUT, int VIEWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(VIEWS == VIEW_QUADS ? 4 : 7, 7))) void k_ara_pu_global(
    PuArgs<1> P) {
    pu_trials<MODE, F64OUT, TAB_GLOBAL, 1, VIEWS>(P);
}

template <int NL>
static PuArgs<NL> pu_args(const PuLaunch &p) {
    PuArgs<NL> A;
    A.off = p.off; A.ev = p.ev; A.trial_begin = p.trial_begin; A.trial_count = p.trial_count;
    A.n_cat = p.n_cat; A.accumulate_pf = p.accumulate_pf;
    A.ylt_layers = p.ylt_layers; A.ylt_pf = p.ylt_pf;
    A.occ_view = p.occ_view; A.occ_stride = p.occ_stride; A.status = p.status;
    for (int u = 0; u < NL; ++u) A.tab[u] = p.tab[u];
    return A;
}

template <int MODE, bool F64OUT, int TAB, int NL, int VIEWS>
static hipError_t pu_lds(const PuLaunch &p, hipStream_t s) {
    const auto kernel = k_ara_pu<MODE, F64OUT, TAB, NL, VIEWS>;
    const int64_t blocks = (p.trial_count + 15) / 16;
    const int64_t cap = (int64_t)p.n_cu * (p.lds <= kPuLdsTwo ? 2 : 1);
    if (p.lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)kPuLdsOne);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks < cap ? blocks : cap)), dim3(1024), p.lds, s,
                       pu_args<NL>(p));
    return hipGetLastError();
}

template <int MODE, bool F64OUT, int VIEWS>
static hipError_t pu_dispatch(const PuLaunch &p, hipStream_t s) {
    if (p.form == PU_DENSE) return pu_lds<MODE, F64OUT, TAB_LDS_DENSE, 1, VIEWS>(p, s);
    if (p.form == PU_BITS) return pu_lds<MODE, F64OUT, TAB_LDS_BITS, 1, VIEWS ? VIEW_QUADS : VIEW_NONE>(p, s);
    if (p.form == PU_SPARSE) {
        if constexpr (VIEWS == VIEW_NONE) {
            if (p.n_layers == 2) return pu_lds<MODE, F64OUT, TAB_LDS_SPARSE, 2, VIEW_NONE>(p, s);
            if (p.n_layers == 3) return pu_lds<MODE, F64OUT, TAB_LDS_SPARSE, 3, VIEW_NONE>(p, s);
            if (p.n_layers == 4) return pu_lds<MODE, F64OUT, TAB_LDS_SPARSE, 4, VIEW_NONE>(p, s);
        }
        return pu_lds<MODE, F64OUT, TAB_LDS_SPARSE, 1, VIEWS>(p, s);
    }
    const int64_t blocks = (p.trial_count + 3) / 4, cap = (int64_t)p.n_cu * 16;
    hipLaunchKernelGGL((k_ara_pu_global<MODE, F64OUT, VIEWS>),
                       dim3((unsigned)(blocks < cap ? blocks : cap)), dim3(256), 0, s, pu_args<1>(p));
    return hipGetLastError();
}

template <int MODE, bool F64OUT>
static hipError_t pu_view(const PuLaunch &p, hipStream_t s) {
    if (!p.occ_view) return pu_dispatch<MODE, F64OUT, VIEW_NONE>(p, s);
    return p.short_trials ? pu_dispatch<MODE, F64OUT, VIEW_SINGLES>(p, s)
                          : pu_dispatch<MODE, F64OUT, VIEW_QUADS>(p, s);
}

hipError_t launch_pu(const PuLaunch &p, int mode, bool f64out, hipStream_t s) {
    if (p.trial_count <= 0) return hipSuccess;
    if (mode == ARA_SUM_NAIVE32) return f64out ? pu_view<ARA_SUM_NAIVE32, true>(p, s)
                                               : pu_view<ARA_SUM_NAIVE32, false>(p, s);
    if (mode == ARA_SUM_KAHAN32) return f64out ? pu_view<ARA_SUM_KAHAN32, true>(p, s)
                                               : pu_view<ARA_SUM_KAHAN32, false>(p, s);
    return f64out ? pu_view<ARA_SUM_F64, true>(p, s) : pu_view<ARA_SUM_F64, false>(p, s);
}

}  // namespace ara
