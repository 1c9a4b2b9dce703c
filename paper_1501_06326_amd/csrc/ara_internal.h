// ara_internal.h -- device data layout shared by the host runtime and the
// kernels of the ARA library (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara.h"

namespace ara {

// Row metadata word: bits 0-15 ELT index in the layer, bits 16-19 flags,
// bits 20-25 / 26-31 the continued-fraction terms of the (a, b) / (b, a)
// branches of the FP32 quantile (of ROW_F64 rows: pairs of terms of the FP64 one,
// 0 where it takes as many as needed).
enum : uint32_t {
    ROW_DET = 1u << 16,    // loss = mean (sigma = 0 or secondary uncertainty off)
    ROW_F64 = 1u << 17,    // shape outside the FP32 quantile's domain: FP64 path
    ROW_CORR = 1u << 18,   // sigma_I > 0 and sigma_C > 0: mix two normals (section 3.2)
    ROW_CONLY = 1u << 19,  // sigma_I = 0, sigma_C > 0: z = u_C
    ROW_FLAGS = 0xFu << 16,
    // layer flags: a row that can pay draws and has no shape slot; such a row of the
    // FP32 quantile's domain, without a mix
    LAYER_SLOW = 1u << 31,
    LAYER_ITER = 1u << 29,
    // layer flag: no event table (an event with more paying rows than a nibble holds,
    // or more rows than a mark indexes)
    LAYER_DENSE = 1u << 30,
};
__host__ __device__ inline int meta_na(uint32_t m) { return (int)((m >> 20) & 63u); }
__host__ __device__ inline int meta_nb(uint32_t m) { return (int)((m >> 26) & 63u); }

// Per-layer record in device memory.
struct LayerDev {
    float occ_r, occ_l, agg_r, agg_l;   // layer terms (FP32; limits may be +inf)
    int32_t elt_begin;                   // first ELT (index into EltDev[])
    int32_t n_elts;
    int64_t row_base;                    // first row of the layer in the row arrays
    int64_t evoff_base;                  // first entry of the layer's ev_off[n_cat + 1]
    int64_t otab_base;                   // first entry of the layer's otab[n_cat] (PU), or -1
    uint32_t flags;                      // OR of the row flags of the layer, LAYER_SLOW
    int32_t n_rows;
    int32_t nnz;                         // non-zero entries of otab (PU)
    uint32_t program_id;                 // keys z_(Prog,E) under ARA_KEYING_PAPER
    int32_t keying;                      // ARA_KEYING_* of the portfolio
    int32_t chunk;                       // occurrences a chunk of the table form takes: 64,
                                         // or fewer so that their hits fit one segment
    int32_t n_f64;                       // paying rows without a slot, for the FP64 quantile
    int32_t n_mix;                       // paying rows of the two-normal mix with a slot
    int64_t live_base;                   // even index of the layer's (ev_off[E], rows of E
                                         // that can pay) pairs in the ev_off array
};

// Per-ELT record: id (keys the draws) and ELT financial terms.
struct EltDev {
    uint32_t elt_id;
    float retention, limit, share;
};

// Per-row secondary-uncertainty constants, event-major inside each layer:
// {max_l, alpha, beta, ln B(alpha, beta)} with ln B evaluated in FP64 at the
// FP32 alpha, beta (so the FP32 and FP64 quantiles solve the same equation).
struct RowQ {
    float scale, a, b, lnb;
};

// Compact record of a row that can pay, read by the fast passes with one
// 16-byte load: the layer's such rows are contiguous, event-major.  rs packs
// the index of the same row in the layer's per-row arrays (bits 5-31, so a
// layer holds fewer than kRowFMaxRows rows) and 1 + the slot of the row's
// Beta shape among the layer's shape tables, or 0 when it has none (bits
// 0-4); cfrac is the two-normal mix weight.  A row without a slot reads its
// Beta parameters from the per-row arrays.
struct __attribute__((aligned(16))) RowF {
    float scale;
    uint32_t meta;
    uint32_t rs;
    float cfrac;
};
constexpr int64_t kRowFMaxRows = (int64_t)1 << 27;
__host__ __device__ inline uint32_t rowf_row(const RowF &F) { return F.rs >> 5; }
__host__ __device__ inline uint32_t rowf_shape(const RowF &F) { return F.rs & 31u; }

// Raw host rows staged on the device for the build kernels.
struct RawRow {
    int32_t event;
    float mean, sigma_i, sigma_c, max_loss;
};

// The Beta fit of one raw row (build staging, indexed like the raw rows).
struct RowFit {
    RowQ q;
    uint32_t flags;
    float cfrac;
    double lnb;
};

// Context-owned device status words.
struct Status {
    int32_t code;          // 0 or an ara_status of the first failure
    int32_t pad;
    int64_t where[3];      // first failing (trial, occurrence, elt_id) or row index
};

constexpr int kWave = 64;
// Occurrences of a trial that a wavefront of the secondary-uncertainty passes holds
// in LDS at a time.
constexpr int kSeg = 512;

// Shapes the FP32 quantile covers (its error stays below ~1e-6 of the root
// there); others take the FP64 path.
constexpr float kF32MinShape = 1.0f;
constexpr float kF32MaxShape = 32.0f;

// Step limit of the FP64 quantile's bracketed iteration; a draw that has not
// converged by then is reported as ARA_E_NUMERIC.
constexpr int kF64QuantileIters = 400;

// Beta shapes shared by many rows.  Each layer has kShapeSlots slots; the
// first distinct (alpha, beta) pairs of its rows on the FP32 quantile path
// take one each.  A slot holds the quantile itself as piecewise polynomials of
// degree 7 (8 FP32 coefficients, one 32-byte segment), interpolated in FP64 at
// the Chebyshev points of each segment when the portfolio is loaded:
//  * by draw: the grid integer p = min(j, 2^24 - j) (z = j 2^-24) picks the
//    half (z <= 1/2 or above) and the octave [2^e, 2^(e+1)), its mantissa is
//    the local coordinate d = m - 1.5 in [-1/2, 1/2), both exact in FP32;
//  * by normal deviate v = Phi^-1(z) (rows of the two-normal mix, which never
//    form z): segments of width 1/2 around i / 2, |i| <= kDevHalf, with the
//    local coordinate d = 2 v - i.
// Over FP32-evaluated draws of shapes across [1, 32]^2 the error is at most
// 2.4e-7 (by draw) and 3.1e-7 (by deviate) of max(root, mean), its mean below
// 5e-10 of the mean in the emulation (seg_fit); the iteration it replaced
// peaked at 1.9e-6 and 6e-8 to 1.7e-7 in the mean of (1.5, 6) and (1, 32).  Octaves and
// half-unit steps are the widest segments that degree 7 holds to that; most
// draws fall in a few of them, so the 64 lanes of a batch touch a handful of
// cache lines (a one-segment-per-lane gather over a larger table was slower
// than the iteration).
constexpr int kShapeSlots = 16;
constexpr int kSegCoefs = 8;
constexpr int kOctaves = 23;                 // p = 1 .. 2^23 - 1
constexpr int kDevHalf = 11;
constexpr int kDevSegs = 2 * kDevHalf + 1;
constexpr float kDevMax = 5.7f;              // |v| the deviate segments serve
// A slot's segments: the octaves of the lower half, of the upper half, the deviates, each
// from a 128-byte line on, so that the octaves of seven draws in eight share a line a half.
constexpr int kSegUpper = 24, kSegDev = 48;
constexpr int kShapeStride = 72 * kSegCoefs;     // floats
// after a portfolio's slots: Phi^-1(p 2^-24) by octave of p, the same segments
constexpr int kNormFloats = kOctaves * kSegCoefs;

// Positions of a segment's hits in the lean pass' LDS (one wavefront's), and the
// bits of a position's mark that hold the layer's record index.
constexpr int kLp = 768;
constexpr int kMarkRow = 22;

// Event table of a layer (catalogues of at most kTabGroups groups): per group of
// 16 events 64 bits of paying-row counts and the group's first record, 3 words.
// kTabGroups is what the LDS of a CU holds beside the segments of 16 wavefronts
// (163,840 - 16 x 4,144 - 1,024 bytes).
constexpr int kTabGroup = 16;
constexpr int kTabGroups = 8032;
constexpr int kTabWaves = 16;
constexpr int32_t kTabWords = 3 * kTabGroups;
// Larger catalogues keep a filter there instead: a bit per 2^filter_shift events.
inline bool ev_filter(int32_t n_cat) { return (n_cat - 1) / kTabGroup >= kTabGroups; }
inline int filter_shift(int32_t n_cat) {
    int s = 0;
    while ((((int64_t)n_cat - 1) >> s) >= (int64_t)kTabWords * 32) ++s;
    return s;
}
inline size_t evtab_words(int32_t n_cat) {
    if (ev_filter(n_cat)) return (size_t)((((int64_t)n_cat - 1) >> filter_shift(n_cat)) / 32 + 1);
    return 3 * (size_t)((n_cat - 1) / kTabGroup + 1);
}

}  // namespace ara

// Host-side handle definitions (not visible to the C-ABI).
struct ara_yet {
    ara_context *ctx;
    int64_t n_trials;
    int32_t n_catalogue;
    const int64_t *d_off;
    const int32_t *d_ev;
    const float *d_times;
    int64_t n_occ;
    int64_t max_trial_len;
};

struct ara_portfolio {
    ara_context *ctx;
    int32_t n_catalogue;
    int32_t n_layers;
    int32_t n_elts;
    int64_t n_rows;
    uint64_t seed;
    int32_t su_enabled;
    int32_t max_layer_elts;
    uint32_t all_flags;
    int32_t chunk;             // the smallest of its layers' (see LayerDev)
    int64_t n_f64, n_mix;      // of its layers together (see LayerDev)
    ara::LayerDev *d_layers;
    ara::EltDev *d_elts;
    uint32_t *d_evoff;
    ara::RowQ *d_rowq;
    ara::RowF *d_rowf;
    float *d_row_mean;
    float *d_row_cfrac;
    uint32_t *d_row_meta;
    double *d_row_lnb;
    uint32_t *d_row_shape;     // per row: 1 + its shape slot, or 0
    unsigned long long *d_shape_keys;   // [layer][kShapeSlots]: (alpha, beta) bits, 0 = unused
    float *d_shape_tab;        // [layer][kShapeSlots][kShapeStride], then [kNormFloats]
    uint32_t *d_evtab;         // per layer: nibbles [2 groups], first records [groups], or the
                               // filter's bits
    float *d_otab;
    uint32_t *d_sp_bits;       // per layer [nw]: bitmap of the non-zero otab entries
    uint32_t *d_sp_rank;       // per layer [nw + 1]: set bits before each word
    float *d_sp_vals;          // per layer [n_cat]: the non-zero otab values, in event order
    void *d_workspace;
    size_t workspace_bytes;
    ara::LayerDev *h_layers;   // host copy
};

namespace ara {
// Batched run with a trial range per portfolio (ranges[2i], ranges[2i+1]),
// portfolio-major; device-side errors go to *status (null: the context's own
// status word).  Defined with the C-ABI, used by the serving loop.
ara_status run_batch_ranges(ara_context *ctx, const ara_yet *yet, int32_t n,
                            ara_portfolio *const *pfs, const ara_run_opts *opts,
                            const ara_batch_config *cfg, void *const *ylt_l, void *const *ylt_p,
                            const int64_t *ranges, void *scratch, size_t bytes, void *stream,
                            Status *status);
// Batch scratch for n portfolios whose trial ranges add up to total_trials.
size_t batch_scratch_need(int32_t n, int64_t total_trials);
}  // namespace ara

