// ara_kernels.h -- host-side launch interface of the ARA kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_internal.h"

namespace ara {

// Events per block of the load's per-event passes (they cover n_cat + 1 offsets).
constexpr int kEvTile = 256;
inline int32_t ev_tiles(int32_t n_cat) { return (int32_t)(((int64_t)n_cat + kEvTile) / kEvTile); }

// One layer of a primary-uncertainty pass: its per-event occurrence losses, dense
// and sparse (bitmap [nw], rank [nw + 1], values [nnz]), and its aggregate terms.
struct PuTable {
    const float *otab;
    const uint32_t *bits, *rank;
    const float *vals;
    int32_t nnz;
    float agg_r, agg_l;
    int32_t layer;
};
constexpr int kPuLayers = 4;                  // layers a pass takes together
constexpr size_t kPuLdsOne = 156 * 1024;      // LDS of one block per CU
constexpr size_t kPuLdsTwo = 78 * 1024;       // of each of two
// Occurrences from which a layer whose table leaves a CU one block (or that needs the
// bitmap form) takes it: each block stages up to 156 KB first.  Catalogues of 100,000 to
// 1M events, scattered loads against LDS: 2M occurrences 14 - 19 us against 13 - 24 us (by trial
// length), 4M 22 - 25 us against 14 - 21 us, 64M 295 - 342 us against 86 - 262 us.
constexpr double kPuLargeOcc = 4e6;
// Occurrences a trial (the mean) below which the view is made from single occurrences a
// lane: quads are scanned in three pieces (head, quads, tail), single ones in pieces of
// 64.  Tables in LDS (sparse; dense alike), quads / singles: 1M trials x 8 594 / 379 us, x 60
// 768 / 524, 600,000 x 100 497 / 395, 400,000 x 150 360 / 336, 300,000 x 200 291 / 297,
// 100,000 x 600 172 / 226.  In global memory, where singles are read once more: 1M x 8
// 704 / 572, x 20 794 / 651, x 40 883 / 863, x 60 995 / 1365.  The bitmap form: 1M x 8 650 /
// 638, x 20 725 / 768, x 60 806 / 1031, quads always.
constexpr double kPuViewLds = 160.0, kPuViewGlobal = 32.0;
enum { PU_GLOBAL = 0, PU_DENSE, PU_SPARSE, PU_BITS };

struct PuLaunch {
    const int64_t *off;
    const int32_t *ev;
    int64_t trial_begin, trial_count;
    PuTable tab[kPuLayers];     // consecutive layers
    int n_layers;               // more than one: PU_SPARSE without a view
    int form;                   // PU_*: where the tables are read from
    size_t lds;                 // bytes of them in LDS
    int32_t n_cat;
    int n_cu;
    void *ylt_layers;
    void *ylt_pf;
    int32_t accumulate_pf;      // 0: ylt_pf = Y, 1: ylt_pf += Y
    bool short_trials;          // a view by single occurrences
    void *occ_view;             // optional occurrence view (see ara_run_opts)
    int64_t occ_stride;
    Status *status;
};

// The passes of a run with secondary uncertainty (ARA_PASS_*).
enum SuForm {
    SU_LEAN = ARA_PASS_LEAN,
    SU_TABLE = ARA_PASS_TABLE,
    SU_FULL = ARA_PASS_FULL,
    SU_ITER = ARA_PASS_ITERATE
};

struct SuLaunch {
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
    uint64_t seed;
    float tail_band;
    float dev_band;           // the band's normal deviate (see SuArgs)
    void *ylt_layers;
    void *ylt_pf;
    int64_t *hits;
    uint64_t *hit_chk;
    Status *status;
    int32_t *redo;            // [trial_count] scratch: flags of trials handed to the full pass
    int redo_grid;            // blocks of the full pass over the flags
    SuForm form;
    size_t lds;               // dynamic LDS of the lean pass (see su_lds)
    const LayerDev *h_layers; // host copies of the layers (the table form)
    const uint32_t *evtab;    // the layers' event tables (the table form)
    int32_t n_cat;
    int n_cu;
    int32_t f64_iters;        // step limit of the FP64 quantile
    const float *shape_tab;   // shape tables [layer][kShapeSlots][kShapeStride]
    const uint32_t *row_shape;   // per row: 1 + shape slot, or 0
    void *occ_view;           // optional occurrence view (see ara_run_opts)
    int64_t occ_stride;
};

// One portfolio of a batched run (device array of these).
struct BatchPf {
    const LayerDev *layers;
    const EltDev *elts;
    const uint32_t *evoff;
    const RowQ *rowq;
    const RowF *rowf;
    const float *row_mean;
    const float *row_cfrac;
    const uint32_t *row_meta;
    const double *row_lnb;
    const float *shape_tab;    // shape tables [layer][kShapeSlots][kShapeStride]
    void *ylt_layers;
    void *ylt_pf;
    uint32_t k0, k1;           // Philox key (the portfolio's seed)
    int32_t n_layers;
    int32_t pad;
    int64_t trial_begin, trial_count;   // the portfolio's trial range
    int64_t tile_base;                  // its first work item (trial-major off)
};

struct BatchArgs {
    const int64_t *off;
    const int32_t *ev;
    int64_t trial_begin, trial_count;
    const BatchPf *pfs;
    int32_t n_pf;
    int32_t tile;                       // trials per work item
    float tail_band;
    float dev_band;                     // the band's normal deviate
    int32_t trial_major;                // 1: one common range, items (tile, portfolio)
    int64_t n_items;                    // work items
    unsigned long long *counter;        // work-item counter
    unsigned long long *redo;           // (portfolio << 32 | trial) handed to the FP64 pass
    uint32_t *redo_count;
    Status *status;
};

hipError_t launch_validate_yet(const int64_t *off, const int32_t *ev, const float *times,
                               int64_t n_trials, int32_t n_cat, Status *st,
                               unsigned long long *max_len, hipStream_t s);
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s);
hipError_t launch_check_rows(const RawRow *raw, int64_t n, int32_t n_cat, int32_t su, Status *st,
                             hipStream_t s);
hipError_t launch_fit_rows(const RawRow *raw, int64_t n, int32_t su, RowFit *fit, hipStream_t s);
// (rank: a word per row of the portfolio; parts: two per tile of kEvTile events, of
// the layer being built)
hipError_t launch_build_layer(const RawRow *raw, const RowFit *fit, const int64_t *elt_row_off,
                              const EltDev *elts,
                              LayerDev *d_layer, const LayerDev &h_layer, int32_t n_cat, int32_t su,
                              int32_t *dat, uint32_t *evoff, uint32_t *liveoff, uint32_t *rank,
                              uint32_t *parts, RowQ *rowq, RowF *rowf, float *row_mean,
                              float *row_cfrac, uint32_t *row_meta, double *row_lnb, float *otab,
                              Status *st, hipStream_t s);
// the layer's event table (see kTabGroup) from its (first record, rows) pairs
hipError_t launch_event_table(const uint32_t *pairs, int32_t n_cat, uint32_t *tab, LayerDev *d_layer,
                              hipStream_t s);
hipError_t launch_pu(const PuLaunch &p, int mode, bool f64out, hipStream_t s);
hipError_t launch_build_sparse(const float *otab, int32_t n_cat, uint32_t *bits, uint32_t *rank,
                               float *vals, LayerDev *d_layer, hipStream_t s);
hipError_t launch_su(const SuLaunch &p, int mode, bool f64out, hipStream_t s);
// form: the pass of the batch's portfolios (not SU_TABLE); lds: see su_lds
hipError_t launch_batch(const BatchArgs &B, int mode, bool f64out, int grid, int redo_grid,
                        SuForm form, size_t lds, hipStream_t s);
hipError_t launch_debug_philox(int64_t n, const uint32_t *ctr, uint64_t key, uint32_t *out,
                               hipStream_t s);
hipError_t launch_debug_quantile(int64_t n, const float *a, const float *b, const double *z,
                                 const double *zc, float tail, const float *tab, float *x,
                                 int32_t *path, hipStream_t s);
// shape tables: the distinct shapes of one layer's paying rows into keys
// [kShapeSlots] (rows get their slot), then the tables of n_slots slots
hipError_t launch_shape_collect(RowF *rowf, const RowQ *rowq, int64_t row_base, int64_t n_rows,
                                const uint32_t *liveoff, int32_t n_cat, uint32_t *row_shape,
                                unsigned long long *keys, LayerDev *d_layer, hipStream_t s);
hipError_t launch_shape_tables(const unsigned long long *keys, int64_t n_slots, float *tab,
                               hipStream_t s);

// measurement probes (ara_probe.hip)
hipError_t launch_probe_stream(const void *src, int64_t n16, uint32_t *sink, int n_cu,
                               hipStream_t s);
hipError_t launch_probe_valu(int kind, int blocks, int32_t iters, float *out, hipStream_t s);
hipError_t launch_probe_row_consts(float a, float b, int32_t *d_out, hipStream_t s);
hipError_t launch_probe_draws(int64_t n, uint64_t seed, uint32_t elt_id, float a, float b,
                              float lnb2, int32_t na, int32_t nb, const float *tab, float *x,
                              hipStream_t s);

// PML / TVaR and the exceedance-probability curve (ara_select.hip)
size_t pml_scratch_bytes(int64_t n);
size_t ep_scratch_bytes(int64_t n, int32_t dtype);
hipError_t launch_ep_curve(const void *ylt, int32_t dtype, int64_t n, void *sorted,
                           double *tail_mean, void *scratch, hipStream_t s);
hipError_t launch_pml_tvar(const void *ylt, int32_t dtype, int64_t n, const int64_t *ks, int32_t n_rp,
                           void *scratch, double *d_out /* [2 * n_rp]: pml, tvar */, hipStream_t s);

}  // namespace ara
