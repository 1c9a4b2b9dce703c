// ara_device.h -- device helpers shared by the kernel files: status reports,
// wavefront sums and scans, the trial sum accumulators, the occurrence view.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_internal.h"
#include "ara_math.h"
#include "ara_kernels.h"

namespace ara {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ void report(Status *st, int32_t code, int64_t a, int64_t b, int64_t c) {
    if (atomicCAS(&st->code, 0, code) == 0) {
        st->where[0] = a;
        st->where[1] = b;
        st->where[2] = c;
    }
}

// A product and the terms applied to it, each rounded: every pass over the same
// hit must give the same bits, so no pass may fuse them.
__device__ __forceinline__ float mul_rn(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}
__device__ __forceinline__ float clampf_terms(float x, float r, float l) {
#pragma clang fp contract(off)
    return fminf(fmaxf(x - r, 0.0f), l);
}
__device__ __forceinline__ double clampd_terms(double x, double r, double l) {
    return fmin(fmax(x - r, 0.0), l);
}

// exclusive prefix sum of v over the 64 lanes of the wavefront (lane order)
__device__ __forceinline__ int wave_excl_scan(int v, int *total) {
    // Inclusive prefix sum over the wavefront with DPP moves: shifts within
    // each row of 16 lanes (lanes shifted in from outside the row read 0),
    // then lane 15 of rows 0 and 2 added into rows 1 and 3, then lane 31
    // added into rows 2 and 3 (the other rows keep the 0 given as old).
    int s = v;
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xf, 0xf, true);   // row_shr:1
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xf, 0xf, true);   // row_shr:2
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xf, 0xf, true);   // row_shr:4
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xf, 0xf, true);   // row_shr:8
    s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xa, 0xf, false);  // row_bcast:15
    s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xc, 0xf, false);  // row_bcast:31
    *total = __builtin_amdgcn_readlane(s, 63);
    return s - v;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// Sum accumulators for a trial's occurrence losses (ara_run_opts.sum_mode).
template <int MODE>
struct Acc;
template <>
struct Acc<ARA_SUM_NAIVE32> {
    float s = 0.0f;
    __device__ void add(float v) { s += v; }
    __device__ double total() {
        float t = s;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) t += __shfl_xor(t, d, 64);
        return (double)t;
    }
};
template <>
struct Acc<ARA_SUM_KAHAN32> {
    float s = 0.0f, c = 0.0f;   // Neumaier: exact sum = s + c (up to c's rounding)
    __device__ void add(float v) {
        const float t = s + v;
        c += (fabsf(s) >= fabsf(v)) ? ((s - t) + v) : ((v - t) + s);
        s = t;
    }
    __device__ double total() {
        float S = s, C = c;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const float So = __shfl_xor(S, d, 64), Co = __shfl_xor(C, d, 64);
            // both lanes of a pair compute the same combination (symmetric order)
            const float a = fmaxf(fabsf(S), fabsf(So)) == fabsf(S) ? S : So;
            const float b = (a == S) ? So : S;
            const float t = a + b;
            const float e = (a - t) + b;
            C = C + Co + e;
            S = t;
        }
        return (double)S + (double)C;
    }
};
template <>
struct Acc<ARA_SUM_F64> {
    double s = 0.0;
    __device__ void add(float v) { s += (double)v; }
    __device__ double total() {
        double t = s;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) t += __shfl_xor(t, d, 64);
        return t;
    }
};

// Occurrence view of 64 consecutive occurrences of one trial and layer, in
// stored order: o (lane's occurrence loss net of the occurrence terms, 0 past
// the end) is scanned into the running sum S (FP64, carried in *cs), the
// aggregate terms give A = min(max(S - AggR, 0), AggL) (carried in *ca), and
// the lane's increment A - A_prev is written at pos when valid.  Every lane
// of the wave calls this (the scan reads all of them).
// A DPP move of an FP64 value (both 32-bit halves with the same control);
// lanes that receive nothing read 0.0.
template <int CTRL, int ROWS, bool BOUND>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, BOUND);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, BOUND);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <bool F64OUT>
__device__ __forceinline__ void occ_chunk(double o, bool valid, int64_t pos, int layer,
                                          void *view, int64_t stride, float agg_r, float agg_l,
                                          double *cs, double *ca, Status *st, int64_t trial) {
    const int lane = threadIdx.x & 63;
    // inclusive FP64 prefix sum over the wavefront, laid out as in wave_excl_scan
    o += dpp_f64<0x111, 0xf, true>(o);    // row_shr:1
    o += dpp_f64<0x112, 0xf, true>(o);    // row_shr:2
    o += dpp_f64<0x114, 0xf, true>(o);    // row_shr:4
    o += dpp_f64<0x118, 0xf, true>(o);    // row_shr:8
    o += dpp_f64<0x142, 0xa, false>(o);   // row_bcast:15
    o += dpp_f64<0x143, 0xc, false>(o);   // row_bcast:31
    const double S = *cs + o;
    const double A = clampd_terms(S, (double)agg_r, (double)agg_l);
    double Ap = __shfl_up(A, 1, 64);
    if (lane == 0) Ap = *ca;
    if (valid) {
        if (pos < stride) {
            const int64_t at = (int64_t)layer * stride + pos;
            if (F64OUT) ((double *)view)[at] = A - Ap;
            else ((float *)view)[at] = (float)(A - Ap);
        } else {
            report(st, ARA_E_WORKSPACE_TOO_SMALL, trial, pos, stride);
        }
    }
    *cs = readlane_f64(S, 63);
    *ca = readlane_f64(A, 63);
}

}  // namespace ara
