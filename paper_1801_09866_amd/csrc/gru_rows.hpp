// The GRU launch's rows: the work lists of all its frames, back to back.
#pragma once

#include "common.hpp"

namespace rn {

struct RowSrc {
    const void *x;      // start of this row's x part (fp32, or bf16 embedding)
    const float *h;     // start of this row's h part
    bool x_bf16;
    bool valid;
};

// The GRU rows of all the launch's frames back to back: entry e's rows are
// [moff[e], moff[e+1]), and their work lists live in its session's scratch
// (sofs[e] bytes after session 0's).
struct Rows {
    int n;
    int moff[kMaxSessions + 1];
    int sess[kMaxSessions];   // relative to the launch's Dev
    long long sofs[kMaxSessions];
};

// sessions of the launch's frames (the GRU needs no other frame argument)
struct SessList {
    int n;
    int sess[kMaxSessions];
};

// The planner's GRU row count of each of the launch's frames, issued as the
// kernel's first loads (entries past the frame count load frame 0's and are
// not used), so that waiting for them waits for nothing issued later.
struct RowCounts {
    long long c[kMaxSessions];
};

__device__ __forceinline__ RowCounts load_row_counts(const Dev &d, const SessList &sl) {
    RowCounts rc;
#pragma unroll
    for (int e = 0; e < kMaxSessions; ++e) {
        const int ee = e < sl.n ? e : 0;
        rc.c[e] = ldg<long long>(shift_ptr(d.ctr, (long long)sl.sess[ee] * d.sess_stride) + C_FRAME_M);
    }
    return rc;
}

__device__ __forceinline__ Rows make_rows(const Dev &d, const SessList &sl, const RowCounts &rc) {
    Rows R;
    R.n = sl.n;
#pragma unroll
    for (int e = 0; e < kMaxSessions; ++e) {
        R.sess[e] = sl.sess[e < sl.n ? e : 0];
        R.sofs[e] = (long long)R.sess[e] * d.sess_stride;
    }
    R.moff[0] = 0;
#pragma unroll
    for (int e = 0; e < kMaxSessions; ++e)
        R.moff[e + 1] = R.moff[e] + (e < sl.n ? __builtin_amdgcn_readfirstlane((int)rc.c[e]) : 0);
    return R;
}

// element `m` (a row of the whole launch) of a per-session work-list array
template <class T>
__device__ __forceinline__ T row_at(const Rows &R, T *arr, int m) {
    if (R.n == 1) return shift_ptr(arr, R.sofs[0])[m];   // one frame (a scalar branch)
    long long o = R.sofs[0];
    int base = 0;
#pragma unroll
    for (int e = 1; e < kMaxSessions; ++e)   // unrolled selects: no indexed private arrays
        if (e < R.n && m >= R.moff[e]) {
            o = R.sofs[e];
            base = R.moff[e];
        }
    return shift_ptr(arr, o)[m - base];
}

__device__ __forceinline__ RowSrc row_source(const Dev &d, const Rows &R, int layer, int m, int M) {
    RowSrc r;
    r.valid = m < M;
    r.x_bf16 = false;
    r.x = nullptr;
    r.h = nullptr;
    if (!r.valid) return r;
    r.h = reinterpret_cast<const float *>(row_at(R, d.f_rowh, m)) + (size_t)layer * d.H;
    if (layer == 0) {
        const int w = row_at(R, d.f_roww, m);
        if (d.wdtype == RNNLM_BF16) {
            r.x = reinterpret_cast<const uint16_t *>(d.emb) + (size_t)w * d.E;
            r.x_bf16 = true;
        } else {
            r.x = reinterpret_cast<const float *>(d.emb) + (size_t)w * d.E;
        }
    } else {
        r.x = reinterpret_cast<const float *>(row_at(R, d.f_rowdst, m)) + (size_t)(layer - 1) * d.H;
    }
    return r;
}

// start of row m of a per-session per-row array of `stride` elements
template <class T>
__device__ __forceinline__ T *row_ptr(const Rows &R, T *arr, int m, size_t stride) {
    long long o = R.sofs[0];
    int base = 0;
    if (R.n > 1) {   // uniform
#pragma unroll
        for (int e = 1; e < kMaxSessions; ++e)
            if (e < R.n && m >= R.moff[e]) {
                o = R.sofs[e];
                base = R.moff[e];
            }
    }
    return shift_ptr(arr, o) + (size_t)(m - base) * stride;
}

// session of row m of the whole launch (absolute), for the packed rows, which
// lie outside the sessions' strided state
__device__ __forceinline__ int row_session(const Dev &d, const Rows &R, int m) {
    int s = R.sess[0];
#pragma unroll
    for (int e = 1; e < kMaxSessions; ++e)
        if (e < R.n && m >= R.moff[e]) s = R.sess[e];
    return d.sess0 + s;
}

}  // namespace rn
