// Launchers of the walk kernels for one activation type, one translation unit each (walk_f32.hip,
// walk_bf16.hip: the instances compile side by side).
#pragma once
#include <algorithm>

#include "walk.h"

namespace mst {

template <typename TIn, int Q, bool OUT, bool DW>
__global__ __launch_bounds__(WALK_NT) void k_walk(const WalkParams wp) {
    extern __shared__ __attribute__((aligned(16))) char walk_lds[];
    walk_body<TIn, Q, OUT, DW>(wp.sd, wp.wa, walk_lds);
}

// The weight gradient alone: either view can drive it, decided on the device (WalkDrive).  The grid covers the larger of the two.
template <typename TIn, int Q>
__global__ __launch_bounds__(WALK_NT) void k_walk_dw(const WalkSide row, const WalkSide col, const WalkArgs wa,
                                                     const WalkDrive drive) {
    extern __shared__ __attribute__((aligned(16))) char walk_lds[];
    const bool c = drive_by_col(drive);
    WalkSide sd;                                      // field by field: the arguments stay in scalar registers
    sd.A = c ? col.A : row.A;
    sd.B = c ? col.B : row.B;
    sd.ptr = c ? col.ptr : row.ptr;
    sd.ent = c ? col.ent : row.ent;
    sd.rowmap = c ? col.rowmap : row.rowmap;
    sd.perm = sd.rowpos = nullptr;                    // (no outputs of this kind)
    sd.K = c ? col.K : row.K;
    sd.KC = c ? col.KC : row.KC;
    sd.R = c ? col.R : row.R;
    sd.NBpad = c ? col.NBpad : row.NBpad;
    sd.nchunk = c ? col.nchunk : row.nchunk;
    sd.nslab = c ? col.nslab : row.nslab;
    walk_body<TIn, Q, false, true>(sd, wa, walk_lds);
}

inline unsigned walk_lds_bytes(int KC, int areas) { return (unsigned)std::max(KC * WT * 4, areas * STAGE_BYTES); }
inline unsigned walk_grid(int ntile, int nslab) { return 8u * (unsigned)cdiv((int64_t)ntile * nslab, 8); }

template <typename TIn, int Q, bool OUT, bool DW>
static int launch_q(const WalkSide& sd, const WalkArgs& wa, int nsplit, hipStream_t s) {
    static_assert(Q <= MAX_WG_BLOCKS, "the last slab reads the pointers of this many blocks");
    static uint64_t done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(&k_walk<TIn, Q, OUT, DW>), KCMAX * WT * 4, done);
    if (rc != MST_OK) return rc;
    k_walk<TIn, Q, OUT, DW><<<dim3(walk_grid(wa.ntile, sd.nslab), (unsigned)nsplit), WALK_NT, walk_lds_bytes(sd.KC, DW ? std::max(2, walk_areas(Q)) : 2), s>>>(WalkParams{sd, wa});
    MST_LAUNCH_CHECK();
    return MST_OK;
}

template <typename TIn>
static int launch_out_any(int q, const WalkSide& sd, const WalkArgs& wa, hipStream_t s) {
    switch (q) {
        case 1: return launch_q<TIn, 1, true, false>(sd, wa, 1, s);
        case 2: return launch_q<TIn, 2, true, false>(sd, wa, 1, s);
        case 3: return launch_q<TIn, 3, true, false>(sd, wa, 1, s);
        case 4: return launch_q<TIn, 4, true, false>(sd, wa, 1, s);
        case 5: return launch_q<TIn, 5, true, false>(sd, wa, 1, s);
        default: return launch_q<TIn, 6, true, false>(sd, wa, 1, s);
    }
}

template <typename TIn>
static int launch_both_any(int q, const WalkSide& sd, const WalkArgs& wa, int nsplit, hipStream_t s) {
    switch (q) {
        case 1: return launch_q<TIn, 1, true, true>(sd, wa, nsplit, s);
        case 2: return launch_q<TIn, 2, true, true>(sd, wa, nsplit, s);
        case 3: return launch_q<TIn, 3, true, true>(sd, wa, nsplit, s);
        default: return launch_q<TIn, 4, true, true>(sd, wa, nsplit, s);
    }
}

template <typename TIn, int Q>
static int launch_dw_q(const WalkSide& row, const WalkSide& col, const WalkArgs& wa, const WalkDrive& drive, hipStream_t s) {
    static_assert(Q <= MAX_WG_BLOCKS, "the last slab reads the pointers of this many blocks");
    static uint64_t done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(&k_walk_dw<TIn, Q>), KCMAX * WT * 4, done);
    if (rc != MST_OK) return rc;
    k_walk_dw<TIn, Q><<<walk_grid(wa.ntile, std::max(row.nslab, col.nslab)), WALK_NT, walk_lds_bytes(std::max(row.KC, col.KC), walk_areas(Q)), s>>>(
        row, col, wa, drive);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

template <typename TIn>
static int launch_dw_any(int q, const WalkSide& row, const WalkSide& col, const WalkArgs& wa, const WalkDrive& drive, hipStream_t s) {
    switch (q) {
        case 1: return launch_dw_q<TIn, 1>(row, col, wa, drive, s);
        case 2: return launch_dw_q<TIn, 2>(row, col, wa, drive, s);
        case 3: return launch_dw_q<TIn, 3>(row, col, wa, drive, s);
        case 4: return launch_dw_q<TIn, 4>(row, col, wa, drive, s);
        case 5: return launch_dw_q<TIn, 5>(row, col, wa, drive, s);
        default: return launch_dw_q<TIn, 6>(row, col, wa, drive, s);
    }
}

}  // namespace mst
