// The products of the sparse path: launch shapes of the walk (walk.h) and the sums that follow it.
#include <algorithm>
#include <cmath>

#include "walk.h"

namespace mst {

// p[0] + p[stride] + ... + p[(ntile - 1) stride], added to `sum` in that order (the order is part of the
// result); sixteen loads are in flight before the first add, a one-by-one loop waits for each.
__device__ inline float ordered_plane_sum(float sum, const float* __restrict__ p, int64_t stride, int ntile) {
    int t = 0;
    for (; t + 16 <= ntile; t += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = p[(int64_t)(t + u) * stride];
#pragma unroll
        for (int u = 0; u < 16; ++u) sum += v[u];
    }
    for (; t < ntile; ++t) sum += p[(int64_t)t * stride];
    return sum;
}

// dW[perm[e]] = sum over token tiles of partial[tile][e], tiles added in ascending order (`more`: on top of
// what earlier token ranges left there).  drive.cost null: the first view.  The blocks from reduce_blocks on add
// the nsplit partial outputs of a walk whose chunks are split over workgroups, out[k] = sum of planes[.][k],
// in ascending order: a launch costs 3 us, more than either sum takes at the batches that split.
struct PlaneSum {
    const float* planes;
    float* out;
    int64_t n;
    int nsplit;
};
__device__ inline void sum_planes_block(const PlaneSum& ps, int64_t block) {
    const int64_t k = 4 * (block * 256 + threadIdx.x);
    if (k >= ps.n) return;
    if (ps.n % 4 == 0) {
        float4 sum = *reinterpret_cast<const float4*>(ps.planes + k);
        for (int z = 1; z < ps.nsplit; ++z) {
            const float4 v = *reinterpret_cast<const float4*>(ps.planes + (int64_t)z * ps.n + k);
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        *reinterpret_cast<float4*>(ps.out + k) = sum;
        return;
    }
    for (int64_t i = k; i < std::min(ps.n, k + 4); ++i) {
        float sum = ps.planes[i];
        for (int z = 1; z < ps.nsplit; ++z) sum += ps.planes[(int64_t)z * ps.n + i];
        ps.out[i] = sum;
    }
}
__global__ __launch_bounds__(256) void k_walk_reduce(const float* __restrict__ partial, int64_t slots_stride, int ntile, int more,
                                                     const int* __restrict__ ptr_end0, const int* __restrict__ perm0,
                                                     const int* __restrict__ ptr_end1, const int* __restrict__ perm1,
                                                     const WalkDrive drive, float* __restrict__ dW, unsigned reduce_blocks,
                                                     const PlaneSum ps) {
    if (blockIdx.x >= reduce_blocks) {
        sum_planes_block(ps, (int64_t)blockIdx.x - reduce_blocks);
        return;
    }
    const bool c = drive.cost && drive_by_col(drive);
    const int64_t n = (int64_t)*(c ? ptr_end1 : ptr_end0) * (2 * OCT);
    const int* __restrict__ perm = c ? perm1 : perm0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)reduce_blocks * 256) {
        const int p = perm[e];
        if (p >= 0) dW[p] = ordered_plane_sum(more ? dW[p] : 0.f, partial + e, slots_stride, ntile);
    }
}

// The weight gradient without partial sums in memory, for a scratch area that does not hold one plane of
// them: eight threads per entry slot, every sum in the order of the walk and of k_walk_reduce.
template <typename TIn>
__global__ __launch_bounds__(256) void k_dw_slots(const TIn* __restrict__ dY, const TIn* __restrict__ X, int T, int O, int I,
                                                  const int* __restrict__ ptr_end0, const int* __restrict__ perm0,
                                                  const int* __restrict__ ptr_end1, const int* __restrict__ perm1,
                                                  const WalkDrive drive, const int* __restrict__ flat,
                                                  float* __restrict__ dW) {
    const bool c = drive_by_col(drive);
    const int64_t n = (int64_t)*(c ? ptr_end1 : ptr_end0) * (2 * OCT);
    const int* __restrict__ perm = c ? perm1 : perm0;
    const int s = threadIdx.x & 7;
    for (int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 3; e < n; e += ((int64_t)gridDim.x * 256) >> 3) {
        const int p = perm[e];
        if (p < 0) continue;                          // (the same for the eight threads of a slot)
        const int f = flat[p], o = f / I, i = f - o * I, g = (int)(e >> 1) & 7;
        float sum = 0.f;
        for (int t0 = 0; t0 < T; t0 += WT) {
            float d = 0.f;
            for (int u = 0; u < 8; ++u) {
                const int t = t0 + lane_token(s, g, u);
                const float x = t < T ? element<TIn>(X + (int64_t)t * I + i) : 0.f;
                const float y = t < T ? element<TIn>(dY + (int64_t)t * O + o) : 0.f;
                d = u == 0 ? x * y : fmaf(x, y, d);
            }
            d += __shfl_xor(d, 7, 8);
            d += __shfl_xor(d, 1, 8);
            d += __shfl_xor(d, 2, 8);
            sum += d;
        }
        if (s == 0) dW[p] = sum;
    }
}

// ---- launch shapes.  A workgroup fills a CU, so a call takes (workgroups / 256, rounded up) rounds of
// one workgroup's time: staging per chunk, the walk in proportion to the octet steps of its blocks, and
// per block the way in (DW) and out (OUT).  Microseconds, from timings of the kernels at four
// shapes and two densities on MI355X (reproduced within 10 %); a step is longest where the partial sums
// of the weight gradient are stored on the way.
struct WalkCost {
    double step, block;
};
static const WalkCost kOut = {0.0060, 1.7}, kBoth = {0.0105, 2.9}, kDw = {0.0090, 1.2};

static double octet_steps(const View& v, double density) {
    const double m = density * v.KC;                                  // entries per row and chunk
    // the longest of eight binomial rows, even.  (Rows share an octet by their lengths in the chunks, which takes 3 to 12 % off
    // that; in the time of a call it is within what the models are unsure of, and the lines drawn with them stay where they are.)
    return m + 1.42 * std::sqrt(m) + 0.5;
}
static double walk_units(const View& v, double density) { return octet_steps(v, density) * v.nchunk * v.NB; }   // see k_view_ptr
static double walk_round(const View& v, double density, int q, int chunks, const WalkCost& wc) {
    const double steps = octet_steps(v, density);
    const double stage = 1.0 + 1.5 * v.KC / KCMAX;
    const double blocks = (double)v.NB / (double)cdiv(v.NB, q);       // of a slab, on average
    return 2.0 + chunks * (stage + blocks * OPB * steps * wc.step) + blocks * wc.block;
}
static double walk_rounds(int64_t wgs) { return (double)cdiv(wgs, 256); }
static double shape_cost(const View& v, int T, double density, int q, const WalkCost& wc) {
    return walk_rounds(cdiv(T, WT) * cdiv(v.NB, q)) * walk_round(v, density, q, v.nchunk, wc);
}

static double view_density(const mst_layer* L) { return (double)L->nnz / (double)L->N; }

struct WalkShape {
    int q, nsplit;
    double cost;
};
static WalkShape pick_shape(const View& v, int T, double density, int qmax, const WalkCost& wc, int max_split) {
    const int64_t ntile = cdiv(T, WT);
    WalkShape best{1, 1, 0.0};
    for (int q = 1; q <= qmax; ++q) {
        const double cost = shape_cost(v, T, density, q, wc);
        if (q == 1 || cost < best.cost) best = WalkShape{q, 1, cost};
    }
    // Short batches leave most CUs without a workgroup and every workgroup with a chain of chunks: the
    // chunks can be split over workgroups (an entry lies in one chunk, so its weight gradient needs nothing
    // more; the outputs of the ranges are partial planes that a small kernel adds)
    for (int ns = 2; ns <= max_split; ++ns) {
        const int cps = (int)cdiv(v.nchunk, ns);
        if (cdiv(v.nchunk, cps) != ns) continue;                      // (no empty range)
        const double cost = walk_rounds(ntile * v.NB * ns) * walk_round(v, density, 1, cps, wc) + 3.0 +
                            1e-6 * (double)T * v.R * (ns + 1);
        if (cost < best.cost) best = WalkShape{1, ns, cost};
    }
    return best;
}

static int g_forced_out = 0, g_forced_both = 0;       // test hooks: row blocks per workgroup, 0 = automatic

// Every accepted pair (the names of the shapes of earlier kernels, which callers may hold) selects a number of row blocks.
// These shapes keep the chunks together and add a row's entries in the same order.
int spmm_force_shape(int tokens, int quads) {
    static const int table[][3] = {{0, 0, 0}, {128, 2, 1}, {128, 3, 2}, {128, 4, 3}, {64, 2, 1}, {64, 3, 2}, {64, 4, 4}, {64, 6, 5}, {64, 8, 6}};
    for (const auto& e : table)
        if (e[0] == tokens && e[1] == quads) {
            g_forced_out = e[2];
            return MST_OK;
        }
    return MST_ERR_ARG;
}
int bwd_fused_force_shape(int waves, int quads) {
    static const int table[][3] = {{0, 0, 0}, {16, 1, 1}, {16, 2, 2}, {8, 3, 2}, {8, 4, 3}, {8, 5, 4}};
    for (const auto& e : table)
        if (e[0] == waves && e[1] == quads) {
            g_forced_both = e[2];
            return MST_OK;
        }
    return MST_ERR_ARG;
}

// Modelled time in microseconds of a product on the sparse path (the launch shapes' costs, scaled to timings of
// whole calls at 115 shapes and densities: 8 % rms error, 12 % for the weight gradient alone).
double walk_us(const mst_layer* L, WalkJob job, int T) {
    const double d = view_density(L);
    // the sum of the planes of partial gradients: one read of each, at about 4 TB/s
    const double reduce = 4.0 + (double)cdiv(T, WT) * walk_units(L->col, d) * (OPB * OCT * 4) / 4.0e6;
    switch (job) {
        case WALK_FWD: return 0.87 * pick_shape(L->row, T, d, 6, kOut, 1).cost;
        case WALK_BWD_INPUT: return 0.87 * pick_shape(L->col, T, d, 6, kOut, 1).cost;
        case WALK_BWD_WEIGHT:
            return 0.8 * (std::min(pick_shape(L->row, T, d, 6, kDw, 1).cost, pick_shape(L->col, T, d, 6, kDw, 1).cost) + reduce) + 0.8;
        default: return 0.88 * (pick_shape(L->col, T, d, 4, kBoth, (int)std::min<int64_t>(8, L->col.nchunk)).cost + reduce);
    }
}

static WalkSide side_of(const View& v, const void* A, const void* B, int q) {
    WalkSide s;
    s.A = A;
    s.B = B;
    s.ptr = v.ptr;
    s.ent = v.ent;
    s.rowmap = v.rowmap;
    s.perm = v.perm;
    s.rowpos = v.rowpos;
    s.K = v.K;
    s.KC = v.KC;
    s.R = v.R;
    s.NBpad = v.NBpad;
    s.nchunk = v.nchunk;
    s.nslab = (int)cdiv(v.NB, q);
    return s;
}
static unsigned reduce_blocks(const mst_layer* L) { return (unsigned)std::min<int64_t>(cdiv(L->nnz * 3 / 2 + 1, 256), 8192); }

int spmm(const mst_layer* L, const View& v, const void* A, float* out, int T, mst_dtype act, hipStream_t s) {
    const int rc = ensure_fresh(L, &v == &L->row, &v == &L->col, s);
    if (rc != MST_OK) return rc;
    const int q = g_forced_out ? g_forced_out : pick_shape(v, T, view_density(L), 6, kOut, 1).q;
    const WalkSide sd = side_of(v, A, nullptr, q);
    const WalkArgs wa{out, nullptr, 0, T, (int)cdiv(T, WT), v.nchunk};
    return act == MST_F32 ? walk_out_f32(q, sd, wa, s) : walk_out_bf16(q, sd, wa, s);
}

int bwd_fused(const mst_layer* L, const void* dY, const void* X, float* dX, float* dW, int T, mst_dtype act,
              const Workspace& ws, hipStream_t s) {
    const View& v = L->col;
    int rc = ensure_fresh(L, false, true, s);
    if (rc != MST_OK) return rc;
    const int64_t planes = (int64_t)(ws.gemm_floats / ((size_t)T * v.R));
    const WalkShape sh = g_forced_both ? WalkShape{g_forced_both, 1, 0.0}
                                       : pick_shape(v, T, view_density(L), 4, kBoth, (int)std::min<int64_t>({8, v.nchunk, planes}));
    const WalkSide sd = side_of(v, dY, X, sh.q);
    const int64_t stride = v.cap_pairs * (2 * OCT);
    const int ntile = (int)cdiv(T, WT);
    const WalkArgs wa{sh.nsplit > 1 ? ws.gemm : dX, ws.partial, stride, T, ntile, (int)cdiv(v.nchunk, sh.nsplit)};
    rc = act == MST_F32 ? walk_both_f32(sh.q, sd, wa, sh.nsplit, s) : walk_both_bf16(sh.q, sd, wa, sh.nsplit, s);
    if (rc != MST_OK) return rc;
    PlaneSum ps{};
    if (sh.nsplit > 1) ps = PlaneSum{ws.gemm, dX, (int64_t)T * v.R, sh.nsplit};
    const unsigned rb = L->nnz > 0 ? reduce_blocks(L) : 0u, sb = (unsigned)cdiv(ps.n, 1024);
    if (rb + sb > 0) {
        k_walk_reduce<<<rb + sb, 256, 0, s>>>(ws.partial, stride, ntile, 0, v.ptr + v.nseg, v.perm, nullptr, nullptr, WalkDrive{}, dW, rb, ps);
        MST_LAUNCH_CHECK();
    }
    return MST_OK;
}

// The weight gradient alone.  `partial` normally holds a plane of partial sums for every token tile; a smaller
// area (the library's own, for the call without a workspace) takes the tiles in ranges, each range's
// sums added on top of those before it: the same additions in the same order.
int sddmm(const mst_layer* L, const void* dY, const void* X, float* dW, int T, mst_dtype act, float* partial,
          size_t partial_floats, hipStream_t s) {
    if (L->nnz == 0) return MST_OK;
    const View &r = L->row, &c = L->col;              // (the entries' values are not read: stale ones will do)
    const int64_t stride = std::max(r.cap_pairs, c.cap_pairs) * (2 * OCT);
    const int64_t fit = (int64_t)(partial_floats / (size_t)stride);
    // one number of blocks per workgroup for both views: the better one for the view that drives a
    // uniform pattern (heavy rows are missing from the row view).  Judged for the whole batch: the view that
    // drives decides the order of the sums, and `partial` decides the ranges.
    const double d = view_density(L);
    const WalkShape best_r = pick_shape(r, T, d, 6, kDw, 1), best_c = pick_shape(c, T, d, 6, kDw, 1);
    const int q = !L->heavy_on && best_r.cost <= best_c.cost ? best_r.q : best_c.q;
    const WalkDrive drive{L->walk_cost, (float)(shape_cost(r, T, d, q, kDw) / walk_units(r, d)),
                          (float)(shape_cost(c, T, d, q, kDw) / walk_units(c, d))};
    if (fit < 1) {
        if (act == MST_F32)
            k_dw_slots<float><<<8192, 256, 0, s>>>((const float*)dY, (const float*)X, T, L->O, L->I, r.ptr + r.nseg, r.perm,
                                                   c.ptr + c.nseg, c.perm, drive, L->flat, dW);
        else
            k_dw_slots<uint16_t><<<8192, 256, 0, s>>>((const uint16_t*)dY, (const uint16_t*)X, T, L->O, L->I, r.ptr + r.nseg, r.perm,
                                                      c.ptr + c.nseg, c.perm, drive, L->flat, dW);
        MST_LAUNCH_CHECK();
        return MST_OK;
    }
    const size_t esz = act == MST_F32 ? 4 : 2;
    int rc = MST_OK;
    for (int64_t t = 0; t < T; t += fit * WT) {
        const int n = (int)std::min<int64_t>(T - t, fit * WT), ntile = (int)cdiv(n, WT);
        const char* x = static_cast<const char*>(X) + (size_t)t * L->I * esz;
        const char* y = static_cast<const char*>(dY) + (size_t)t * L->O * esz;
        const WalkSide sr = side_of(r, x, y, q), sc = side_of(c, y, x, q);
        const WalkArgs wa{nullptr, partial, stride, n, ntile, std::max(r.nchunk, c.nchunk)};
        rc = act == MST_F32 ? walk_dw_f32(q, sr, sc, wa, drive, s) : walk_dw_bf16(q, sr, sc, wa, drive, s);
        if (rc != MST_OK) return rc;
        k_walk_reduce<<<reduce_blocks(L), 256, 0, s>>>(partial, stride, ntile, t > 0 ? 1 : 0, r.ptr + r.nseg, r.perm, c.ptr + c.nseg,
                                                       c.perm, drive, dW, reduce_blocks(L), PlaneSum{});
        MST_LAUNCH_CHECK();
    }
    return MST_OK;
}

}  // namespace mst
