// The C-ABI entry points that launch device work: argument checks on the host, then
// dispatch to the sparse kernels or, for dense layers, to the masked dense MFMA path.
#include <algorithm>
#include <mutex>

#include "common.h"

namespace mst {

// ---- scratch of the entry point that allocates nothing (mst_sparse_fc_bwd_weight_static):
// the SDDMM's per-token-tile partial sums live in this file-scope device array instead of a
// caller workspace.  Each GPU the library runs on holds its own copy at its own address until
// the process ends; host code never uses the array's name as an address, only the pointer
// hipGetSymbolAddress returns for the current device.
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static void* g_scratch_ptr[MAX_DEVICES] = {};
static std::mutex g_scratch_mutex;

// device address of `scratch` on the current device, looked up once per device
static int static_scratch(void** out) {
    int dev = -1;
    MST_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return MST_ERR_STATE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        MST_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return MST_ERR_STATE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MST_OK;
}

// out[k] = sum over the nparts partial outputs (stride apart, added in ascending order) at
// the k-th active position: the split sum of the dense gradient is only formed where the
// weight gradient is wanted.  (For a whole dense gradient, and for kernels that write no active positions alone.)
// (a thread takes four consecutive active positions: one 16-byte read of their indices, the four
// gathers of a part in flight together, one 16-byte store; flat and out are 16-byte aligned)
__global__ void k_gather_flat(const float* __restrict__ G, int64_t stride, int nparts, const int* __restrict__ flat,
                              int64_t nnz, float* __restrict__ out) {
    const int64_t k = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    if (k >= nnz) return;
    if (k + 4 <= nnz) {
        const int4 f = *reinterpret_cast<const int4*>(flat + k);
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int z = 0; z < nparts; ++z) {
            const float* g = G + (int64_t)z * stride;
            const float a = g[f.x], b = g[f.y], c = g[f.z], d = g[f.w];
            sum.x += a;
            sum.y += b;
            sum.z += c;
            sum.w += d;
        }
        *reinterpret_cast<float4*>(out + k) = sum;
        return;
    }
    for (int64_t i = k; i < nnz; ++i) {
        const float* g = G + flat[i];
        float sum = 0.f;
        for (int z = 0; z < nparts; ++z) sum += g[(int64_t)z * stride];
        out[i] = sum;
    }
}

// Y (dX) on the sparse matrix instructions where that is ahead: *done says whether it ran.  The packed weights are kept
// up while products read them (see common.h); the first product on a mask learns how even it is and may leave the work to the
// dense kernels after all.
static int pairs_product(const mst_layer* Lc, bool y, const void* A, float* C, int T, mst_dtype act, int64_t split_floats, hipStream_t s, bool* done) {
    mst_layer* L = const_cast<mst_layer*>(Lc);       // caches of vals[], not layer state
    *done = false;
    if (!L->pairs_y.blocks) return MST_OK;
    L->pairs_calls = std::min(L->pairs_calls + 1, PAIRS_CALLS);
    int tokens = pairs_tokens(L, y, act, T, split_floats, 0.0);
    if (tokens == 0) return MST_OK;
    const bool measured = L->pairs_measured;
    bool made = false;
    const int rcd = ensure_dense_copy(L, s, &made);
    if (rcd != MST_OK) return rcd;
    made &= L->pairs_recorded;                        // (then the dense copy brings them along)
    bool recording = false;
    if (!(L->pairs_valid && L->pairs_recorded && measured)) {
        const int rc = stream_recording(s, &recording);
        if (rc != MST_OK) return rc;
    }
    if (L->pairs_valid) {
        L->pairs_recorded |= recording;
        if (!recording && !L->pairs_measured) {       // (an update made them)
            const int rc = measure_pairs(L, s);
            if (rc != MST_OK) return rc;
        }
    } else if (!made) {
        // A recording makes them in every replay, and where replays of a hand-over may leave them behind every product does.  It
        // then waits for the choice of the pairs alone, once on every mask.
        if (recording || L->pairs_missed) {
            tokens = pairs_tokens(L, y, act, T, split_floats, making_pairs_us(L, recording && !L->pairs_matched));
            if (tokens == 0) return MST_OK;
        }
        const bool wait = !(L->pairs_missed && L->pairs_matched && L->pairs_measured);
        int rc = make_pairs(L, s);
        if (rc == MST_OK && wait) rc = weights_made(L, false, true, s);
        if (rc != MST_OK) return rc;
    }
    if (!measured && L->pairs_measured) {
        const double making_us = L->pairs_missed ? making_pairs_us(L, false) : 0.0;
        tokens = pairs_tokens(L, y, act, T, split_floats, making_us);
        if (tokens == 0) {
            L->pairs_unread = mst_layer::PAIRS_UNREAD;
            return MST_OK;
        }
    }
    L->pairs_unread = 0;
    *done = true;
    gemm_note_tile(24);
    return gemm_pairs(A, act, y ? L->pairs_y : L->pairs_x, C, T, tokens, s);
}

// What a dense product reads besides the activations, for Y (dX): the dense copy, and the weights' planes where the product takes
// those.  They are kept up (sync_values and updates make them), or are made now: with the dense copy if a product has read
// them before, else by themselves (see weights_made; where replays may leave them behind every product makes them and none
// waits: two that meet write the same bits).
static int ensure_weights(const mst_layer* Lc, bool y, mst_dtype act, int M, int N, int Kdim, bool full, const uint16_t*& planes, hipStream_t s) {
    mst_layer* L = const_cast<mst_layer*>(Lc);       // caches of vals[], not layer state
    bool made = false;
    int rc = ensure_dense_copy(L, s, &made);
    made &= L->planes_kept();                         // (a recording that makes them does not say that they are there)
    planes = nullptr;
    if (rc != MST_OK || !gemm_wants_planes(act, M, N, Kdim, full)) return rc;
    planes = y ? L->planes_y : L->planes_x;
    if (L->planes_valid || made) return MST_OK;
    L->planes_used = true;
    rc = make_planes(L, s);
    return rc == MST_OK && !L->planes_missed ? weights_made(L, true, false, s) : rc;
}

// (full: see full_precision(); split_ws: room for partial outputs of a split of the contraction range, used where the output
// has too few tiles to fill the chip; null: one workgroup per tile whatever their number)
int dense_products_fwd(const mst_layer* L, const void* X, float* Y, int T, mst_dtype act, hipStream_t s, bool full) {
    bool done = false;
    int rc = full ? MST_OK : pairs_product(L, true, X, Y, T, act, 0, s, &done);
    if (rc != MST_OK || done) return rc;
    const uint16_t* planes;
    rc = ensure_weights(L, true, act, T, L->O, L->I, full, planes, s);
    if (rc != MST_OK) return rc;
    return gemm_mfma(GEMM_NT, X, act, L->Wd, MST_F32, planes, Y, T, L->O, L->I, nullptr, 0, s, full);
}

int dense_products_bwd_input(const mst_layer* L, const void* dY, float* dX, int T, mst_dtype act, hipStream_t s, bool full,
                             float* split_ws, int64_t split_ws_floats) {
    bool done = false;
    int rc = full ? MST_OK : pairs_product(L, false, dY, dX, T, act, split_ws ? split_ws_floats : 0, s, &done);
    if (rc != MST_OK || done) return rc;
    const uint16_t* planes;
    rc = ensure_weights(L, false, act, T, L->I, L->O, full, planes, s);
    if (rc != MST_OK) return rc;
    return gemm_mfma(GEMM_NN, dY, act, L->Wd, MST_F32, planes, dX, T, L->I, L->O, split_ws, split_ws_floats, s, full);
}

int dense_products_bwd_weight(const mst_layer* L, const void* dY, const void* X, float* dW, int T,
                              mst_dtype act, const Workspace& ws, hipStream_t s, bool full) {
    int nparts = 1;
    ActiveOut active{L, dW};
    int rc = gemm_mfma(GEMM_TN, dY, act, X, act, nullptr, ws.G, L->O, L->I, T, ws.gemm, (int64_t)ws.gemm_floats, s, full, &nparts, &active);
    if (rc != MST_OK) return rc;
    if (active.done) return nparts > 1 ? sum_split_planes(ws.gemm, active.stride, nparts, dW, L->nnz, s) : MST_OK;
    if (L->nnz > 0) {
        k_gather_flat<<<(unsigned)cdiv(L->nnz, 1024), 256, 0, s>>>(nparts > 1 ? ws.gemm : ws.G, L->N, nparts, L->flat,
                                                                  L->nnz, dW);
        MST_LAUNCH_CHECK();
    }
    return MST_OK;
}

static bool act_ok(mst_dtype a) { return a == MST_F32 || a == MST_BF16; }

// remembered for the next update's decision whether the index views will be walked
static void note_call(const mst_layer* L, mst_dtype act, int T) {
    mst_layer* m = const_cast<mst_layer*>(L);
    m->hint_T = T;
    m->hint_act = (int)act;
}

}  // namespace mst

using namespace mst;

extern "C" {

int mst_spmm_force_shape(int tokens_per_workgroup, int quads_per_wavefront) {
    return spmm_force_shape(tokens_per_workgroup, quads_per_wavefront);
}

int mst_gemm_force_fp32_mfma(int on) { return gemm_force_fp32_mfma(on); }

int mst_gemm_last_tile(void) { return gemm_last_tile(); }

int mst_heavy_rows(int on) { return heavy_rows_enable(on); }

int mst_bwd_force_shape(int wavefronts_per_workgroup, int quads_per_wavefront) {
    return bwd_fused_force_shape(wavefronts_per_workgroup, quads_per_wavefront);
}

int mst_sparse_fc_fwd(const mst_layer_t* L, const void* X_dev, float* Y_dev, int T, mst_dtype act,
                      mst_stream_t stream) {
    if (!L || !X_dev || !Y_dev || T < 1 || !act_ok(act) || !aligned16(X_dev) || !aligned16(Y_dev)) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    hipStream_t s = (hipStream_t)stream;
    note_call(L, act, T);
    // (unbuilt views and no workspace to build them with: the dense product, same result within tolerance)
    bool views;
    int rc = views_there(L, s, &views);
    if (rc != MST_OK) return rc;
    if (use_dense_path(L, WALK_FWD, act, T) || !views)
        return dense_products_fwd(L, X_dev, Y_dev, T, act, s, full_precision(L, WALK_FWD, act, T));
    rc = spmm(L, L->row, X_dev, Y_dev, T, act, s);
    if (rc != MST_OK || !L->heavy_on) return rc;
    return heavy_fwd(L, X_dev, Y_dev, T, act, s);        // the rows the view leaves out (returns at once without any)
}

int mst_sparse_fc_bwd_input(const mst_layer_t* L, const void* dY_dev, float* dX_dev, int T, mst_dtype act,
                            mst_stream_t stream) {
    if (!L || !dY_dev || !dX_dev || T < 1 || !act_ok(act) || !aligned16(dY_dev) || !aligned16(dX_dev)) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    hipStream_t s = (hipStream_t)stream;
    note_call(L, act, T);
    bool views;
    const int rc = views_there(L, s, &views);
    if (rc != MST_OK) return rc;
    if (use_dense_path(L, WALK_BWD_INPUT, act, T) || !views)
        return dense_products_bwd_input(L, dY_dev, dX_dev, T, act, s, full_precision(L, WALK_BWD_INPUT, act, T));
    return spmm(L, L->col, dY_dev, dX_dev, T, act, s);
}

int mst_sparse_fc_bwd_weight(const mst_layer_t* L, const void* dY_dev, const void* X_dev, float* dW_dev, int T,
                             mst_dtype act, void* ws_dev, size_t ws_bytes, mst_stream_t stream) {
    if (!L || !dY_dev || !X_dev || !dW_dev || !ws_dev || T < 1 || !act_ok(act)) return MST_ERR_ARG;
    if (!aligned16(dY_dev) || !aligned16(X_dev) || !aligned16(dW_dev) || !aligned16(ws_dev)) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    const Workspace ws = carve_workspace(ws_dev, L->O, L->I, L->cap, T);
    if (ws_bytes < ws.total) return MST_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    note_call(L, act, T);
    if (use_dense_weight_grad(L, act, T))
        return dense_products_bwd_weight(L, dY_dev, X_dev, dW_dev, T, act, ws, s, full_precision(L, WALK_BWD_WEIGHT, act, T));
    const int rc = ensure_views(L, ws, s);
    if (rc != MST_OK) return rc;
    return sddmm(L, dY_dev, X_dev, dW_dev, T, act, ws.partial, ws.partial_floats, s);
}

size_t mst_static_scratch_bytes(void) { return STATIC_SCRATCH_BYTES; }

int mst_sparse_fc_bwd_weight_static(const mst_layer_t* L, const void* dY_dev, const void* X_dev, float* dW_dev, int T,
                                    mst_dtype act, mst_stream_t stream) {
    if (!L || !dY_dev || !X_dev || !dW_dev || T < 1 || !act_ok(act)) return MST_ERR_ARG;
    if (!aligned16(dY_dev) || !aligned16(X_dev) || !aligned16(dW_dev)) return MST_ERR_ARG;
    if (!L->built || !L->views_valid) return MST_ERR_STATE;      // (it has no workspace to build unbuilt views with)
    // the documented limit: ceil(T / 128) planes of 8 floats per pair of four-row slices of 128 indices at the
    // layer's capacity.  (The planes of the walk are other ones; a batch that needs more of them than the
    // array holds is taken in ranges of tokens.)
    auto plane = [&](int K, int R) {
        const int64_t quads = cdiv(K, 128) * cdiv(R, 16) * 4;
        return cdiv((L->cap + quads) / 2 + 1 + 16, 8) * 8 * 8;
    };
    const size_t need = (size_t)cdiv(T, 128) * (size_t)std::max(plane(L->I, L->O), plane(L->O, L->I)) * sizeof(float);
    if (need > STATIC_SCRATCH_BYTES) return MST_ERR_WORKSPACE;
    void* base = nullptr;
    const int rc = static_scratch(&base);
    if (rc != MST_OK) return rc;
    // (every slot the second kernel reads is written by the first)
    return sddmm(L, dY_dev, X_dev, dW_dev, T, act, static_cast<float*>(base), STATIC_SCRATCH_BYTES / sizeof(float),
                 (hipStream_t)stream);
}

int mst_sparse_fc_bwd(const mst_layer_t* L, const void* dY_dev, const void* X_dev, float* dX_dev, float* dW_dev,
                      int T, mst_dtype act, void* ws_dev, size_t ws_bytes, mst_stream_t stream) {
    if (!L || !dY_dev || !X_dev || !dX_dev || !dW_dev || !ws_dev || T < 1 || !act_ok(act)) return MST_ERR_ARG;
    if (!aligned16(dY_dev) || !aligned16(X_dev) || !aligned16(dX_dev) || !aligned16(dW_dev) || !aligned16(ws_dev))
        return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    const Workspace ws = carve_workspace(ws_dev, L->O, L->I, L->cap, T);
    if (ws_bytes < ws.total) return MST_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    note_call(L, act, T);
    if (use_fused_backward(L, act, T)) {
        const int rcv = ensure_views(L, ws, s);
        if (rcv != MST_OK) return rcv;
        return bwd_fused(L, dY_dev, X_dev, dX_dev, dW_dev, T, act, ws, s);
    }
    // the dense weight gradient (the split area of the workspace serves a dense dX first, then the weight
    // gradient: same stream)
    const bool full = full_precision(L, WALK_BWD, act, T);
    int rc;
    if (use_sparse_input_grad(L, act, T)) {
        rc = ensure_views(L, ws, s);
        if (rc == MST_OK) rc = spmm(L, L->col, dY_dev, dX_dev, T, act, s);
    } else {
        rc = dense_products_bwd_input(L, dY_dev, dX_dev, T, act, s, full, ws.gemm, (int64_t)ws.gemm_floats);
    }
    if (rc != MST_OK) return rc;
    return dense_products_bwd_weight(L, dY_dev, X_dev, dW_dev, T, act, ws, s, full);
}

int mst_layer_uses_dense(const mst_layer_t* L, mst_dtype act, int T, int weight_gradient) {
    if (!L || !act_ok(act) || T < 1) return MST_ERR_ARG;
    // Y and dX have no workspace to build unbuilt views with: they then run dense whatever the density
    if (weight_gradient == 2) return use_fused_backward(L, act, T) ? 0 : 1;
    if (weight_gradient == 0 || weight_gradient == 3)
        return use_dense_path(L, weight_gradient == 0 ? WALK_FWD : WALK_BWD_INPUT, act, T) || !L->views_valid || L->views_pending ? 1 : 0;
    return use_dense_weight_grad(L, act, T) ? 1 : 0;
}

int mst_gather_active(const mst_layer_t* L, const float* G_dev, float* dW_dev, mst_stream_t stream) {
    if (!L || !G_dev || !dW_dev || !aligned16(G_dev) || !aligned16(dW_dev)) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    if (L->nnz > 0) {
        k_gather_flat<<<(unsigned)cdiv(L->nnz, 1024), 256, 0, (hipStream_t)stream>>>(G_dev, L->N, 1, L->flat, L->nnz, dW_dev);
        MST_LAUNCH_CHECK();
    }
    return MST_OK;
}

int mst_layer_format_stats(const mst_layer_t* L, mst_format_stats* out, mst_stream_t stream) {
    if (!L || !out) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    hipStream_t s = (hipStream_t)stream;
    if (!L->views_valid) {                            // unbuilt (layer on the dense contractions): nothing stored
        out->nnz = L->nnz;
        out->row_view_slots = out->col_view_slots = 0;
        out->row_view_efficiency = out->col_view_efficiency = 0.0;
        out->heavy_rows = out->heavy_entries = 0;
        return MST_OK;
    }
    int pr = 0, pc = 0, hv[2] = {0, 0};
    MST_HIP(hipMemcpyAsync(&pr, L->row.ptr + L->row.nseg, 4, hipMemcpyDeviceToHost, s));
    MST_HIP(hipMemcpyAsync(&pc, L->col.ptr + L->col.nseg, 4, hipMemcpyDeviceToHost, s));
    if (L->heavy_on) {
        MST_HIP(hipMemcpyAsync(&hv[0], L->heavy, 4, hipMemcpyDeviceToHost, s));
        MST_HIP(hipMemcpyAsync(&hv[1], L->heavy + HEAVY_MAX + 1, 4, hipMemcpyDeviceToHost, s));
    }
    MST_HIP(hipStreamSynchronize(s));
    out->nnz = L->nnz;
    out->heavy_rows = hv[0];
    out->heavy_entries = hv[1];
    out->row_view_slots = (int64_t)pr * (2 * OCT);
    out->col_view_slots = (int64_t)pc * (2 * OCT);
    out->row_view_efficiency = pr ? (double)(L->nnz - hv[1]) / (double)out->row_view_slots : 1.0;
    out->col_view_efficiency = pc ? (double)L->nnz / (double)out->col_view_slots : 1.0;
    return MST_OK;
}

int mst_dense_grad(const void* dY_dev, const void* X_dev, float* G_dev, int T, int O, int I, mst_dtype act,
                   void* ws_dev, size_t ws_bytes, mst_stream_t stream) {
    if (!dY_dev || !X_dev || !G_dev || T < 1 || O < 1 || I < 1 || !act_ok(act)) return MST_ERR_ARG;
    if (!aligned16(dY_dev) || !aligned16(X_dev) || !aligned16(G_dev) || (ws_dev && !aligned16(ws_dev))) return MST_ERR_ARG;
    return gemm_mfma(GEMM_TN, dY_dev, act, X_dev, act, nullptr, G_dev, O, I, T, (float*)ws_dev,
                     ws_dev ? (int64_t)(ws_bytes / 4) : 0, (hipStream_t)stream);
}

// the dense gradient scores gradient growth and, with a prune score that has a gradient
// term, pruning; an update that does neither does not need it
static bool needs_gradient(const mst_layer* L, const mst_update_stats& st) {
    return st.n_grad > 0 || (L->prune_lambda != 0.f && st.n_prune > 0);
}

static int update_common(mst_layer_t* L, const float* G, uint64_t seed, const Workspace& ws,
                         mst_update_stats* stats_out, hipStream_t s, const mst_update_stats& st) {
    if (stats_out) *stats_out = st;
    if (st.n_prune == 0 && st.n_grow == 0) return MST_OK;     // nothing moves
    const UpdateItem item{L, G, st, seed, ws};
    return mask_update_device(&item, 1, s);
}

int mst_mask_update_from_scores(mst_layer_t* L, const float* G_dev, double target_density, double zeta,
                                double rand_ratio, uint64_t rng_seed, void* ws_dev, size_t ws_bytes,
                                mst_update_stats* stats_out, mst_stream_t stream) {
    if (!L || !G_dev || !ws_dev || !aligned16(G_dev) || !aligned16(ws_dev)) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    mst_update_stats st;
    int rc = mst_update_counts(L->N, L->nnz, target_density, zeta, rand_ratio, &st);
    if (rc != MST_OK) return rc;
    if (st.nnz_after > L->cap) return MST_ERR_STATE;
    const Workspace ws = carve_workspace(ws_dev, L->O, L->I, L->cap, 1);
    if (ws_bytes < ws.total) return MST_ERR_WORKSPACE;
    return update_common(L, G_dev, rng_seed, ws, stats_out, (hipStream_t)stream, st);
}

int mst_mask_update_from_scores_multi(int n_layers, mst_layer_t* const* layers, const float* const* G_dev,
                                      const double* target_density, double zeta, double rand_ratio,
                                      const uint64_t* rng_seed, void* const* ws_dev, const size_t* ws_bytes,
                                      mst_update_stats* stats_out, const mst_stream_t* streams) {
    if (n_layers < 0 || (n_layers > 0 && (!layers || !G_dev || !target_density || !rng_seed || !ws_dev || !ws_bytes || !streams)))
        return MST_ERR_ARG;
    // everything that can be refused is refused before the first launch
    for (int j = 0; j < n_layers; ++j) {
        mst_layer_t* L = layers[j];
        if (!L || !G_dev[j] || !ws_dev[j] || !aligned16(G_dev[j]) || !aligned16(ws_dev[j])) return MST_ERR_ARG;
        for (int u = 0; u < j; ++u)
            if (layers[u] == L || ws_dev[u] == ws_dev[j] || G_dev[u] == G_dev[j]) return MST_ERR_ARG;
        if (!L->built) return MST_ERR_STATE;
        mst_update_stats st;
        const int rc = mst_update_counts(L->N, L->nnz, target_density[j], zeta, rand_ratio, &st);
        if (rc != MST_OK) return rc;
        if (st.nnz_after > L->cap) return MST_ERR_STATE;
        if (ws_bytes[j] < carve_workspace(nullptr, L->O, L->I, L->cap, 1).total) return MST_ERR_WORKSPACE;
    }
    // One chain of launches per stream, for all its layers.  (One for all layers, with events between the streams, is slower: a
    // hipStreamWaitEvent costs the host 14 us and the GPU as much, the chains of four layers side by side 77 launches of 4 us.)
    for (int j0 = 0; j0 < n_layers; ++j0) {
        bool first = true;
        for (int u = 0; u < j0; ++u) first = first && streams[u] != streams[j0];
        if (!first) continue;
        UpdateItem items[BATCH_MAX];
        int n = 0;
        for (int j = j0; j < n_layers; ++j) {
            if (streams[j] == streams[j0]) {
                mst_update_stats st;
                int rc = mst_update_counts(layers[j]->N, layers[j]->nnz, target_density[j], zeta, rand_ratio, &st);
                if (rc != MST_OK) return rc;
                if (stats_out) stats_out[j] = st;
                if (st.n_prune > 0 || st.n_grow > 0)                 // (otherwise nothing moves)
                    items[n++] = UpdateItem{layers[j], G_dev[j], st, rng_seed[j], carve_workspace(ws_dev[j], layers[j]->O, layers[j]->I, layers[j]->cap, 1)};
            }
            if (n == BATCH_MAX || (n > 0 && j == n_layers - 1)) {
                const int rc = mask_update_device(items, n, (hipStream_t)streams[j0]);
                if (rc != MST_OK) return rc;
                n = 0;
            }
        }
    }
    return MST_OK;
}

int mst_mask_update(mst_layer_t* L, const void* dY_dev, const void* X_dev, int T, mst_dtype act,
                    double target_density, double zeta, double rand_ratio, uint64_t rng_seed, void* ws_dev,
                    size_t ws_bytes, mst_update_stats* stats_out, mst_stream_t stream) {
    if (!L || !dY_dev || !X_dev || !ws_dev || T < 1 || !act_ok(act)) return MST_ERR_ARG;
    if (!aligned16(dY_dev) || !aligned16(X_dev) || !aligned16(ws_dev)) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    mst_update_stats st;
    int rc = mst_update_counts(L->N, L->nnz, target_density, zeta, rand_ratio, &st);
    if (rc != MST_OK) return rc;
    if (st.nnz_after > L->cap) return MST_ERR_STATE;
    const Workspace ws = carve_workspace(ws_dev, L->O, L->I, L->cap, 1);
    if (ws_bytes < ws.total) return MST_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    note_call(L, act, T);
    if (needs_gradient(L, st)) {
        rc = gemm_mfma(GEMM_TN, dY_dev, act, X_dev, act, nullptr, ws.G, L->O, L->I, T, ws.gemm, (int64_t)ws.gemm_floats, s);
        if (rc != MST_OK) return rc;
    }
    return update_common(L, ws.G, rng_seed, ws, stats_out, s, st);
}

int mst_sparse_fc_bwd_weight_update(mst_layer_t* L, const void* dY_dev, const void* X_dev, float* dW_dev, int T,
                                    mst_dtype act, double target_density, double zeta, double rand_ratio,
                                    uint64_t rng_seed, void* ws_dev, size_t ws_bytes, mst_update_stats* stats_out,
                                    mst_stream_t stream) {
    if (!L || !dY_dev || !X_dev || !dW_dev || !ws_dev || T < 1 || !act_ok(act)) return MST_ERR_ARG;
    if (!aligned16(dY_dev) || !aligned16(X_dev) || !aligned16(dW_dev) || !aligned16(ws_dev)) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    mst_update_stats st;
    int rc = mst_update_counts(L->N, L->nnz, target_density, zeta, rand_ratio, &st);
    if (rc != MST_OK) return rc;
    if (st.nnz_after > L->cap) return MST_ERR_STATE;
    const Workspace ws = carve_workspace(ws_dev, L->O, L->I, L->cap, T);
    if (ws_bytes < ws.total) return MST_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    note_call(L, act, T);
    if (needs_gradient(L, st)) {
        // one dense gradient serves both: the weight gradient is read from it at the positions
        // that are active now, then the update scores growth with it
        rc = gemm_mfma(GEMM_TN, dY_dev, act, X_dev, act, nullptr, ws.G, L->O, L->I, T, ws.gemm, (int64_t)ws.gemm_floats, s);
        if (rc != MST_OK) return rc;
        if (L->nnz > 0) {
            k_gather_flat<<<(unsigned)cdiv(L->nnz, 1024), 256, 0, s>>>(ws.G, L->N, 1, L->flat, L->nnz, dW_dev);
            MST_LAUNCH_CHECK();
        }
    } else {
        if (use_dense_weight_grad(L, act, T)) {
            rc = dense_products_bwd_weight(L, dY_dev, X_dev, dW_dev, T, act, ws, s, full_precision(L, WALK_BWD_WEIGHT, act, T));
        } else {
            rc = ensure_views(L, ws, s);
            if (rc == MST_OK) rc = sddmm(L, dY_dev, X_dev, dW_dev, T, act, ws.partial, ws.partial_floats, s);
        }
        if (rc != MST_OK) return rc;
    }
    return update_common(L, ws.G, rng_seed, ws, stats_out, s, st);
}

}  // extern "C"
