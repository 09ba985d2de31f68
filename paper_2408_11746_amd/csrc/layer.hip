// Layer object, storage format and its construction on the device.
//
// Storage (not prescribed by the paper, which only names the binary mask M of
// Sec. 3.2): the active weights are kept once in canonical order (ascending flat
// index o*I + i) as vals[] / flat[], plus two "views" that the product kernels walk:
//   row view  S = W    [O x I]  -> forward
//   col view  S = W^T  [I x O]  -> input gradient
// (the weight gradient walks whichever of the two is cheaper, see build_views).
// A view cuts the contraction index into chunks and stores, per (chunk, block of 128 rows,
// octet), an ELL slice of eight rows (see View in common.h).  perm[] maps an
// entry slot back to its canonical position, so that values can be refreshed after an
// optimiser step and weight gradients can be returned in canonical order.
#include <algorithm>

#include "common.h"
#include "active.h"

namespace mst {

thread_local int g_last_hip_error = 0;

// Chunks of equal size (a short last chunk would cost the same barriers for less work), each of
// whole sub-chunks of KS indices.  An octet segment holds max(len of its eight rows) steps rounded up
// to even: at most (sum of the eight lens) + 1, and at most the chunk's length.
View view_shape(int R, int K, int64_t cap) {
    View v;
    v.R = R;
    v.K = K;
    const int64_t n = cdiv(K, KCMAX), per = cdiv(K, n);
    v.msub = (int)cdiv(per, KSMAX);
    v.KS = (int)(cdiv(cdiv(per, v.msub), 4) * 4);
    v.KC = v.msub * v.KS;
    v.nchunk = (int)cdiv(K, v.KC);
    v.NB = (int)cdiv(R, RB);
    v.NBpad = v.NB + MAX_WG_BLOCKS;
    v.nseg = (int64_t)v.nchunk * v.NBpad * OPB;
    const int64_t nos = (int64_t)v.nchunk * v.NB * OPB;
    v.cap_pairs = cdiv(std::min((cap + nos) / 2 + 1, nos * (v.KC / 2)) + PAIR_TAIL, 8) * 8;
    return v;
}

// Sparse or dense.  The dense products cost the same at every density, the sparse ones about in proportion to
// nnz.  Large batches on whole tiles run at rates that hardly depend on the shape, and the two meet at
// densities that do not either (measured at GPT-2 small / medium / large layer shapes, T >= 2048): fp32 Y and
// dX 0.065-0.085, weight gradient 0.04-0.06, both gradients from one walk against two dense products
// 0.075-0.105; bfloat16 0.05 at T = 16384 and 0.07-0.1 at shorter batches, below 0.03, and 0.03-0.04.  Everywhere else the
// modelled times of the two are compared up to a density of 0.30 (dense from there on): partial tiles and few workgroups move
// the line anywhere between 0.03 and 0.3 (a line at 0.30 lost 12 to 37 %).  Of 150 products Y and dX whose modelled times are
// within a third of each other the choice loses 1.5 % on average and 23 % at the worst; the models favour neither side, and
// deciding ties for one of them by 5 % loses 1.6 or 2.2.
static bool whole_tiles(const mst_layer* L, mst_dtype act, int T) {
    const int tile = act == MST_BF16 ? 256 : 128;
    return T >= 2048 && T % tile == 0 && L->O % tile == 0 && L->I % tile == 0;
}
static bool mostly_dense(const mst_layer* L) { return (double)L->nnz > 0.30 * (double)L->N; }
// (The sum of the k ranges as part of a gather from whole partial outputs.  Rows of whole eights have had neither since their kernels write
// the active positions alone, up to a quarter sooner; the lines drawn with this model stay where they are, on the side of the walk.)
static double dense_wgrad_us(const mst_layer* L, mst_dtype act, int T, bool full) {
    return 3.0 + gemm_mfma_us(GEMM_TN, act, L->O, L->I, T, GEMM_WS_SPLITS, false, full);
}

// The dense kernels of whole tiles take two bfloat16 parts per fp32 operand, 16 of its 24 bits.  Up to these densities
// an automatic product has its fp32 operands in full, whether the walk or the full-precision dense kernels (six products
// per term instead of three) run it: speed alone does not move a layer that the sparse kernels serve well to fewer
// bits.  The choice between the two is between their times.  Above, the dense kernels are ahead by so much that
// two parts are the rule.  Largest error of Y at 768 -> 3072, 1024 tokens, density 0.149, in units of the
// largest output: walk 4.4e-7, full dense 5.5e-7, two parts 7.0e-6.
bool full_precision(const mst_layer* L, WalkJob job, mst_dtype act, int T) {
    if (L->path != MST_PATH_AUTO) return false;
    const int tile = act == MST_BF16 ? 256 : 128;
    const bool whole = T % (job == WALK_BWD_WEIGHT ? 64 : tile) == 0 && L->O % tile == 0 && L->I % tile == 0;
    double line = 0.30;
    if (whole && T >= 2048) line = job == WALK_BWD ? (act == MST_F32 ? 0.07 : 0.03) : job == WALK_BWD_WEIGHT ? 0.035 : act == MST_F32 ? 0.055 : 0.045;
    else if (whole && act == MST_F32) line = 0.15;
    return (double)L->nnz <= line * (double)L->N;
}

// The models take a microsecond of host time, so the answers for the last (T, type) are kept with the layer
// until its active set changes: bits 0-4 known, 5-9 the answers (bit = WalkJob, or SPARSE_DX), 10 the type, 11.. T.
constexpr int SPARSE_DX = 4;
template <typename F>
static bool remembered(const mst_layer* L, int job, mst_dtype act, int T, F&& decide) {
    std::atomic<uint64_t>& word = const_cast<mst_layer*>(L)->choice;
    const uint64_t key = (uint64_t)T << 11 | (uint64_t)(act == MST_BF16) << 10, w = word.load(std::memory_order_relaxed);
    const bool mine = (w & ~(uint64_t)0x3FF) == key;
    if (mine && (w >> job & 1)) return w >> (5 + job) & 1;
    const bool yes = decide();
    word.store((mine ? w : key) | (uint64_t)1 << job | (uint64_t)yes << (5 + job), std::memory_order_relaxed);
    return yes;
}

static double dense_us(const mst_layer* L, WalkJob job, mst_dtype act, int T) {       // Y or dX
    const bool full = full_precision(L, job, act, T);
    return job == WALK_FWD ? gemm_mfma_us(GEMM_NT, act, T, L->O, L->I, 1, true, full)
                           : gemm_mfma_us(GEMM_NN, act, T, L->I, L->O, 1, true, full);
}

// Y and dX, each for itself (job WALK_FWD or WALK_BWD_INPUT): a layer that is wide on one side has its cross-over at
// different densities for the two (3392 -> 448, 504 tokens, 0.09: dX 8.5 us sparse, 15.6 dense; Y 27 dense, a model's 47
// sparse).  One answer for both cost one of them more than 15 % at a tenth of 13800 shapes, by the models.
bool use_dense_path(const mst_layer* L, WalkJob job, mst_dtype act, int T) {
    if (L->path == MST_PATH_DENSE) return true;
    if (L->path == MST_PATH_SPARSE) return false;
    if (whole_tiles(L, act, T)) return (double)L->nnz > (act == MST_F32 ? 0.075 : T >= 8192 ? 0.045 : 0.065) * (double)L->N;
    if (mostly_dense(L)) return true;
    return remembered(L, job, act, T, [&] { return walk_us(L, job, T) > dense_us(L, job, act, T); });
}

// The one-call backward: one walk for both gradients, the two dense products, or, with bfloat16 activations on other than whole
// tiles, a sparse dX beside the dense weight gradient, whose operands need no parts (gemm_wgrad.hip: one product per
// term where dX takes three).  A step of 4099 tokens of 1024 -> 4096, density 0.04: 205 us by one walk, 196 to 200 by dX's walk and
// the dense gradient; 7356 tokens of 4288 -> 3170, 0.048: 1056 -> 923.
// The modelled time of the dense gradient is 5 % above the measured one for rows of whole 16-byte units (sd 4 %) and 14 %
// below it for others (sd 6 %), which is made good here; the two margins are what all three models are unsure of.
// 630 layers of 250 to 5000, 1500 to 9000 tokens, densities 0.03 to 0.1: 3.6 % faster on average than without this choice (up to
// 43 %), nine 3 to 9 % slower (without the correction, margins 1.03 and 1.15: 4.2 %, twenty-four 3 to 14 % slower).
// With fp32 activations a sparse dX beside a dense dW is never the fastest.
static double dense_backward_us(const mst_layer* L, mst_dtype act, int T) {
    const bool full = full_precision(L, WALK_BWD, act, T);
    return gemm_mfma_us(GEMM_NN, act, T, L->I, L->O, GEMM_WS_SPLITS * L->N / ((int64_t)T * L->I), true, full) + dense_wgrad_us(L, act, T, full);
}
bool use_sparse_input_grad(const mst_layer* L, mst_dtype act, int T) {
    if (act != MST_BF16 || L->path != MST_PATH_AUTO || whole_tiles(L, act, T) || !full_precision(L, WALK_BWD, act, T)) return false;
    return remembered(L, SPARSE_DX, act, T, [&] {
        const double modelled = dense_wgrad_us(L, act, T, true), wgrad = (L->O % 8 == 0 && L->I % 8 == 0 ? 0.95 : 1.14) * modelled;
        const double us = walk_us(L, WALK_BWD_INPUT, T) + wgrad + 1.0e-6 * (double)L->N;   // (a read of G by the gather, also where there is none: see dense_wgrad_us)
        return 1.05 * us < walk_us(L, WALK_BWD, T) && 1.2 * us < dense_backward_us(L, act, T) - modelled + wgrad;
    });
}
bool use_fused_backward(const mst_layer* L, mst_dtype act, int T) {
    if (L->path == MST_PATH_DENSE) return false;
    if (L->path == MST_PATH_SPARSE) return true;
    if (whole_tiles(L, act, T)) return (double)L->nnz <= (act == MST_F32 ? 0.085 : 0.035) * (double)L->N;
    if (mostly_dense(L) || use_sparse_input_grad(L, act, T)) return false;
    return remembered(L, WALK_BWD, act, T, [&] { return walk_us(L, WALK_BWD, T) <= dense_backward_us(L, act, T); });
}

bool use_dense_weight_grad(const mst_layer* L, mst_dtype act, int T) {
    if (L->path == MST_PATH_DENSE) return true;
    if (L->path == MST_PATH_SPARSE) return false;
    if (whole_tiles(L, act, T)) return (double)L->nnz > (act == MST_F32 ? 0.05 : 0.03) * (double)L->N;
    if (mostly_dense(L)) return true;
    return remembered(L, WALK_BWD_WEIGHT, act, T, [&] { return walk_us(L, WALK_BWD_WEIGHT, T) > dense_wgrad_us(L, act, T, full_precision(L, WALK_BWD_WEIGHT, act, T)); });
}

constexpr int CSEG = 2048;         // positions per wavefront of build_canonical

struct LayerCarve {
    size_t mask, vals, flat, rowptr, Wd;
    size_t rptr, rent, rperm, rmap, rpos, cptr, cent, cperm, cmap, cpos, cost, heavy, Hd, runs, sy, sx, py, px;
    size_t total;
};

// the tile of gemm_planes.hip divides the outputs of one product, its k step the contraction range
static bool has_planes(int O, int I) { return O % 32 == 0 && I % 32 == 0 && (O % 256 == 0 || I % 256 == 0); }

// rows of whole eights of the mask, and outputs whose bytes an unsigned holds
static bool has_runs(int O, int I) { return I % 8 == 0 && (int64_t)O * I < (int64_t)1 << 30; }

// whole steps of gemm_pairs.hip in both directions
static bool has_pairs(int O, int I) { return O % 64 == 0 && I % 64 == 0; }

static LayerCarve carve_layer(int O, int I, int64_t cap) {
    LayerCarve c{};
    const int64_t N = (int64_t)O * I;
    const View r = view_shape(O, I, cap), k = view_shape(I, O, cap);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    c.mask = take((size_t)N);
    c.vals = take((size_t)cap * 4);
    c.flat = take((size_t)cap * 4);
    c.rowptr = take((size_t)(O + 1) * 4);
    c.Wd = take((size_t)N * 4);
    c.rptr = take((size_t)(r.nseg + 1) * 4);
    c.rent = take((size_t)r.cap_pairs * OCT * 16);
    c.rperm = take((size_t)r.cap_pairs * OCT * 8);
    c.rmap = take((size_t)r.NBpad * RB * 4);
    c.rpos = take((size_t)r.NBpad * RB * 4);
    c.cptr = take((size_t)(k.nseg + 1) * 4);
    c.cent = take((size_t)k.cap_pairs * OCT * 16);
    c.cperm = take((size_t)k.cap_pairs * OCT * 8);
    c.cmap = take((size_t)k.NBpad * RB * 4);
    c.cpos = take((size_t)k.NBpad * RB * 4);
    c.cost = take(16 + 4);
    c.heavy = take((size_t)(HEAVY_MAX + 2) * 4);
    c.Hd = take((size_t)HEAVY_MAX * I * 4);
    c.runs = take(has_runs(O, I) ? (size_t)O * (size_t)cdiv(I, 32) * sizeof(uint2) : 0);
    c.sy = take(has_pairs(O, I) ? pairs_view(nullptr, O, I).bytes : 0);
    c.sx = take(has_pairs(O, I) ? pairs_view(nullptr, I, O).bytes : 0);
    c.py = take(has_planes(O, I) ? (size_t)N * 4 : 0);
    c.px = take(has_planes(O, I) ? (size_t)N * 4 : 0);
    c.total = off;
    return c;
}

static bool shape_ok(int O, int I, int64_t cap) {
    if (O < 1 || I < 1 || O > 65535 || I > 65535) return false;
    const int64_t N = (int64_t)O * I;
    if (N >= (int64_t)1 << 31) return false;
    if (cap < 0 || cap > N) return false;
    return true;
}

Workspace carve_workspace(void* base, int O, int I, int64_t cap, int T) {
    Workspace w{};
    const int64_t N = (int64_t)O * I;
    const View r = view_shape(O, I, cap), k = view_shape(I, O, cap);
    // per-row-per-sub-chunk counts of either view, rows padded to whole blocks
    const int64_t cnt_r = (int64_t)r.nsub() * r.NBpad * RB, cnt_c = (int64_t)k.nsub() * k.NBpad * RB;
    const int64_t ntile = cdiv(T > 0 ? T : 1, WT);
    char* b = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return b ? b + o : nullptr; };
    w.G = (float*)take((size_t)N * 4);
    w.Wd = (float*)take((size_t)N * 4);
    w.cidx = (int*)take((size_t)N * 4);
    w.sel = (uint8_t*)take((size_t)N);
    w.psel = (uint8_t*)take((size_t)(cap > 0 ? cap : 1));
    w.segcnt[0] = (int*)take((size_t)(std::max(cnt_r, cdiv(N, CSEG)) + 1) * 4);      // (build_canonical counts per segment of CSEG)
    w.segcnt[1] = (int*)take((size_t)(cnt_c + 1) * 4);
    w.qlen[0] = (int*)take((size_t)(r.nseg + 1) * 4);
    w.qlen[1] = (int*)take((size_t)(k.nseg + 1) * 4);
    w.rowcnt = (int*)take((size_t)(O + 1) * 4);
    w.blk = (uint32_t*)take((size_t)(cdiv(N, SELECT_BLOCK) + cdiv(cap > 0 ? cap : 1, SELECT_BLOCK) + 4) * 4);
    w.sel_state = (uint64_t*)take((size_t)SEL_STATES * SEL_STATE_WORDS * 8);
    w.gemm_floats = (size_t)GEMM_WS_SPLITS * (size_t)N;
    w.gemm = (float*)take(w.gemm_floats * 4);
    w.partial_floats = (size_t)ntile * 2 * OCT * (size_t)std::max(r.cap_pairs, k.cap_pairs);
    w.partial = (float*)take(w.partial_floats * 4);
    w.total = off;
    return w;
}

// ------------------------------------------------------------------ kernels

// one block per row r of the mask: active count per sub-chunk of KS columns and per row; blocks past
// the last row (the padding rows of the view) write zero counts
__device__ inline void count_row_block(const uint8_t* __restrict__ mask, int O, int I, int KS, int nsub, int Rpad,
                                       int* __restrict__ segcnt, int* __restrict__ rowcnt, int r, int* cnt /* [nsub] */) {
    if (r >= O) {
        for (int c = threadIdx.x; c < nsub; c += blockDim.x) segcnt[(size_t)c * Rpad + r] = 0;
        return;
    }
    for (int c = threadIdx.x; c < nsub; c += blockDim.x) cnt[c] = 0;
    __syncthreads();
    const uint8_t* m = mask + (size_t)r * I;
    int total = 0;
    for (int i = threadIdx.x; i < I; i += blockDim.x) {
        if (m[i]) { atomicAdd(&cnt[i / KS], 1); }
    }
    __syncthreads();
    if (segcnt)
        for (int c = threadIdx.x; c < nsub; c += blockDim.x) segcnt[(size_t)c * Rpad + r] = cnt[c];
    if (threadIdx.x == 0) {
        for (int c = 0; c < nsub; ++c) total += cnt[c];
        rowcnt[r] = total;
    }
}

// [KSMAX rows x 64 columns] of the mask into LDS (rows beyond the sub-chunk or O and columns beyond I
// read as zero); 256 threads, 32 bytes each.  Row stride 68 bytes: the 64 lanes of a wavefront read
// one row's 64 bytes without bank conflicts.
constexpr int MT_COLS = 64, MT_LD = 68;
__device__ inline void load_mask_tile(const uint8_t* __restrict__ mask, int O, int I, int o0, int nrows, int i0,
                                      uint8_t* __restrict__ m, int tid) {
    const int r = tid >> 1, half = tid & 1;
    const int o = r < nrows ? o0 + r : O, ib = i0 + 32 * half;
    uint8_t* dst = m + r * MT_LD + 32 * half;
    const uint8_t* src = mask + (size_t)o * I + ib;
    if (o < O && ib + 32 <= I && ((reinterpret_cast<uintptr_t>(src) & 3) == 0)) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            reinterpret_cast<uint32_t*>(dst)[u] = reinterpret_cast<const uint32_t*>(src)[u];
    } else {
        for (int u = 0; u < 32; ++u) dst[u] = (o < O && ib + u < I) ? src[u] : (uint8_t)0;
    }
}

// block (bx, c) = (64 columns, sub-chunk c of KS rows): active count of every column inside the sub-chunk.
// Thread (column j, row group rg of 32 rows) counts its rows from the LDS tile.
__device__ inline void count_col_block(const uint8_t* __restrict__ mask, int O, int I, int KS, int Rpad, int* __restrict__ segcnt,
                                       int bx, int c, uint8_t* m, int (*part)[MT_COLS]) {
    const int tid = threadIdx.x, j = tid & 63, rg = tid >> 6, i0 = bx * MT_COLS;
    load_mask_tile(mask, O, I, c * KS, KS, i0, m, tid);
    __syncthreads();
    int n = 0;
#pragma unroll
    for (int k = 0; k < 32; ++k) n += m[(32 * rg + k) * MT_LD + j] != 0;
    part[rg][j] = n;
    __syncthreads();
    // (columns past the matrix read as empty: the padding rows of the view get zero counts)
    if (rg == 0 && i0 + j < Rpad) segcnt[(size_t)c * Rpad + i0 + j] = part[0][j] + part[1][j] + part[2][j] + part[3][j];
}

// The counts of both views (segcnt_c null: of the rows alone): the first row_blocks blocks of a layer take a row each
struct CountArgs {
    const uint8_t* mask;
    int O, I, KS_r, nsub_r, Rpad_r, KS_c, Rpad_c, row_blocks, col_tiles;
    int *segcnt_r, *rowcnt, *segcnt_c;
};
template <int CAP>
__global__ __launch_bounds__(256) void k_count(const Batch<CountArgs, CAP> batch) {
    extern __shared__ int cnt[];
    __shared__ __attribute__((aligned(16))) uint8_t m[KSMAX * MT_LD];
    __shared__ int part[4][MT_COLS];
    if (batch.surplus()) return;
    const unsigned b = blockIdx.x;
    const CountArgs a = batch.entry();
    if (b < (unsigned)a.row_blocks) {
        count_row_block(a.mask, a.O, a.I, a.KS_r, a.nsub_r, a.Rpad_r, a.segcnt_r, a.rowcnt, (int)b, cnt);
    } else {
        const unsigned t = b - (unsigned)a.row_blocks;
        count_col_block(a.mask, a.O, a.I, a.KS_c, a.Rpad_c, a.segcnt_c, (int)(t % (unsigned)a.col_tiles), (int)(t / (unsigned)a.col_tiles), m, part);
    }
}

// One workgroup per row block (thread j = row j): decides which rows share an octet, then writes the pairs of every
// (chunk, octet) segment of the block.  A segment is as long as the longest of its eight rows in that chunk, so rows should share
// an octet that are long in the same chunks.
//   - By total length, longest first, lower row first on ties (the empty padding blocks keep the identity).  With h rows
//     spread over whole octets (h <= #empty rows / 7) the octets cost about
//       sum_{j<h} ceil(len_j / 8)  +  sum over the octets of the other rows of their longest row,
//     h is the value that minimises it (0 for every mask without empty rows).
//   - By halves: the longer and the shorter half of the rows in the first part of the chunks, each of those by the next
//     part, four times (with two chunks: quarters by the first, then by the second).  Of rows of equal density the total says
//     little about a chunk, and every split narrows one of them: real entries of all steps at 12.8 a row and chunk 0.75 -> 0.85
//     with two chunks, 0.73 -> 0.81 with three, 0.71 -> 0.76 with five, 0.71 -> 0.73 with eight.  Octets that lie four
//     apart, and so meet on a SIMD unit of the walk, hold both halves of every split.
// No row spread: whichever takes fewer pairs.
// Bound by the latency of its reads of the counts (there are only as many workgroups as row blocks), so
// all of them are issued together, once, and kept by chunk in LDS.
struct ViewArgs {                                     // of one view: the first nb_r blocks of k_block_rank are the row view's
    const int* segcnt;
    int msub, nchunk, Rpad, NBpad, NB;
    int64_t nseg;
    int *rowmap, *rowpos, *qlen, *ptr;
};
struct RankArgs {
    ViewArgs row, col;
};
template <int CAP>
__global__ __launch_bounds__(RB) void k_block_rank(const Batch<RankArgs, CAP> batch) {
    extern __shared__ uint16_t cnt_s[];               // [nchunk][RB] entries of a row in a chunk
    __shared__ __attribute__((aligned(16))) uint32_t code_s[RB];
    __shared__ int sorted[RB], row_s[2][RB];          // row_s: rows by place, ranked and halved
    __shared__ int h_s, nzero_s, gain_s;
    if (batch.surplus()) return;
    const unsigned bu = blockIdx.x;
    const RankArgs both = batch.entry();
    const bool col = bu >= (unsigned)both.row.NBpad;
    const ViewArgs v = col ? both.col : both.row;
    const int j = threadIdx.x, b = (int)bu - (col ? both.row.NBpad : 0);
    const int msub = v.msub, nchunk = v.nchunk, Rpad = v.Rpad, NBpad = v.NBpad;
    const int* __restrict__ segcnt = v.segcnt;
    int *__restrict__ rowmap = v.rowmap, *__restrict__ rowpos = v.rowpos, *__restrict__ qlen = v.qlen;
    if (j == 0) h_s = nzero_s = gain_s = 0;
    // the row's entries by chunk; keys: in all, and in the parts of the chunks that the splits go by
    const int nkey = nchunk >= 3 ? 4 : nchunk == 2 ? 2 : 0;
    int len = 0, key[4] = {0, 0, 0, 0};
    constexpr int MSUB = KCMAX / KSMAX, AT_ONCE = 4;
    for (int c0 = 0; c0 < nchunk; c0 += AT_ONCE) {
        int x[AT_ONCE][MSUB];
#pragma unroll
        for (int d = 0; d < AT_ONCE; ++d)
#pragma unroll
            for (int u = 0; u < MSUB; ++u) x[d][u] = segcnt[(size_t)(min(c0 + d, nchunk - 1) * msub + min(u, msub - 1)) * Rpad + b * RB + j];
#pragma unroll
        for (int d = 0; d < AT_ONCE; ++d) {
            const int c = c0 + d;
            if (c >= nchunk) break;
            int n = 0;
#pragma unroll
            for (int u = 0; u < MSUB; ++u) n += u < msub ? x[d][u] : 0;
            cnt_s[c * RB + j] = (uint16_t)n;
            len += n;
            const int part = nchunk <= 4 ? c : 4 * c / nchunk;
#pragma unroll
            for (int q = 0; q < 4; ++q) key[q] += part == q ? n : 0;
        }
    }
    if (nchunk == 3) key[3] = len;
    // this row's place among the block's by ascending codes, which differ
    auto place = [&](uint32_t code) {
        code_s[j] = code;
        __syncthreads();
        int at = 0;
#pragma unroll 8
        for (int u = 0; u < RB; u += 4) {
            const uint4 x = *reinterpret_cast<const uint4*>(code_s + u);
            at += (x.x < code) + (x.y < code) + (x.z < code) + (x.w < code);
        }
        return at;
    };
    const int rank = place((uint32_t)(0xFFFF - len) << 7 | (uint32_t)j);
    sorted[rank] = len;
    if (len == 0) atomicAdd(&nzero_s, 1);
    __syncthreads();
    if (j < 32) {                                    // candidate h = j on lane j of the first wavefront
        int cost = 0x7FFFFFFF;
        if (j <= OPB && 7 * j <= nzero_s) {
            cost = 0;
            for (int u = 0; u < j; ++u) cost += (sorted[u] + 7) >> 3;
            for (int p = j; p < RB - 7 * j; p += OCT) cost += sorted[p];
        }
        int best = cost, at = j;
        for (int d = 16; d >= 1; d >>= 1) {
            const int oc = __shfl_xor(best, d, 32), oa = __shfl_xor(at, d, 32);
            if (oc < best || (oc == best && oa < at)) { best = oc; at = oa; }
        }
        if (j == 0) h_s = at;
    }
    __syncthreads();
    const int h = h_s, p = rank;
    int slot, flag_row = 0;
    if (p < h) { slot = OCT * p; flag_row = SPREAD_FLAG; }               // spread row: lane group 0 of octet p
    else if (p < RB - 7 * h) slot = OCT * h + (p - h);                   // ordinary rows fill the other octets
    else { const int e = p - (RB - 7 * h); slot = OCT * (e / 7) + 1 + e % 7; }   // empty rows own the rest
    row_s[0][slot] = j;
    int halved = 0;
    const bool split = h == 0 && nkey > 0 && sorted[0] > 0;
    if (split) {
        // splits: place among the rows by (group so far, key, row), the group's next bits from it
        int group = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q >= nkey) break;
            if (q > 0) __syncthreads();
            halved = place((uint32_t)group << 23 | (uint32_t)(0xFFFF - key[q]) << 7 | (uint32_t)j);
            group = nkey == 4 ? halved >> (6 - q) : halved >> (q == 0 ? 5 : 3);
        }
        // group: the splits' results, the first one highest; octets four apart differ in each of them
        const int octet = nkey == 4 ? ((group >> 3) & 1) << 3 | ((group >> 1) & 1) << 2 | ((group >> 3 ^ group >> 2) & 1) << 1 | ((group >> 1 ^ group) & 1)
                                    : (group & 12) | (((group >> 2) + group) & 3);
        halved = OCT * octet + (halved & (OCT - 1));
        row_s[1][halved] = j;
    }
    __syncthreads();
    // pairs of a segment: longest of its eight rows (a spread row: an eighth of it), rounded up to even, halved
    auto pairs = [&](int how, int c, int o) {
        const uint16_t* cnt = cnt_s + c * RB;
        const int* rows = row_s[how] + o * OCT;
        int L = cnt[rows[0]];
        if (o < h) {
            L = (L + 7) >> 3;
        } else {
#pragma unroll
            for (int g = 1; g < OCT; ++g) L = max(L, (int)cnt[rows[g]]);
        }
        return (L + 1) >> 1;
    };
    int how = 0;
    if (split) {
        int gain = 0;
        for (int idx = j; idx < nchunk * OPB; idx += RB) gain += pairs(0, idx / OPB, idx % OPB) - pairs(1, idx / OPB, idx % OPB);
        for (int d = 32; d >= 1; d >>= 1) gain += __shfl_xor(gain, d, 64);
        if ((j & 63) == 0) atomicAdd(&gain_s, gain);
        __syncthreads();
        how = gain_s > 0 ? 1 : 0;
    }
    if (how) slot = halved;
    const int flag_oct = slot / OCT < h ? SPREAD_FLAG : 0;
    rowmap[b * RB + slot] = (b * RB + j) | flag_oct;
    rowpos[b * RB + j] = slot | flag_row;
    for (int idx = j; idx < nchunk * OPB; idx += RB) {
        const int c = idx / OPB, o = idx % OPB;
        qlen[((size_t)c * NBpad + b) * OPB + o] = pairs(how, c, o);
    }
}

// exclusive scan by ONE block of 1024 threads: out[j] = sum_{j' < j} in[j'], out[n] = total (in == out
// is allowed).  Each of the 16 wavefronts owns one contiguous segment and reads it with its 64
// lanes side by side (coalesced, several rows of 64 in flight): first the segment's sum, then,
// with the sums of the segments before it as carry, the running values (a 64-lane scan per row).
__device__ inline void block_scan_excl(const int* in, int* out, int64_t n, int* wsum) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwave = blockDim.x >> 6;
    const int64_t rows = (n + 63) / 64;                            // rows of 64 elements
    const int64_t rpw = (rows + nwave - 1) / nwave;                // rows per wavefront
    const int64_t r0 = (int64_t)wave * rpw, r1 = min(rows, r0 + rpw);
    int tot = 0;
#pragma unroll 4
    for (int64_t r = r0; r < r1; ++r) {
        const int64_t j = r * 64 + lane;
        tot += (j < n) ? in[j] : 0;
    }
    for (int d = 32; d >= 1; d >>= 1) tot += __shfl_xor(tot, d, 64);
    __syncthreads();                                 // wsum free again (an earlier scan of this block may still read it)
    if (lane == 0) wsum[wave] = tot;
    __syncthreads();
    int carry = 0;
    for (int w = 0; w < wave; ++w) carry += wsum[w];
    int v_next = (r0 < r1 && r0 * 64 + lane < n) ? in[r0 * 64 + lane] : 0;
    for (int64_t r = r0; r < r1; ++r) {
        const int64_t j = r * 64 + lane;
        const int v = v_next;
        if (r + 1 < r1) v_next = ((r + 1) * 64 + lane < n) ? in[(r + 1) * 64 + lane] : 0;   // read before the row is written: in may be out
        int x = v;
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        if (j < n) out[j] = carry + x - v;
        carry += __shfl(x, 63, 64);
    }
    if (wave == nwave - 1 && lane == 0) out[n] = carry;            // the last segment ends at n (or is empty): the total
}

struct ScanArgs {
    const int* in;
    int* out;
    int64_t n;
};
template <int CAP>
__global__ __launch_bounds__(1024) void k_scan_excl(const Batch<ScanArgs, CAP> batch) {     // a block each
    __shared__ int wsum[16];
    const ScanArgs a = batch.entry();
    block_scan_excl(a.in, a.out, a.n, wsum);
}

// One block does what follows the segment lengths of a view: (row view only) the canonical row
// pointers from the per-row counts; the first pair of every octet segment; the view's cost
// for the weight gradient, which either view can drive -- the wavefronts of a workgroup take one
// octet of a block each and wait at every chunk for the longest, so a view costs the sum over
// (chunk, block) of the most pairs of an octet.
struct PtrArgs {
    RankArgs views;
    const int* rowcnt;                                // counts per row
    int* rowptr;
    int nrows;
    unsigned long long* cost;
    const int* heavy;
    int* dense_live;
    int live;
};
template <int CAP>
__global__ __launch_bounds__(1024) void k_view_ptr(const Batch<PtrArgs, CAP> batch) {    // two blocks per layer: row view, col view
    __shared__ int wsum[16];
    __shared__ unsigned long long cost_s;
    const bool col = blockIdx.x != 0;
    const PtrArgs a = batch.entry();
    const ViewArgs v = col ? a.views.col : a.views.row;
    const int* const qlen = v.qlen;
    int* const ptr = v.ptr;
    const int NBpad = v.NBpad, NB = v.NB, nchunk = v.nchunk;
    if (!col) block_scan_excl(a.rowcnt, a.rowptr, a.nrows, wsum);
    block_scan_excl(qlen, ptr, v.nseg, wsum);
    if (threadIdx.x == 0) cost_s = 0ull;
    __syncthreads();                                  // ptr[] written by this block is visible to it
    unsigned long long mine = 0ull;
    for (int idx = threadIdx.x; idx < nchunk * NB; idx += blockDim.x) {
        const int c = idx / NB, b = idx % NB;
        const int* pp = ptr + ((int64_t)c * NBpad + b) * OPB;
        int worst = 0;
        for (int o = 0; o < OPB; ++o) worst = max(worst, pp[o + 1] - pp[o]);
        mine += (unsigned long long)worst;
    }
    if (mine) atomicAdd(&cost_s, mine);
    __syncthreads();
    // (a row view that leaves heavy rows out cannot drive the weight gradient)
    if (threadIdx.x == 0) {
        a.cost[col ? 1 : 0] = (!col && a.heavy && a.heavy[0] > 0) ? (1ull << 50) : cost_s;
        if (!col) *a.dense_live = a.live;
    }
}

// entry slot (as index into ent viewed as uint2[], and into perm) of step j of a row
__device__ inline int64_t entry_slot(int pair0, int g, int j) {
    return (((int64_t)pair0 + (j >> 1)) * OCT + g) * 2 + (j & 1);
}

// entry j of a row inside a chunk: its lane group's step j, or dealt to the eight lane groups (spread row)
__device__ inline int64_t row_slot(int pair0, int g, bool spread, int j) {
    return spread ? entry_slot(pair0, j & 7, j >> 3) : entry_slot(pair0, g, j);
}

// Slots of a row's lane group (of the whole octet for a spread row) past its `run` entries, up
// to the octet's length: zero-weight padding (offset 0, perm -1).  The seven empty rows that
// share a spread octet own no slots.  `lanes` threads of the caller share the work.
__device__ inline void pad_row_slots(uint2* __restrict__ ent, int* __restrict__ perm, int pair0, int npairs, int g,
                                     bool spread, int run, int lane, int lanes) {
    const int total = spread ? 16 * npairs : 2 * npairs;
    for (int j = run + lane; j < total; j += lanes) {
        const int64_t e = row_slot(pair0, g, spread, j);
        ent[e] = make_uint2(0u, 0u);
        perm[e] = -1;
    }
}

// one wavefront per (row, part of its sub-chunks) (incl. the padding rows of the last block, which
// only pad): ordered compaction of the row into canonical arrays and the row view.  A layer of
// few long rows gives every row `nparts` wavefronts of `spp` sub-chunks each (one per row would leave
// the 1280 rows of a 5120-wide layer on 320 workgroups); a part finds its first canonical index and
// its place in its first chunk from the counts of the sub-chunks before it (a heavy row, whose counts
// were cleared, from the mask itself).
struct FillArgs {                                     // of one view
    const uint8_t* mask;
    const float* W;
    int O, I, KS, msub, nsub, NBpad, NB, Rpad;
    const int *rowptr, *ptr, *rowpos, *rowmap, *segcnt, *heavy;
    float* vals;
    int *flat, *cidx, *perm;
    uint2* ent;
    int nparts, spp;                                  // (row view)
    int col_tiles;                                    // (col view)
};
template <int CAP>
__global__ __launch_bounds__(256) void k_fill_row(const Batch<FillArgs, CAP> batch) {
    if (batch.surplus()) return;
    const unsigned blk = blockIdx.x;
    const FillArgs a = batch.entry();
    const uint8_t* __restrict__ mask = a.mask;
    const float* __restrict__ W = a.W;
    const int O = a.O, I = a.I, KS = a.KS, msub = a.msub, nsub = a.nsub, NBpad = a.NBpad, NB = a.NB, Rpad = a.Rpad;
    const int *__restrict__ rowptr = a.rowptr, *__restrict__ ptr = a.ptr, *__restrict__ rowpos = a.rowpos, *__restrict__ rowmap = a.rowmap;
    const int *__restrict__ heavy = a.heavy, *__restrict__ segcnt = a.segcnt;
    float* __restrict__ vals = a.vals;
    int *__restrict__ flat = a.flat, *__restrict__ cidx = a.cidx, *__restrict__ perm = a.perm;
    uint2* __restrict__ ent = a.ent;
    const int nparts = a.nparts, spp = a.spp;
    const int lane = threadIdx.x & 63;
    const int unit = (int)blk * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int r = unit / nparts, s0 = (unit % nparts) * spp, s1 = min(nsub, s0 + spp);
    if (r >= NB * RB) return;
    // a heavy row (HEAVY_MAX = 64 list entries, one per lane) fills the canonical arrays only
    const bool hv = heavy != nullptr && __ballot(lane < heavy[0] && heavy[1 + lane] == r) != 0ull;
    const int b = r / RB, rp = rowpos[r], rank = rp & ~SPREAD_FLAG, g = rank % OCT, o = rank / OCT;
    const bool spread = (rp & SPREAD_FLAG) != 0;
    // an empty row placed in a spread octet: the octet's slots belong to the spread row
    const bool guest = !spread && (rowmap[b * RB + OCT * o] & SPREAD_FLAG) != 0;
    const bool real = r < O;
    const uint8_t* m = mask + (size_t)r * I;
    const float* w = W + (size_t)r * I;
    int canon = real ? rowptr[r] : 0, run = 0;        // run: entries of this row in the current chunk so far
    if (real && s0 > 0) {                             // entries of this row in the sub-chunks before s0
        const int cs = s0 / msub * msub;              // first sub-chunk of s0's chunk
        int before = 0, here = 0;
        if (hv) {                                     // (a heavy row's counts were cleared: count the mask)
            for (int i = lane; i < s0 * KS && i < I; i += 64) before += m[i] != 0;
        } else {
            for (int c = lane; c < s0; c += 64) {
                const int n = segcnt[(size_t)c * Rpad + r];
                before += n;
                if (c >= cs) here += n;
            }
        }
        for (int d = 32; d >= 1; d >>= 1) { before += __shfl_xor(before, d, 64); here += __shfl_xor(here, d, 64); }
        canon += before;
        run = here;
    }
    const int KC = KS * msub;
    for (int sc = s0; sc < s1; ++sc) {
        const int c = sc / msub;
        if (sc == c * msub) run = 0;
        const size_t seg = ((size_t)c * NBpad + b) * OPB + o;
        const int pair0 = ptr[seg], npairs = ptr[seg + 1] - pair0;
        const int i1 = real ? min(I, (sc + 1) * KS) : 0;
        for (int i0 = sc * KS; i0 < i1; i0 += 64) {
            const int i = i0 + lane;
            const bool on = i < i1 && m[i] != 0;
            const unsigned long long bal = __ballot(on);
            if (on) {
                const int at = __popcll(bal & ((1ull << lane) - 1ull));
                const int k = canon + at;
                const float v = w[i];
                vals[k] = v;
                flat[k] = r * I + i;
                cidx[(size_t)r * I + i] = k;
                if (!hv) {
                    const int64_t e = row_slot(pair0, g, spread, run + at);
                    ent[e] = make_uint2(lds_off((uint32_t)(i - c * KC)), __float_as_uint(v));
                    perm[e] = k;
                }
            }
            run += __popcll(bal);
            canon += __popcll(bal);
        }
        // the part that holds the chunk's last sub-chunk knows the row's whole count in it: it pads
        if (!guest && sc == min(nsub, (c + 1) * msub) - 1) pad_row_slots(ent, perm, pair0, npairs, g, spread, hv ? 0 : run, lane, 64);
    }
}

// ---- vals / flat / rowptr alone.  Canonical order is ascending flat index, so the arrays are
// the ordered compaction of the mask as ONE sequence of N positions: a wavefront owns a segment of
// CSEG consecutive positions whatever the layer's shape is (one wavefront per row leaves a
// layer of few long rows with a handful of workgroups).
__device__ inline int nonzero_bytes(uint32_t x) {
    const uint32_t t = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
    return __popc(t);
}

// active positions of every segment
struct CanonicalArgs {
    const uint8_t* mask;
    const float* W;
    int O, I;
    int64_t N;
    int nseg;
    int *segcnt, *rowptr, *flat;
    float* vals;
    uint2* runs;               // null: not wanted, or rows that end inside a word
};
template <int CAP>
__global__ __launch_bounds__(256) void k_count_seg(const Batch<CanonicalArgs, CAP> batch) {
    if (batch.surplus()) return;
    const unsigned blk = blockIdx.x;
    const CanonicalArgs a = batch.entry();
    const uint8_t* __restrict__ mask = a.mask;
    const int64_t N = a.N;
    const int nseg = a.nseg;
    int* __restrict__ segcnt = a.segcnt;
    const int lane = threadIdx.x & 63;
    const int sg = (int)blk * 4 + (threadIdx.x >> 6);
    if (sg >= nseg) return;
    const int64_t base = (int64_t)sg * CSEG;
    int c = 0;
#pragma unroll
    for (int j = 0; j < CSEG; j += 1024) {           // 16 bytes per lane and round
        const int64_t p = base + j + 16 * lane;
        if (p + 16 <= N) {
            const uint4 m = *reinterpret_cast<const uint4*>(mask + p);
            c += nonzero_bytes(m.x) + nonzero_bytes(m.y) + nonzero_bytes(m.z) + nonzero_bytes(m.w);
        } else {
            for (int u = 0; u < 16; ++u) c += (p + u < N && mask[p + u] != 0) ? 1 : 0;
        }
    }
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
    if (lane == 0) segcnt[sg] = c;
}

// segptr[sg] = active positions before segment sg.  A lane takes four consecutive positions of a
// window of 256; the row pointers are written by the wavefront whose segment holds the row's
// first position (rowptr[O] by the last one).  Eight lanes have a word of active.h (a launch of its own: 4 to 8 us per layer of an
// update, of a GPT-2-large block).
template <int CAP>
__global__ __launch_bounds__(256) void k_fill_canonical(const Batch<CanonicalArgs, CAP> batch) {
    if (batch.surplus()) return;
    const unsigned blk = blockIdx.x;
    const CanonicalArgs a = batch.entry();
    const uint8_t* __restrict__ mask = a.mask;
    const float* __restrict__ W = a.W;
    const int O = a.O, I = a.I, nseg = a.nseg;
    const int64_t N = a.N;
    const int* __restrict__ segptr = a.segcnt;
    int* __restrict__ rowptr = a.rowptr;
    float* __restrict__ vals = a.vals;
    int* __restrict__ flat = a.flat;
    const int lane = threadIdx.x & 63;
    const int sg = (int)blk * 4 + (threadIdx.x >> 6);
    if (sg >= nseg) return;
    const int64_t base = (int64_t)sg * CSEG, end = min(N, base + (int64_t)CSEG);
    const unsigned long long below = (1ull << lane) - 1ull;
    int canon = segptr[sg];
    int64_t row = (base + I - 1) / I;                 // first row that starts at or after base
    for (int64_t w0 = base; w0 < end; w0 += 256) {
        const int64_t p = w0 + 4 * lane;
        bool on[4] = {false, false, false, false};
        float w[4] = {0.f, 0.f, 0.f, 0.f};
        if (p + 4 <= end) {
            const uint32_t m4 = *reinterpret_cast<const uint32_t*>(mask + p);
            if (m4) {
                const float4 w4 = *reinterpret_cast<const float4*>(W + p);
                w[0] = w4.x; w[1] = w4.y; w[2] = w4.z; w[3] = w4.w;
            }
            on[0] = (m4 & 0xFFu) != 0; on[1] = (m4 & 0xFF00u) != 0; on[2] = (m4 & 0xFF0000u) != 0; on[3] = (m4 & 0xFF000000u) != 0;
        } else {
            for (int u = 0; u < 4; ++u)
                if (p + u < end && mask[p + u] != 0) { on[u] = true; w[u] = W[p + u]; }
        }
        unsigned long long bal[4];
        int before = 0, total = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bal[u] = __ballot(on[u]);
            before += __popcll(bal[u] & below);
            total += __popcll(bal[u]);
        }
        int k = canon + before;
        if (a.runs) {
            uint32_t bits = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) bits |= (on[u] ? 1u : 0u) << (4 * (lane & 7) + u);
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) bits |= (uint32_t)__shfl_xor((int)bits, d, 64);
            if ((lane & 7) == 0 && p < end) a.runs[p >> 5] = make_uint2(~bits, (uint32_t)k);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (on[u]) { vals[k] = w[u]; flat[k] = (int)(p + u); ++k; }
        const int64_t wend = min(end, w0 + 256);
        for (int64_t q = row * I; q < wend; q += I, ++row) {   // rows that start inside the window
            const int l = (int)(q - w0) >> 2, u0 = (int)(q - w0) & 3;
            const unsigned long long lt = (1ull << l) - 1ull;
            int cnt = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) cnt += __popcll(bal[u] & lt) + ((u < u0) ? (int)((bal[u] >> l) & 1ull) : 0);
            if (lane == 0) rowptr[row] = canon + cnt;
        }
        canon += total;
    }
    if (sg == nseg - 1 && lane == 0) rowptr[O] = canon;
}

// block = (64 columns, sub-chunk sc of KS rows): rows i0 .. i0+63 of the col view.  The
// mask tile sits in LDS; thread (column j, row group rg of 32 rows) counts its rows, the
// counts of the chunk's earlier sub-chunks and of the row groups before it give the position of its
// first entry in the column's list, then it writes its entries in row order.
template <int CAP>
__global__ __launch_bounds__(256) void k_fill_col(const Batch<FillArgs, CAP> batch) {
    __shared__ __attribute__((aligned(16))) uint8_t m[KSMAX * MT_LD];
    __shared__ int part[4][MT_COLS];
    if (batch.surplus()) return;
    const unsigned blk = blockIdx.x;
    const FillArgs a = batch.entry();
    const uint8_t* __restrict__ mask = a.mask;
    const float* __restrict__ W = a.W;
    const int O = a.O, I = a.I, KS = a.KS, msub = a.msub, nsub = a.nsub, NBpad = a.NBpad, NB = a.NB, Rpad = a.Rpad;
    const int *__restrict__ segcnt = a.segcnt, *__restrict__ ptr = a.ptr, *__restrict__ rowpos = a.rowpos, *__restrict__ rowmap = a.rowmap;
    const int* __restrict__ cidx = a.cidx;
    uint2* __restrict__ ent = a.ent;
    int* __restrict__ perm = a.perm;
    const int tid = threadIdx.x, j = tid & 63, rg = tid >> 6;
    const int i0 = (int)(blk % (unsigned)a.col_tiles) * MT_COLS, sc = (int)(blk / (unsigned)a.col_tiles), c = sc / msub, i = i0 + j;
    const int o0 = sc * KS, oc0 = c * msub * KS;
    load_mask_tile(mask, O, I, o0, KS, i0, m, tid);
    __syncthreads();
    uint32_t bits = 0;                                // this thread's 32 rows of its column
#pragma unroll
    for (int k = 0; k < 32; ++k) bits |= (uint32_t)(m[(32 * rg + k) * MT_LD + j] != 0) << k;
    part[rg][j] = __popc(bits);
    __syncthreads();
    if (i >= NB * RB) return;                         // (columns past the matrix only pad)
    int jj = 0;
    for (int u = c * msub; u < sc; ++u) jj += segcnt[(size_t)u * Rpad + i];
    for (int r = 0; r < rg; ++r) jj += part[r][j];
    const int b = i / RB, rp = rowpos[i], rank = rp & ~SPREAD_FLAG, g = rank % OCT, o = rank / OCT;
    const bool spread = (rp & SPREAD_FLAG) != 0;
    const bool guest = !spread && (rowmap[b * RB + OCT * o] & SPREAD_FLAG) != 0;
    const size_t seg = ((size_t)c * NBpad + b) * OPB + o;
    const int pair0 = ptr[seg], npairs = ptr[seg + 1] - pair0;
    // A wavefront's columns hold their entries in different rows: it takes as many turns as the fullest of
    // them has entries, not one per row that any has, and four entries' reads go out together.
    while (bits) {
        int ol[4], ci[4];
        float w[4];
        bool has[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            has[q] = bits != 0;
            ol[q] = has[q] ? 32 * rg + __ffs((int)bits) - 1 : ol[0];
            bits &= bits - 1;
            const size_t f = (size_t)(o0 + ol[q]) * I + i;
            w[q] = W[f];
            ci[q] = cidx[f];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!has[q]) continue;
            const int64_t e = row_slot(pair0, g, spread, jj);
            ent[e] = make_uint2(lds_off((uint32_t)(o0 + ol[q] - oc0)), __float_as_uint(w[q]));
            perm[e] = ci[q];
            ++jj;
        }
    }
    // the last row group of the chunk's last sub-chunk knows the column's whole count in the chunk: it pads
    if (rg == 3 && !guest && sc == min(nsub, (c + 1) * msub) - 1) pad_row_slots(ent, perm, pair0, npairs, g, spread, jj, 0, 1);
}

// The entries of one or both views in one launch: the first `row_blocks` blocks refresh the row
// view's, the next `col_blocks` the col view's, then (with row blocks) HEAVY_MAX blocks the dense
// matrix of the heavy rows, the rest the dense copy.  A thread takes four slots: one 16-byte read of their
// canonical indices.  LATE: a view that was left out of earlier hand-overs takes what the last one handed over,
// which the dense copy holds; vals[] may have changed since.  Without a live dense copy nothing was left out.
template <bool LATE>
__global__ __launch_bounds__(256) void k_sync_views(const float* __restrict__ vals, unsigned row_blocks, unsigned col_blocks,
                             const int* __restrict__ ptr_r, int64_t nseg_r, const int* __restrict__ perm_r,
                             uint2* __restrict__ ent_r,
                             const int* __restrict__ ptr_c, int64_t nseg_c, const int* __restrict__ perm_c,
                             uint2* __restrict__ ent_c, const int* __restrict__ heavy, const int* __restrict__ rowptr,
                             const int* __restrict__ flat, int I, float* __restrict__ Hd, unsigned heavy_blocks,
                             float* __restrict__ Wd, int64_t nnz, int* __restrict__ dense_live) {
    if (LATE) {
        if (*dense_live == 0) return;
    } else if (blockIdx.x == 0 && threadIdx.x == 0) {
        *dense_live = gridDim.x > row_blocks + col_blocks + heavy_blocks;
    }
    auto value = [&](int k) { return LATE ? Wd[flat[k]] : vals[k]; };
    if (blockIdx.x >= row_blocks + col_blocks) {
        const unsigned b = blockIdx.x - row_blocks - col_blocks;
        if (b < heavy_blocks) {
            heavy_fill_row((int)b, heavy, rowptr, flat, value, I, Hd);
        } else {
            const int64_t k = (int64_t)(b - heavy_blocks) * 256 + threadIdx.x;
            if (k < nnz) Wd[flat[k]] = vals[k];
        }
        return;
    }
    const bool col = blockIdx.x >= row_blocks;
    const int* __restrict__ perm = col ? perm_c : perm_r;
    uint2* __restrict__ ent = col ? ent_c : ent_r;
    const int64_t n4 = (int64_t)(col ? ptr_c[nseg_c] : ptr_r[nseg_r]) * (2 * OCT / 4);
    const int64_t stride = (int64_t)(col ? col_blocks : row_blocks) * 256;
    for (int64_t e = (int64_t)(blockIdx.x - (col ? row_blocks : 0u)) * 256 + threadIdx.x; e < n4; e += stride) {
        const int4 p = reinterpret_cast<const int4*>(perm)[e];
        uint2* d = ent + 4 * e;
        if (p.x >= 0) d[0].y = __float_as_uint(value(p.x));
        if (p.y >= 0) d[1].y = __float_as_uint(value(p.y));
        if (p.z >= 0) d[2].y = __float_as_uint(value(p.z));
        if (p.w >= 0) d[3].y = __float_as_uint(value(p.w));
    }
}

// dense_live: null where Wd is not the layer's own dense copy
__global__ void k_scatter_dense(const float* __restrict__ vals, const int* __restrict__ flat,
                                int64_t nnz, float* __restrict__ Wd, int* __restrict__ dense_live) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nnz) Wd[flat[k]] = vals[k];
    if (k == 0 && dense_live) *dense_live = 1;
}

// W . M as a dense array and the mask beside it (either may be null), one launch.  The first blocks own up to EXPORT_RUN
// positions each, `rows` whole rows or a part of one: the active values go to their places in a zeroed run of LDS and the run is written
// once, where a fill of the array with a scatter of single values behind it wrote every line twice.  The other blocks copy 4 KB of
// the mask each.  (Four layers of a GPT-2-small block, W and M: 72 us with a fill, a scatter and a copy for each, 30 like this; GPT-2-large: 91, 45.)
// A part of a long row finds its active positions by 256 samples of the row's, and a thread's next four are loaded together.  (Every
// part read all of its row's, one after the other, each value behind its position: 256 x 65535 full 204 us, now 44, a scatter 67; 32 x
// 65535 84, 8.4, 10.4; 4000 x 8193 full 175, 110, 125; 1280 x 5120 full 30, 21, 26; 3072 x 768 full 8.2, 5.6, 11.)
constexpr int EXPORT_RUN = 4096;
__global__ __launch_bounds__(256) void k_export_dense(const float* __restrict__ vals, const int* __restrict__ flat,
                                                      const int* __restrict__ rowptr, const uint8_t* __restrict__ mask,
                                                      int64_t nnz, int64_t N, int O, int I, int rows, int parts, int part, unsigned run_blocks,
                                                      float* __restrict__ W, uint8_t* __restrict__ M, int* __restrict__ dense_live) {
    __shared__ __attribute__((aligned(16))) float run[EXPORT_RUN];
    const int tid = threadIdx.x;
    if (blockIdx.x >= run_blocks) {
        const int64_t p = ((int64_t)(blockIdx.x - run_blocks) * 256 + tid) * 16;
        if (p + 16 <= N) *reinterpret_cast<uint4*>(M + p) = *reinterpret_cast<const uint4*>(mask + p);
        else for (int64_t i = p; i < N; ++i) M[i] = mask[i];
        return;
    }
    const int r = (int)(blockIdx.x / (unsigned)parts) * rows, r1 = min(r + rows, O), c0 = (int)(blockIdx.x % (unsigned)parts) * part;
    const int n = min((r1 - r) * I - c0, part);
    int k0 = nnz > 0 ? rowptr[r] : 0, k1 = nnz > 0 ? rowptr[r1] : 0;
    for (int i = 4 * tid; i < n; i += 1024) *reinterpret_cast<float4*>(run + i) = make_float4(0.f, 0.f, 0.f, 0.f);
    const int64_t base = (int64_t)r * I + c0;
    if (parts > 1 && k1 - k0 > 1024) {
        const int step = (k1 - k0 + 255) / 256, at = k0 + tid * step;
        const int64_t f = at < k1 ? (int64_t)flat[at] : (int64_t)1 << 32;
        const int before = __syncthreads_count(f < base), within = __syncthreads_count(f < base + n);
        k1 = min(k1, k0 + within * step);             // (sample `within` is the first one past the part, `before` the first one in it)
        k0 += max(before - 1, 0) * step;
    } else {
        __syncthreads();
    }
    if (k1 - k0 <= 256) {                             // (four each would be the same one four times: 3072 x 768 at 0.04 4.0 us, so 3.9)
        if (tid < k1 - k0) {
            const int64_t at = (int64_t)flat[k0 + tid] - base;
            const float v = vals[k0 + tid];
            if (at >= 0 && at < n) run[at] = v;
        }
        k0 = k1;
    }
    for (int k = k0 + tid; k < k1; k += 1024) {
        int64_t at[4];
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = min(k + 256 * u, k1 - 1);
            at[u] = (int64_t)flat[j] - base;
            v[u] = vals[j];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (at[u] >= 0 && at[u] < n) run[at[u]] = v[u];        // (the last one up to four times, the same value)
    }
    __syncthreads();
    const int n4 = (base & 3) == 0 ? n & ~3 : 0;
    for (int i = 4 * tid; i < n4; i += 1024) *reinterpret_cast<float4*>(W + base + i) = *reinterpret_cast<const float4*>(run + i);
    for (int i = n4 + tid; i < n; i += 256) W[base + i] = run[i];
    if (blockIdx.x == 0 && tid == 0 && dense_live) *dense_live = 1;
}

__global__ void k_fill_u32(uint32_t* __restrict__ dst, uint32_t value, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[k] = value;
}

__global__ void k_copy_i32(const int* __restrict__ src, int* __restrict__ dst, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[k] = src[k];
}

// ------------------------------------------------------------------ build

// out[j] = sum of in[0 .. j), out[n] = total; in == out is allowed
static int scan_excl_i32(const int* in, int* out, int64_t n, hipStream_t s) {
    Batch<ScanArgs, 1> b;
    b.add(ScanArgs{in, out, n}, 1);
    k_scan_excl<<<b.grid(), 1024, 0, s>>>(b);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

// Clears device memory with a kernel (safe to record into a HIP graph, unlike a memset node).
int fill_u32(void* dst, uint32_t value, int64_t n_words, hipStream_t s) {
    if (n_words <= 0) return MST_OK;
    k_fill_u32<<<(unsigned)cdiv(n_words, 256), 256, 0, s>>>((uint32_t*)dst, value, n_words);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

// Rebuilds vals / flat / rowptr and both views of the layers from their masks and dense weight arrays: counts per (row, sub-chunk)
// of both views -> ranking of every block's rows with the segments' lengths -> pointers of the octet segments (with the views'
// costs for the weight gradient) -> ordered compaction of the row views -> of the col views, which need the canonical
// indices that the row views' pass writes to ws.cidx.  Five launches for all layers and both views (eight per layer before);
// nothing is cleared beforehand: the count kernel writes the padding rows' zero counts and the fill kernels their own padding.
int build_views(const BuildItem* items, int n, hipStream_t s) {
    Batch<CountArgs> count;
    Batch<RankArgs> rank;
    Batch<PtrArgs> ptr;
    Batch<FillArgs> fill_r, fill_c;
    int nsub_max = 1, nchunk_max = 1;
    for (int x = 0; x < n; ++x) {
        mst_layer* L = items[x].L;
        const Workspace& ws = items[x].ws;
        L->views_valid = false;
        const View &r = L->row, &c = L->col;
        const int O = L->O, I = L->I, Rpad_r = r.NBpad * RB, Rpad_c = c.NBpad * RB;
        nsub_max = std::max(nsub_max, r.nsub());
        nchunk_max = std::max({nchunk_max, r.nchunk, c.nchunk});
        const int tiles = (int)cdiv(Rpad_c, MT_COLS);
        count.add(CountArgs{L->mask, O, I, r.KS, r.nsub(), Rpad_r, c.KS, Rpad_c, Rpad_r, tiles, ws.segcnt[0], ws.rowcnt, ws.segcnt[1]},
                  Rpad_r + (int64_t)tiles * c.nsub());
        auto view = [&](const View& v, int which) {
            return ViewArgs{ws.segcnt[which], v.msub, v.nchunk, v.NBpad * RB, v.NBpad, v.NB, v.nseg, v.rowmap, v.rowpos, ws.qlen[which], v.ptr};
        };
        const RankArgs views{view(r, 0), view(c, 1)};
        rank.add(views, r.NBpad + c.NBpad);
        ptr.add(PtrArgs{views, ws.rowcnt, L->rowptr, O, L->walk_cost, L->heavy_on ? L->heavy : nullptr, L->dense_live, items[x].keep_dense_copy ? 1 : 0}, 2);
        const int nrows = r.NB * RB, nparts = std::max(1, std::min(r.nsub(), 8192 / nrows));
        fill_r.add(FillArgs{L->mask, items[x].Wsrc, O, I, r.KS, r.msub, r.nsub(), r.NBpad, r.NB, Rpad_r, L->rowptr, r.ptr, r.rowpos, r.rowmap,
                            ws.segcnt[0], L->heavy_on ? L->heavy : nullptr, L->vals, L->flat, ws.cidx, r.perm, reinterpret_cast<uint2*>(r.ent),
                            nparts, (int)cdiv(r.nsub(), nparts), 0},
                   cdiv((int64_t)nrows * nparts, 4));
        const int ctiles = (int)cdiv(c.NB * RB, MT_COLS);
        fill_c.add(FillArgs{L->mask, items[x].Wsrc, O, I, c.KS, c.msub, c.nsub(), c.NBpad, c.NB, Rpad_c, nullptr, c.ptr, c.rowpos, c.rowmap,
                            ws.segcnt[1], nullptr, nullptr, nullptr, ws.cidx, c.perm, reinterpret_cast<uint2*>(c.ent), 0, 0, ctiles},
                   (int64_t)ctiles * c.nsub());
    }
    launch_batch(count, [&](const auto& b) { k_count<<<b.grid(), 256, (size_t)nsub_max * 4, s>>>(b); });
    MST_LAUNCH_CHECK();
    for (int x = 0; x < n; ++x)
        if (items[x].L->heavy_on) {
            const int rc = heavy_mark(items[x].L, items[x].ws, items[x].L->row.NBpad * RB, s);  // heavy rows leave the view
            if (rc != MST_OK) return rc;
        }
    launch_batch(rank, [&](const auto& b) { k_block_rank<<<b.grid(), RB, (size_t)nchunk_max * RB * 2, s>>>(b); });
    MST_LAUNCH_CHECK();
    launch_batch(ptr, [&](const auto& b) { k_view_ptr<<<b.grid(), 1024, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    launch_batch(fill_r, [&](const auto& b) { k_fill_row<<<b.grid(), 256, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    for (int x = 0; x < n; ++x)
        if (items[x].L->heavy_on) {
            const int rc = heavy_fill(items[x].L, s);
            if (rc != MST_OK) return rc;
        }
    launch_batch(fill_c, [&](const auto& b) { k_fill_col<<<b.grid(), 256, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    for (int x = 0; x < n; ++x) {
        mst_layer* L = items[x].L;
        L->views_valid = true;
        L->views_pending = L->row_stale = L->col_stale = false;
        if (!items[x].keep_dense_copy) L->Wd_valid = L->Wd_zeros = L->Wd_pending = L->planes_valid = L->pairs_valid = L->pairs_matched = false;
    }
    return MST_OK;
}

// vals / flat / rowptr alone (three launches): what layers served by the dense contractions need
int build_canonical(const BuildItem* items, int n, bool recording, hipStream_t s) {
    Batch<CanonicalArgs> seg;
    Batch<ScanArgs> scan;
    for (int x = 0; x < n; ++x) {
        mst_layer* L = items[x].L;
        int* const cnt = items[x].ws.segcnt[0];
        const int nseg = (int)cdiv(L->N, CSEG);
        L->views_valid = false;
        uint2* const runs = L->runs_kept(recording) && L->I % 32 == 0 ? L->runs : nullptr;
        seg.add(CanonicalArgs{L->mask, items[x].Wsrc, L->O, L->I, L->N, nseg, cnt, L->rowptr, L->flat, L->vals, runs}, cdiv(nseg, 4));
        scan.add(ScanArgs{cnt, cnt, nseg}, 1);
    }
    launch_batch(seg, [&](const auto& b) { k_count_seg<<<b.grid(), 256, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    launch_batch(scan, [&](const auto& b) { k_scan_excl<<<b.grid(), 1024, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    launch_batch(seg, [&](const auto& b) { k_fill_canonical<<<b.grid(), 256, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    for (int x = 0; x < n; ++x)
        if (items[x].L->runs_kept(recording) && items[x].L->I % 32 == 0) items[x].L->runs_valid = items[x].L->runs != nullptr;
    return MST_OK;
}

// Which of each 32 columns of a row are inactive, and the canonical index of the first active one: a wavefront per row, a lane per 32 positions.
struct RunArgs {
    const uint8_t* mask;
    const int* rowptr;
    uint2* runs;
    int O, I;
};
template <int CAP>
__global__ __launch_bounds__(256) void k_active_runs(const Batch<RunArgs, CAP> batch) {
    if (batch.surplus()) return;
    const RunArgs a = batch.entry();
    const int row = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= a.O) return;
    const uint8_t* const m = a.mask + (int64_t)row * a.I;
    const int words = (a.I + 31) / 32;
    int first = a.rowptr[row];
    for (int w0 = 0; w0 < words; w0 += 64) {
        const int w = w0 + lane;
        uint32_t bits = 0;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            if (32 * w + 8 * h >= a.I) continue;
            const uint2 u = *reinterpret_cast<const uint2*>(m + 32 * w + 8 * h);
            const uint32_t d[2] = {u.x, u.y};
#pragma unroll
            for (int e = 0; e < 8; ++e) bits |= ((d[e >> 2] >> (8 * (e & 3)) & 0xFFu) != 0u ? 1u : 0u) << (8 * h + e);
        }
        const int n = __popc(bits);
        int upto = n;
        for (int d = 1; d < 64; d <<= 1) {
            const int below = __shfl_up(upto, d, 64);
            if (lane >= d) upto += below;
        }
        if (w < words) a.runs[(int64_t)row * words + w] = make_uint2(~bits, (uint32_t)(first + upto - n));
        first += __shfl(upto, 63, 64);
    }
}
// (those that have them are left out; whether they are there is for the caller to say: behind the launch where it changes the mask, behind a wait
// where it is a product)
int make_runs(mst_layer* const* layers, int n, hipStream_t s) {
    Batch<RunArgs> batch;
    for (int x = 0; x < n; ++x) {
        const mst_layer* L = layers[x];
        if (!L->runs || L->runs_valid) continue;
        batch.add(RunArgs{L->mask, L->rowptr, L->runs, L->O, L->I}, cdiv(L->O, 4));
    }
    if (batch.n == 0) return MST_OK;
    launch_batch(batch, [&](const auto& b) { k_active_runs<<<b.grid(), 256, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    return MST_OK;
}

static ActiveRuns runs_of(const mst_layer* L) { return ActiveRuns{L->runs, (int)cdiv(L->I, 32), (uint32_t)(4 * L->nnz)}; }

// For a product that reads them.  Made by the product itself they are not there for other streams before it has waited for them,
// once behind an update that found them unread, and it says that they are there after the wait (two that meet, from two threads, each make
// them: the same bits); a recording cannot wait and leaves them.
int active_runs(ActiveOut* active, hipStream_t s, ActiveRuns& runs, int64_t& stride) {
    if (!active) return MST_OK;
    mst_layer* L = const_cast<mst_layer*>(active->L);        // a cache of the mask, not layer state
    if (!L->runs || L->runs_missed || L->nnz == 0) return MST_OK;
    // Small layers with many active weights stay on whole outputs: their planes stay in the caches, and the gather of them takes what the stores
    // of single values take more.  Whole and a gather, active positions alone (us): bfloat16, 1288 x 1040, 3000 tokens, densities 0.2, 0.5, 0.9:
    // 30.7 and 30.4, 31.1 and 32.6, 32.0 and 34.1; 768 x 2304, 4096 tokens: 36.9 and 31.5, 37.7 and 34.0, 39.1 and 38.0.  fp32 loses less by it:
    // the first 67.0 and 63.6, 66.6 and 64.7, 67.1 and 65.8; 768 x 768, 8192 tokens, at 0.9: 53.2 and 53.8.  Above the line 4096 x 1024, 4096
    // tokens, at 0.5 and 0.9: bfloat16 51.1 and 46.2, 53.4 and 51.4, fp32 103 and 97, 106 and 104.
    if (4 * L->nnz > L->N && L->N < (int64_t)1 << 21) return MST_OK;
    bool recording = false;
    if (!L->runs_valid || !L->runs_recorded) {
        const int rc = stream_recording(s, &recording);
        if (rc != MST_OK) return rc;
    }
    if (!L->runs_valid) {
        if (recording) return MST_OK;
        const int rc = make_runs(&L, 1, s);
        if (rc != MST_OK) return rc;
        MST_HIP(hipStreamSynchronize(s));
        L->runs_valid = true;
    }
    L->runs_recorded |= recording;
    L->runs_unread = 0;
    runs = runs_of(L);
    active->stride = stride = (int64_t)align_up((size_t)L->nnz, 4);
    active->done = true;
    return MST_OK;
}

// W . M to W and / or the mask to M (dense_live: null where W is not the layer's own dense copy)
static int export_dense(const mst_layer* L, float* W, uint8_t* M, int* dense_live, hipStream_t s) {
    // Rows of a run: one, several where a layer has far more rows than the chip holds blocks, then whole fours so that runs begin on 16 bytes
    const int parts = (int)cdiv(L->I, EXPORT_RUN);
    int rows = std::max(1, std::min(EXPORT_RUN / L->I, L->O / 1024));
    if (rows >= 4) rows &= ~3;
    const int part = parts > 1 ? (int)(cdiv(cdiv(L->I, parts), 4) * 4) : EXPORT_RUN;
    const unsigned run_blocks = W ? (unsigned)(cdiv(L->O, rows) * parts) : 0u, mask_blocks = M ? (unsigned)cdiv(L->N, 4096) : 0u;
    if (run_blocks + mask_blocks == 0) return MST_OK;
    k_export_dense<<<run_blocks + mask_blocks, 256, 0, s>>>(L->vals, L->flat, L->rowptr, L->mask, L->nnz, L->N, L->O, L->I, rows, parts, part,
                                                            run_blocks, W, M, dense_live);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

static int refresh_dense_copy(mst_layer* L, bool recording, hipStream_t s) {
    if (!L->Wd_zeros || L->Wd_pending) {
        const int rc = export_dense(L, L->Wd, nullptr, L->dense_live, s);
        if (rc != MST_OK) return rc;
    } else if (L->nnz > 0) {                         // the active set is unchanged since the last time: only values move
        k_scatter_dense<<<(unsigned)cdiv(L->nnz, 256), 256, 0, s>>>(L->vals, L->flat, L->nnz, L->Wd, L->dense_live);
        MST_LAUNCH_CHECK();
    }
    L->Wd_valid = L->Wd_zeros = true;
    L->Wd_pending = recording;
    L->planes_valid = L->pairs_valid = false;
    const bool planes = L->planes_kept(), pairs = L->pairs_recorded;
    if (!planes && !pairs) return MST_OK;
    int rc = planes ? make_planes(L, s) : MST_OK;    // (recorded products read them without asking)
    if (rc == MST_OK && pairs) rc = make_pairs(L, s);
    return rc == MST_OK ? weights_made(L, planes, pairs, s) : rc;
}

// refreshed: it was out of date, or formed by a recording
int ensure_dense_copy(mst_layer* L, hipStream_t s, bool* refreshed) {
    *refreshed = false;
    if (L->Wd_valid && !L->Wd_pending) return MST_OK;
    bool recording;
    const int rc = stream_recording(s, &recording);
    if (rc != MST_OK || (L->Wd_valid && recording)) return rc;
    *refreshed = true;
    return refresh_dense_copy(L, recording, s);
}

// The planes of Wd (its packed pairs) were made on s, by a product and not by the hand-over or the update that changed the
// weights.  Products on other streams are ordered after those and not after this call, so it waits before it says that they are
// there (and where the pairs are of a mask that nothing is known of, it learns how even that is).  A recording cannot wait and
// runs later or never: it says nothing about them.
int weights_made(mst_layer* L, bool planes, bool pairs, hipStream_t s) {
    bool recording;
    int rc = stream_recording(s, &recording);
    if (rc != MST_OK || recording) return rc;
    if (pairs && !L->pairs_measured) {
        rc = measure_pairs(L, s);
        if (rc != MST_OK) return rc;
    } else {
        MST_HIP(hipStreamSynchronize(s));
    }
    L->planes_valid |= planes;
    L->pairs_valid |= pairs && !L->pairs_missed;
    L->pairs_matched |= pairs;
    return MST_OK;
}

// new values into the entries of the row view (and the dense rows beside it) and / or of the col view, and into
// a dense copy that is zero at every inactive position: one launch.  late: the entries take the dense copy's values
static int refresh_views(const mst_layer* L, bool row, bool col, bool dense, bool late, hipStream_t s) {
    if (L->nnz == 0 || (!row && !col && !dense)) return MST_OK;
    const View &r = L->row, &c = L->col;
    // about 1.5 slots per entry, four slots per thread; the kernel strides over whatever there is
    const unsigned nb = (unsigned)std::min<int64_t>(cdiv(L->nnz * 3 / 2 + 1, 1024), 4096);
    const unsigned rb = row ? nb : 0u, cb = col ? nb : 0u;
    const unsigned hb = row && L->heavy_on ? HEAVY_MAX : 0u, db = dense ? (unsigned)cdiv(L->nnz, 256) : 0u;
    const auto kernel = late ? k_sync_views<true> : k_sync_views<false>;
    kernel<<<rb + cb + hb + db, 256, 0, s>>>(
        L->vals, rb, cb, r.ptr, r.nseg, r.perm, reinterpret_cast<uint2*>(r.ent), c.ptr, c.nseg, c.perm,
        reinterpret_cast<uint2*>(c.ent), L->heavy, L->rowptr, L->flat, L->I, L->Hd, hb, L->Wd, L->nnz, L->dense_live);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

// A product is about to walk these (built) views: entries that missed a hand-over take it now, once in a layer's
// life.  They take what was handed over last, not what vals[] holds by now.  Products on other streams are ordered after mst_layer_sync_values, not after this
// call, so it waits for the new entries before it says that they are there.  A recording cannot wait and runs
// later or never: it takes the refresh with it and leaves the view stale for whoever walks it first.
int ensure_fresh(const mst_layer* Lc, bool row, bool col, hipStream_t s) {
    mst_layer* L = const_cast<mst_layer*>(Lc);       // caches of vals[], not layer state
    if (row) L->row_walked = true;
    if (col) L->col_walked = true;
    row = row && L->row_stale;
    col = col && L->col_stale;
    if (!row && !col) return MST_OK;
    int rc = refresh_views(L, row, col, false, true, s);
    bool recording = false;
    if (rc == MST_OK) rc = stream_recording(s, &recording);
    if (rc != MST_OK || recording) return rc;
    MST_HIP(hipStreamSynchronize(s));
    if (row) L->row_stale = false;
    if (col) L->col_stale = false;
    return MST_OK;
}

// The views of a layer whose last update left them unbuilt, from the mask and the dense copy.
int ensure_views(const mst_layer* Lc, const Workspace& ws, hipStream_t s) {
    bool there, refreshed;
    int rc = views_there(Lc, s, &there);
    if (rc != MST_OK || there) return rc;
    mst_layer* L = const_cast<mst_layer*>(Lc);       // a cache of (mask, vals), not layer state
    rc = ensure_dense_copy(L, s, &refreshed);
    if (rc != MST_OK) return rc;
    const BuildItem item{L, L->Wd, ws, true};
    rc = build_views(&item, 1, s);
    if (rc != MST_OK) return rc;
    return stream_recording(s, &L->views_pending);
}

// Can a call on s walk the views?
int views_there(const mst_layer* L, hipStream_t s, bool* there) {
    *there = L->views_valid;
    if (!L->views_valid || !L->views_pending) return MST_OK;
    return stream_recording(s, there);
}

// After an update: will a sparse kernel walk the views?  Judged at the batch size and type of
// the last product call; a layer that has seen none yet, or is pinned to the sparse kernels, says yes.  Y and dX are
// judged together: both views are built or none, and where only one of the two gains by less than the other loses
// the views are not worth their build.
bool views_wanted(const mst_layer* L) {
    if (L->path == MST_PATH_SPARSE) return true;
    if (L->path == MST_PATH_DENSE) return false;
    if (L->hint_T <= 0) return true;
    const mst_dtype act = (mst_dtype)L->hint_act;
    const int T = L->hint_T;
    const bool y = use_dense_path(L, WALK_FWD, act, T), dx = use_dense_path(L, WALK_BWD_INPUT, act, T);
    const bool both = y == dx ? y : walk_us(L, WALK_FWD, T) + walk_us(L, WALK_BWD_INPUT, T) >
                                        dense_us(L, WALK_FWD, act, T) + dense_us(L, WALK_BWD_INPUT, act, T);
    return !(both && use_dense_weight_grad(L, act, T));
}

}  // namespace mst

using namespace mst;

extern "C" {

int mst_last_hip_error(void) { return g_last_hip_error; }

size_t mst_layer_device_bytes(int O, int I, int64_t nnz_capacity) {
    if (!shape_ok(O, I, nnz_capacity)) return 0;
    return carve_layer(O, I, nnz_capacity).total;
}

size_t mst_workspace_bytes(int O, int I, int64_t nnz_capacity, int T) {
    if (!shape_ok(O, I, nnz_capacity) || T < 1) return 0;
    return carve_workspace(nullptr, O, I, nnz_capacity, T).total;
}

int mst_layer_create(mst_layer_t** out, int O, int I, int64_t nnz_capacity, void* buf_dev,
                     size_t buf_bytes) {
    if (!out || !buf_dev || !aligned16(buf_dev)) return MST_ERR_ARG;
    if (!shape_ok(O, I, nnz_capacity)) return MST_ERR_SHAPE;
    const LayerCarve c = carve_layer(O, I, nnz_capacity);
    if (buf_bytes < c.total) return MST_ERR_WORKSPACE;
    mst_layer* L = new (std::nothrow) mst_layer();
    if (!L) return MST_ERR_STATE;
    char* b = static_cast<char*>(buf_dev);
    L->O = O; L->I = I; L->N = (int64_t)O * I; L->cap = nnz_capacity; L->nnz = 0;
    L->buf = buf_dev; L->buf_bytes = buf_bytes;
    L->mask = (uint8_t*)(b + c.mask);
    L->vals = (float*)(b + c.vals);
    L->flat = (int*)(b + c.flat);
    L->rowptr = (int*)(b + c.rowptr);
    L->Wd = (float*)(b + c.Wd);
    L->walk_cost = (unsigned long long*)(b + c.cost);
    L->dense_live = (int*)(b + c.cost + 16);
    L->heavy = (int*)(b + c.heavy);
    L->Hd = (float*)(b + c.Hd);
    if (has_runs(O, I)) L->runs = (uint2*)(b + c.runs);
    if (has_pairs(O, I)) {
        L->pairs_y = pairs_view(b + c.sy, O, I);
        L->pairs_x = pairs_view(b + c.sx, I, O);
    }
    if (has_planes(O, I)) {
        L->planes_y = (uint16_t*)(b + c.py);
        L->planes_x = (uint16_t*)(b + c.px);
    }
    auto init_view = [&](View& v, int R, int K, size_t optr, size_t oent, size_t operm, size_t omap, size_t opos) {
        v = view_shape(R, K, nnz_capacity);
        v.ptr = (int*)(b + optr); v.ent = (uint4*)(b + oent); v.perm = (int*)(b + operm);
        v.rowmap = (int*)(b + omap); v.rowpos = (int*)(b + opos);
    };
    init_view(L->row, O, I, c.rptr, c.rent, c.rperm, c.rmap, c.rpos);
    init_view(L->col, I, O, c.cptr, c.cent, c.cperm, c.cmap, c.cpos);
    *out = L;
    return MST_OK;
}

int mst_layer_destroy(mst_layer_t* layer) {
    delete layer;
    return MST_OK;
}

int mst_layer_load_dense(mst_layer_t* L, const float* W_dev, const uint8_t* M_dev, void* ws_dev,
                         size_t ws_bytes, mst_stream_t stream) {
    if (!L || !W_dev || !M_dev || !ws_dev || !aligned16(W_dev) || !aligned16(M_dev) || !aligned16(ws_dev))
        return MST_ERR_ARG;
    const Workspace ws = carve_workspace(ws_dev, L->O, L->I, L->cap, 1);
    if (ws_bytes < ws.total) return MST_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    // learn the active count first so that nothing is written when it does not fit
    Batch<CountArgs> count;
    count.add(CountArgs{M_dev, L->O, L->I, L->row.KS, L->row.nsub(), 0, 0, 0, L->O, 1, nullptr, ws.rowcnt, nullptr}, L->O);
    launch_batch(count, [&](const auto& b) { k_count<<<b.grid(), 256, (size_t)L->row.nsub() * 4, s>>>(b); });
    MST_LAUNCH_CHECK();
    int rcs = scan_excl_i32(ws.rowcnt, L->rowptr, L->O, s);          // rebuilt below anyway
    if (rcs != MST_OK) return rcs;
    int total = 0;
    MST_HIP(hipMemcpyAsync(&total, L->rowptr + L->O, 4, hipMemcpyDeviceToHost, s));
    MST_HIP(hipStreamSynchronize(s));
    if ((int64_t)total > L->cap) return MST_ERR_STATE;
    MST_HIP(hipMemcpyAsync(L->mask, M_dev, (size_t)L->N, hipMemcpyDeviceToDevice, s));
    L->nnz = total;
    L->pairs_unknown();
    L->choice.store(0, std::memory_order_relaxed);
    L->built = false;                                   // a failed rebuild leaves no usable layer
    L->runs_valid = false;
    // Heavy rows (heavy.hip).  The dense pass costs a launch after every sparse forward, a read of
    // X and T scattered stores per heavy row: a layer of less than 2^20 positions does not earn
    // that back (measured: 768 x 768 at T = 16384 loses 10 us, 768 x 2304 gains 19 us), and a layer
    // whose loaded mask has no heavy row (every uniformly random mask) should not pay the launch.
    // So the rule is tried on this first build of a large layer and kept for the layer's lifetime
    // only if it found rows; the forced mode of the hook keeps it for every layer.
    const int mode = heavy_rows_mode();
    L->heavy_on = mode == 2 || (mode == 1 && L->N >= ((int64_t)1 << 20));
    const BuildItem item{L, W_dev, ws, false};
    const int rc = build_views(&item, 1, s);
    if (rc != MST_OK) return rc;
    if (L->heavy_on && mode == 1) {
        int found = 0;
        MST_HIP(hipMemcpyAsync(&found, L->heavy, 4, hipMemcpyDeviceToHost, s));
        MST_HIP(hipStreamSynchronize(s));
        L->heavy_on = found > 0;
    }
    const int rcr = make_runs(&L, 1, s);
    if (rcr != MST_OK) return rcr;
    L->runs_valid = L->runs != nullptr;
    L->built = true;
    return MST_OK;
}

int mst_layer_export_dense(const mst_layer_t* L, float* W_dev, uint8_t* M_dev, mst_stream_t stream) {
    if (!L) return MST_ERR_ARG;
    if ((W_dev && !aligned16(W_dev)) || (M_dev && !aligned16(M_dev))) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    return export_dense(L, W_dev, M_dev, nullptr, (hipStream_t)stream);
}

int mst_layer_values(mst_layer_t* L, float** vals_dev, int64_t* nnz) {
    if (!L) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    if (vals_dev) *vals_dev = L->vals;
    if (nnz) *nnz = L->nnz;
    return MST_OK;
}

int mst_layer_sync_values(mst_layer_t* L, mst_stream_t stream) {
    if (!L) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    hipStream_t s = (hipStream_t)stream;
    // A dense copy that is in use (zero at every inactive position) takes the new values now rather
    // than at the next product, so that products recorded into a graph never see stale weights.
    const bool dense = L->Wd_zeros && L->nnz > 0, views = L->nnz > 0 && L->views_valid;   // unbuilt views take the values when they are built
    L->Wd_valid = dense;
    bool row = views, col = views, planes = dense && L->planes_valid, pairs = dense && L->pairs_valid && pairs_kept(L);
    L->planes_valid = planes;
    L->pairs_valid = pairs;
    bool recording = false;
    if (dense && (L->planes_y || L->pairs_y.blocks || (views && !(L->row_walked && L->col_walked)))) {
        // Views that nothing has walked are left out, since the dense copy holds the values for their first walk.
        // A recording refreshes every built view and changes no flag of theirs: its replays come at any time, between
        // calls that walk a view for the first time, and it has not run yet.  It takes the planes along if a product has read them
        // or the last product call had bfloat16 activations that did not go to the packed pairs, in both directions; otherwise they count as missed.
        // (Recorded regardless, a replayed fp32 step of the GPT-2-small block took 1.217 ms instead of 1.194.)
        const int rcr = stream_recording(s, &recording);
        if (rcr != MST_OK) return rcr;
        if (recording) {
            // (the packed pairs if products read them)
            pairs = pairs_kept(L);
            L->pairs_missed |= L->pairs_y.blocks && !pairs;
            planes = !L->planes_missed && (L->planes_used || (L->planes_y && L->hint_act == MST_BF16 && !(pairs && pairs_wanted(L, true))));
            L->planes_missed |= L->planes_y && !planes;
        } else {
            if (views) {
                row = L->row_walked;
                col = L->col_walked;
                L->row_stale |= !row;
                L->col_stale |= !col;
            }
            L->pairs_unread += pairs && L->pairs_unread < mst_layer::PAIRS_UNREAD;
        }
    }
    // (the packing brings the values to the dense copy itself where it can; a view's entries before it, since they say that the dense copy is out of use)
    const bool with_pairs = pairs && L->runs_valid && !L->runs_missed;
    const int rc = refresh_views(L, row, col, dense && !with_pairs, false, s);
    // (made again from the dense copy: 8.5 us at 1024 x 4096.  Scattering 5 % of the positions into them took 11, 10 % of 1280 x
    // 5120 took 30: four stores of two bytes per value, two of them far apart.)
    if (rc != MST_OK) return rc;
    if (with_pairs) {
        L->runs_recorded |= recording;
        L->runs_unread = 0;
        const ActiveRuns words = runs_of(L);
        const int rcw = make_pairs(L, s, &words);
        if (rcw != MST_OK) return rcw;
        pairs = false;
    }
    const int rcp = planes ? make_planes(L, s) : MST_OK;
    return rcp == MST_OK && pairs ? make_pairs(L, s) : rcp;
}

int mst_layer_indices(const mst_layer_t* L, int32_t* flat_dev, mst_stream_t stream) {
    if (!L || !flat_dev) return MST_ERR_ARG;
    if (!L->built) return MST_ERR_STATE;
    if (L->nnz == 0) return MST_OK;
    k_copy_i32<<<(unsigned)cdiv(L->nnz, 256), 256, 0, (hipStream_t)stream>>>(L->flat, flat_dev, L->nnz);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

int mst_layer_set_path(mst_layer_t* L, mst_path path) {
    if (!L || path < MST_PATH_AUTO || path > MST_PATH_DENSE) return MST_ERR_ARG;
    L->path = path;
    return MST_OK;
}

int mst_layer_set_prune_lambda(mst_layer_t* L, float lambda) {
    if (!L || !(lambda >= 0.f) || lambda > 3.4028234e38f) return MST_ERR_ARG;
    L->prune_lambda = lambda;
    return MST_OK;
}

int64_t mst_layer_nnz(const mst_layer_t* L) { return L ? L->nnz : -1; }

}  // extern "C"
