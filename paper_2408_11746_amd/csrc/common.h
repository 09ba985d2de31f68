// Internal declarations shared by the translation units of libmst_hip.so.
#pragma once

#include <algorithm>
#include <atomic>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/mst.h"

namespace mst {

// ---- tiling constants shared by the format builder and the product kernels ----
// The contraction dimension of a view is cut into equal chunks of at most KCMAX indices; one chunk
// of the dense operand for WT tokens (160 KB at most: the whole LDS of a CU) is what a workgroup
// stages at a time.
constexpr int KCMAX = 640;       // contraction indices per chunk, at most
constexpr int KSMAX = 128;       // ... and per sub-chunk, the unit in which the format builder counts
constexpr int WT = 64;           // tokens per LDS tile
constexpr int OCT = 8;           // rows per octet: one per lane group of eight lanes
constexpr int OPB = 16;          // octets per row block: one per wavefront of a workgroup
constexpr int RB = OCT * OPB;    // rows per row block
constexpr int MAX_WG_BLOCKS = 6; // most row blocks one workgroup may own (checked at every launch shape, walk_launch.h)
constexpr int SPREAD_FLAG = 1 << 30;   // in rowmap / rowpos: the octet holds ONE row spread over its eight lane groups
constexpr int HEAVY_MAX = 64;    // rows a layer may keep out of its row view as a small dense matrix (heavy.hip)
constexpr int PAIR_TAIL = 16;    // readable step pairs past the last one (a whole entry batch may be fetched there)

// LDS tile layout: row k (one contraction index) holds WT tokens = 256 bytes as 16 slots of four
// consecutive tokens; slot u of tokens 4u .. 4u+3 sits at byte (u ^ ((k >> 2) & 3)) * 16.  A 16-byte
// LDS read is served in sets of four lane quads, {0, 3, 5, 6} and {1, 2, 4, 7} of every 32 lanes,
// and is free of conflicts when the four quads of a set read four different 64-byte quarters of a
// row: the swizzle therefore stays inside a quarter (with a swizzle over eight slots the walk
// counted 3 conflict cycles per read); it spreads the transposing stores that stage the walk's tile.
__host__ __device__ inline uint32_t lds_off(uint32_t k) { return (k << 8) | (((k >> 2) & 3u) << 4); }

// Sparse matrix S [R x K] as the product kernels walk it.  Rows are grouped in blocks of
// RB = 128 consecutive rows.  Inside a block every row has a place; the row of place 8o + g
// belongs to octet o and lane group g.  The places are ranks by the rows' total length (longest
// first, lower index first on ties), or, where that takes fewer pairs, come from halving the block
// by the lengths in parts of the chunks (k_block_rank): the eight rows of an octet have similar
// lengths, in every chunk (little ELL padding even when row lengths are very uneven).
// rowmap[128b + place] is that row.  For every
// (chunk c of K, block b, octet o) the eight rows' entries inside the chunk are stored side
// by side, padded with zero-weight entries to the longest of the eight and to an even
// count (an ELL slice of height 8): step j of the octet holds one entry per lane group.
// Two steps form a pair = uint4[8]: element g is {off_j, w_j, off_j+1, w_j+1} of lane
// group g, off = lds_off(k - c*KC), w = fp32 bits.
// A very long row can take a whole octet ("spread"): its entries are dealt to the eight lane
// groups in turn (entry j of a chunk: lane group j & 7, step j >> 3), the kernels add the
// eight lane groups' sums at the end.  The other seven places of such an octet are given to
// seven EMPTY rows of the block (they own the output positions, which receive zero), so a
// block spreads at most as many rows as it has sevens of empty rows.  All eight rowmap
// entries of a spread octet and the rowpos entry of the spread row carry SPREAD_FLAG.
struct View {
    int R = 0, K = 0, nchunk = 0;
    int KC = 0;            // indices per chunk: msub * KS
    int KS = 0, msub = 0;  // indices per sub-chunk (a multiple of 4), sub-chunks per chunk
    int NB = 0;            // row blocks: ceil(R / 128)
    int NBpad = 0;         // block stride of ptr: NB + MAX_WG_BLOCKS (the extra blocks stay empty)
    int64_t nseg = 0;      // nchunk * NBpad * 16 octet segments
    int64_t cap_pairs = 0; // pairs the arrays can hold (incl. tail)
    int* ptr = nullptr;    // [nseg + 1] first pair of segment (c*NBpad + b)*16 + o
    uint4* ent = nullptr;  // [cap_pairs * 8]
    int* perm = nullptr;   // [cap_pairs * 16] canonical index of entry slot (pair*8 + g)*2 + half, -1 = padding
    int* rowmap = nullptr; // [NBpad * 128] place inside the block -> row (identity in the empty blocks)
    int* rowpos = nullptr; // [NBpad * 128] row -> place inside its block
    int nsub() const { return nchunk * msub; }
};

// S [R x K] as the products on the sparse matrix instructions read it (gemm_pairs.hip): bands of 256 rows, steps of 64 k
struct PairsView {
    int R = 0, K = 0, nk = 0, bands = 0;
    uint16_t* slots = nullptr; // [band][step][32] where the k pairs (2 p, 2 p + 1) of a step go in LDS
    uint32_t* flags = nullptr; // [band][step] a byte per two tiles of 32 rows: 1 if one of them has second weights
    uint8_t* over = nullptr;   // [band][step] 1: by the mask some row has second weights
    uint32_t* count = nullptr; // [2] (the row view's) how many of those there are in either view
    char* blocks = nullptr;    // [band][2 nk] packed tiles of the steps, then those of the third and fourth weights among four k
    uint32_t* sel = nullptr;   // [band][2 nk] their selectors
    size_t bytes = 0;
};
// Hd row j = row heavy[1 + j] of W . M, from the canonical arrays, by one block (heavy rows, heavy.hip);
// value(k) = the k-th active weight.  Every thread of the block must call it; j at or past the count does nothing.
template <typename F>
__device__ inline void heavy_fill_row(int j, const int* __restrict__ heavy, const int* __restrict__ rowptr,
                                      const int* __restrict__ flat, F&& value, int I, float* __restrict__ Hd) {
    if (j >= min(heavy[0], HEAVY_MAX)) return;
    const int h = heavy[1 + j];
    float* row = Hd + (int64_t)j * I;
    for (int i = threadIdx.x; i < I; i += blockDim.x) row[i] = 0.f;
    __syncthreads();
    const int k1 = rowptr[h + 1];
    for (int k = rowptr[h] + threadIdx.x; k < k1; k += blockDim.x) row[flat[k] - h * I] = value(k);
}

}  // namespace mst

struct mst_layer {
    int O = 0, I = 0;
    int64_t N = 0, cap = 0, nnz = 0;
    bool built = false;        // the device arrays are meaningful only after mst_layer_load_dense has succeeded
    int path = MST_PATH_AUTO;
    float prune_lambda = 0.f;  // prune score |w| + prune_lambda |grad| (0: magnitude only)
    void* buf = nullptr;
    size_t buf_bytes = 0;
    uint8_t* mask = nullptr;   // [N]
    float* vals = nullptr;     // [cap] canonical (ascending flat index) values
    int* flat = nullptr;       // [cap] canonical flat indices
    int* rowptr = nullptr;     // [O + 1] canonical CSR row pointers
    float* Wd = nullptr;       // [N] dense W . M, maintained only while the dense path is in use
    bool Wd_valid = false;     // Wd equals W . M
    bool Wd_zeros = false;     // Wd is zero at every inactive position (survives a change of the values)
    bool Wd_pending = false;   // ... but it was formed by a recording, which may not have run yet: eager calls form it anew
    // The two bfloat16 parts of Wd in the order that the products of bfloat16 activations want (gemm_planes.hip), for Y and for
    // dX; null where no such product has whole tiles.  Made by the first product that reads them, kept up with Wd from then on:
    // sync_values and the updates that leave Wd valid make them again.  A hand-over that was recorded while the layer
    // worked on fp32 activations does not carry their making, and its replays leave them behind at times
    // that the host does not see: products of bfloat16 activations then make them each for itself.
    uint16_t *planes_y = nullptr, *planes_x = nullptr;
    bool planes_used = false;  // some product has read them
    bool planes_missed = false;  // a hand-over without them has been recorded
    bool planes_valid = false; // they hold the parts of Wd
    bool planes_kept() const { return planes_used && !planes_missed; }
    // The packed weights of Y and dX on the sparse matrix instructions: made by the first product that reads them, kept up with Wd while
    // products do.  A hand-over makes them again unless the last PAIRS_UNREAD of them did so for nobody (another batch size, a mask
    // that turned out uneven), an update where the products that came last would read them at its density.  (No layer of
    // another shape has them: blocks null.)
    mst::PairsView pairs_y, pairs_x;
    static constexpr int PAIRS_UNREAD = 8;
    int pairs_unread = PAIRS_UNREAD;             // hand-overs since a product read them
    bool pairs_missed = false, pairs_valid = false;      // as those of the planes (missed: products make them each for itself)
    // A recorded product reads them without making them.  Its replays come when they like, so they are made whenever Wd changes, at any density.
    bool pairs_recorded = false;
    bool pairs_matched = false;    // their slots were chosen for the present active set
    // Y, dX: share of the steps with a second one, against that of a uniform mask, and whether it was measured on the present mask.  A loading
    // makes it unknown, so does an update behind PAIRS_CALLS products (pairs_calls: those since the last measurement).
    float pairs_skew[2] = {0.f, 0.f};
    bool pairs_measured = false;
    int pairs_calls = 0;
    void pairs_unknown() { pairs_skew[0] = pairs_skew[1] = 0.f; pairs_measured = false; }
    // The index views are built lazily: an update of a layer that the dense contractions serve
    // (path choice at the batch size and type of the last product call) leaves them unbuilt; a
    // call that needs them and has a workspace builds them, one without runs the dense product.
    bool views_valid = false;
    bool views_pending = false;    // ... but they were built by a recording, which may not have run yet: eager calls treat them as unbuilt
    // While a dense copy is in use mst_layer_sync_values refreshes the entries of a built view only if a product
    // has ever walked that view of the layer (recorded products included: recording is a call, and its replays
    // outlive rebuilt views); the entries of the others are stale and take the dense copy's values before their
    // first walk.  Same for the dense rows beside the row view.  (A layer on the dense contractions would spend
    // 50 us a step on them.)
    bool row_walked = false, col_walked = false;
    bool row_stale = false, col_stale = false;
    int* dense_live = nullptr; // device: Wd holds the values handed over last (0: every built view holds them)
    int hint_T = 0;            // batch size and activation type of the last product call (0: none yet)
    int hint_act = 0;
    // Which of every 32 columns are active and where they lie in vals (see active.h), for layers with rows of whole eights (null: none).  Made when
    // the layer is loaded; an update makes them again if a product or a hand-over has read them, unless the last RUNS_UNREAD updates did so for
    // nobody (the ultra-sparse phase walks; they are 2 us of an update of the four layers of a GPT-2-small block, 7 to 10 of a
    // GPT-2-large one), and always once a recording has read them, since its replays do so without asking.  Otherwise the next product does.
    uint2* runs = nullptr;
    bool runs_valid = false, runs_recorded = false;
    bool runs_missed = false;  // an update without them has been recorded: its replays leave them behind, products do without
    static constexpr int RUNS_UNREAD = 8;
    int runs_unread = -1;                        // updates since something read them (-1: nothing has)
    bool runs_kept(bool recording) const { return runs_recorded || (runs_unread >= 0 && (recording || runs_unread < RUNS_UNREAD)); }
    std::atomic<uint64_t> choice{0};   // sparse-or-dense choices at the last batch size and type (see remembered(); 0: none)
    mst::View row;             // S = W   [O x I], used by fwd (and bwd_weight)
    mst::View col;             // S = W^T [I x O], used by bwd_input
    unsigned long long* walk_cost = nullptr;   // device: cost of the row and of the col view for bwd_weight (k_view_ptr)
    // Heavy rows (see heavy.hip): device list [0] = count, [1 + j] = row; Hd [HEAVY_MAX x I] their dense weights.
    // Both follow the views: written when they are built, Hd again whenever the values change.
    int* heavy = nullptr;
    float* Hd = nullptr;
    bool heavy_on = false;     // the rule applies to this layer (decided when it is loaded)
};

namespace mst {

extern thread_local int g_last_hip_error;

#define MST_HIP(call)                                                     \
    do {                                                                  \
        hipError_t e__ = (call);                                          \
        if (e__ != hipSuccess) {                                          \
            mst::g_last_hip_error = (int)e__;                             \
            return MST_ERR_HIP;                                           \
        }                                                                 \
    } while (0)

#define MST_LAUNCH_CHECK() MST_HIP(hipGetLastError())

// Is s being recorded into a graph?  (The null stream cannot be.  Asked for it as well, the first product of a layer took 0.7 us
// more of the host: 3072 x 768, 64 tokens, 27.1 us until its end, so 28.)
inline int stream_recording(hipStream_t s, bool* recording) {
    *recording = false;
    if (s == nullptr) return MST_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    MST_HIP(hipStreamIsCapturing(s, &capture));
    *recording = capture != hipStreamCaptureStatusNone;
    return MST_OK;
}

// More than 64 KB of LDS has to be asked for, once per kernel and device (`done`: a bit per device; two
// threads that meet here repeat the call).  The kernels that ask take the dynamic array alone, and the walk
// reads it from LDS address 0: a kernel with static LDS in front of it is refused.
inline int allow_lds(const void* kernel, int bytes, uint64_t& done) {
    int dev = 0;
    MST_HIP(hipGetDevice(&dev));
    const uint64_t bit = 1ull << (dev & 63);
    if (__atomic_load_n(&done, __ATOMIC_RELAXED) & bit) return MST_OK;
    hipFuncAttributes attr;
    MST_HIP(hipFuncGetAttributes(&attr, kernel));
    if (attr.sharedSizeBytes != 0) return MST_ERR_STATE;
    MST_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    __atomic_fetch_or(&done, bit, __ATOMIC_RELAXED);
    return MST_OK;
}

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }
inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// true when a layer of this density should run the masked dense MFMA kernels (`job`: the product)
enum WalkJob { WALK_FWD = 0, WALK_BWD_INPUT, WALK_BWD_WEIGHT, WALK_BWD };
bool use_dense_path(const mst_layer* L, WalkJob job, mst_dtype act, int T);
bool use_dense_weight_grad(const mst_layer* L, mst_dtype act, int T);
bool use_fused_backward(const mst_layer* L, mst_dtype act, int T);
bool use_sparse_input_grad(const mst_layer* L, mst_dtype act, int T);
// ... and the dense kernels take fp32 operands in full there
bool full_precision(const mst_layer* L, WalkJob job, mst_dtype act, int T);

// ---- workspace carving (one place so that mst_workspace_bytes and the users agree) ----
struct Workspace {
    float* G = nullptr;        // [N] dense gradient (mst_mask_update)
    float* Wd = nullptr;       // [N] dense scratch of the weights during a rebuild
    int* cidx = nullptr;       // [N] canonical index of each active position
    uint8_t* sel = nullptr;    // [N] selection flags of the grow step
    uint8_t* psel = nullptr;   // [cap] selection flags of the prune step
    int* segcnt[2] = {nullptr, nullptr};   // active count per (sub-chunk, row) of the row view and of the col view
    int* qlen[2] = {nullptr, nullptr};     // pairs per octet segment of either
    int* rowcnt = nullptr;     // [O + 1]
    uint32_t* blk = nullptr;   // tie counts of the flag pass's blocks: [blocks(N) + 1] of the gradient growth, then [blocks(cap) + 1] of the prune selection
    uint64_t* sel_state = nullptr;   // [SEL_STATES][SEL_STATE_WORDS] radix-select state + histogram
    float* gemm = nullptr;     // [GEMM_WS_SPLITS * N] split-k partial outputs of the dense GEMM
    size_t gemm_floats = 0;
    float* partial = nullptr;  // weight-gradient partial sums [token tile][entry slots of the larger view]
    size_t partial_floats = 0;
    size_t total = 0;
};
Workspace carve_workspace(void* base, int O, int I, int64_t cap, int T);

constexpr int GEMM_WS_SPLITS = 8;
constexpr int SELECT_BLOCK = 2048;   // a block of the flag pass has more elements than this
constexpr int SEL_DIGIT_BITS = 8;                        // digit of the end of the random selection
constexpr int SEL_BINS = 1 << SEL_DIGIT_BITS;
constexpr int SEL_CTRL = 16;
constexpr int SEL_STATE_WORDS = SEL_CTRL + 7168 / 2;     // one selection: control words + the uint32 histograms of its digits
constexpr int SEL_STATES = 3;                            // prune, gradient growth, random growth

View view_shape(int R, int K, int64_t cap);
int fill_u32(void* dst, uint32_t value, int64_t n_words, hipStream_t s);

// ---- several layers in one launch ----
// The chains of small kernels of an update and of a view build take a batch of layers: one launch per link of the chain,
// whatever the number of layers.  Block (b, j) is block b of entry j, whose parameters lie in the kernel's arguments; a chain
// for one layer (layers on streams of their own) takes arguments of one entry.  The kernels are short, so reading the arguments
// counts: eight entries for every chain, and the entry found by a search over the block number, cost a quarter to half a
// microsecond of each of them.  Updates of one layer, such arguments -> these: 256 x 320 at density 0.77 103.5 -> 96.5 us,
// 636 x 448 at 0.03 131 -> 127, 3072 -> 256 at 0.99 192.5 -> 190, 3392 -> 1090 at 0.49 254 -> 251.
constexpr int BATCH_MAX = 8;
template <typename P, int CAP = BATCH_MAX>
struct Batch {
    struct Entry {
        unsigned blocks;
        P p;
    };
    Entry e[CAP];
    int n = 0;
    unsigned most = 0;         // blocks of an entry
    void add(const P& entry, int64_t blocks) {
        e[n++] = Entry{(unsigned)blocks, entry};
        most = std::max(most, (unsigned)blocks);
    }
    dim3 grid() const { return dim3(most, (unsigned)n); }
    __device__ bool surplus() const { return CAP > 1 && blockIdx.x >= e[blockIdx.y].blocks; }
    __device__ P entry() const { return e[CAP > 1 ? blockIdx.y : 0].p; }
    Batch<P, 1> first() const {
        Batch<P, 1> one;
        one.add(e[0].p, e[0].blocks);
        return one;
    }
};
// launch(batch) with the arguments that the number of layers needs
template <typename P, typename F>
void launch_batch(const Batch<P>& batch, F&& launch) {
    if (batch.n == 1) launch(batch.first());
    else launch(batch);
}
// one layer's part of a batched build or update
struct BuildItem {
    mst_layer* L;
    const float* Wsrc;         // dense weights, read at the active positions
    Workspace ws;
    bool keep_dense_copy;
};
struct UpdateItem {
    mst_layer* L;
    const float* G;
    mst_update_stats st;
    uint64_t seed;
    Workspace ws;
};

// ---- internal entry points implemented across the .hip files ----
int build_views(const BuildItem* items, int n, hipStream_t s);          // n up to BATCH_MAX
int build_canonical(const BuildItem* items, int n, bool recording, hipStream_t s);
int ensure_views(const mst_layer* L, const Workspace& ws, hipStream_t s);
int views_there(const mst_layer* L, hipStream_t s, bool* there);
bool views_wanted(const mst_layer* L);
int ensure_fresh(const mst_layer* L, bool row, bool col, hipStream_t s);
// the products of the sparse path; see walk.hip
int spmm(const mst_layer* L, const View& v, const void* A, float* out, int T, mst_dtype act, hipStream_t s);
int spmm_force_shape(int tokens_per_workgroup, int quads_per_wavefront);
int sddmm(const mst_layer* L, const void* dY, const void* X, float* dW, int T, mst_dtype act, float* partial,
          size_t partial_floats, hipStream_t s);
// dX and dW from one walk of the col view
int bwd_fused(const mst_layer* L, const void* dY, const void* X, float* dX, float* dW, int T, mst_dtype act,
              const Workspace& ws, hipStream_t s);
int bwd_fused_force_shape(int waves, int quads);
// C[M x N] (fp32) = op(A) op(B) on the matrix cores; see gemm_mfma.hip.  full: fp32 operands in full whatever the shape
enum GemmKind { GEMM_TN = 0, GEMM_NT = 1, GEMM_NN = 2 };
// (active: a GEMM_TN product of which only L's active outputs are wanted; where its kernel can leave the others out, the active ones
// go to dW, or to the partial outputs `stride` apart, and done says so)
struct ActiveRuns;
struct ActiveOut {
    const mst_layer* L;
    float* dW;
    int64_t stride = 0;
    bool done = false;
};
int active_runs(ActiveOut* active, hipStream_t s, ActiveRuns& runs, int64_t& stride);
int make_runs(mst_layer* const* layers, int n, hipStream_t s);           // n up to BATCH_MAX
int gemm_mfma(GemmKind kind, const void* A, mst_dtype a_dt, const void* B, mst_dtype b_dt, const uint16_t* planes, float* C,
              int M, int N, int Kdim, float* split_ws, int64_t split_ws_floats, hipStream_t s, bool full = false,
              int* left_unsummed = nullptr, ActiveOut* active = nullptr);
bool gemm_wants_planes(mst_dtype a_dt, int M, int N, int Kdim, bool full);
// G of bfloat16 activations, M and N multiples of 8; see gemm_wgrad.hip
int gemm_wgrad16(const uint16_t* A, const uint16_t* B, float* C, int M, int N, int Kdim, int k_per_split, int64_t split_stride,
                 const ActiveRuns& runs, hipStream_t s);
// Y and dX of bfloat16 activations from the split weights' planes; see gemm_planes.hip
int gemm_planes(const uint16_t* A, const uint16_t* P, float* C, int M, int N, int Kdim, hipStream_t s);
int make_planes(const mst_layer* L, hipStream_t s);
int weights_made(mst_layer* L, bool planes, bool pairs, hipStream_t s);
// the same at densities of a tenth and below, for both activation types; see gemm_pairs.hip
PairsView pairs_view(void* mem, int R, int K);
bool pairs_kept(const mst_layer* L);
bool pairs_wanted(const mst_layer* L, bool both);
struct ActiveRuns;
int make_pairs(mst_layer* L, hipStream_t s, const ActiveRuns* words = nullptr);
int measure_pairs(mst_layer* L, hipStream_t s);
// A measurement waits for its stream: an update behind fewer products than these leaves the last one standing.  (Updates are hundreds of
// steps apart in earnest; a loop that updates after every step would wait in every step.)
constexpr int PAIRS_CALLS = 64;
int pairs_tokens(const mst_layer* L, bool y, mst_dtype act, int T, int64_t split_floats, double making_us);
double making_pairs_us(const mst_layer* L, bool match);
int gemm_pairs(const void* A, mst_dtype act, const PairsView& v, float* C, int T, int tokens, hipStream_t s);
double gemm_two_parts_us(GemmKind kind, mst_dtype a_dt, int M, int N, int Kdim, int64_t max_split);
bool gemm_pairs_forced();
void gemm_note_tile(int tile);
// the same at full fp32 precision for any shape (B fp32); see gemm_exact.hip
int gemm_exact(GemmKind kind, const void* A, mst_dtype a_dt, const float* B, float* C, int M, int N, int Kdim,
               float* split_ws, int64_t split_ws_floats, hipStream_t s, int* left_unsummed, ActiveOut* active = nullptr);
int gemm_exact_tile(int tile);
int gemm_stream_tn_bf16(const uint16_t* A, const uint16_t* B, float* C, int M, int N, int Kdim, int k_per_split, int64_t split_stride,
                        hipStream_t s);
double xcd_rounds(int64_t n, int places, int lone_places, double full, double lone);
// modelled times in microseconds (max_split: k ranges there is room for; summed: their sum included)
double gemm_mfma_us(GemmKind kind, mst_dtype a_dt, int M, int N, int Kdim, int64_t max_split, bool summed, bool full);
double gemm_exact_us(mst_dtype a_dt, int M, int N, int Kdim, int64_t max_split, bool summed);
double walk_us(const mst_layer* L, WalkJob job, int T);
int sum_split_planes(const float* part, int64_t stride, int nsplit, float* C, int64_t n, hipStream_t s);
int gemm_force_fp32_mfma(int on);
int gemm_last_tile();
int mask_update_device(const UpdateItem* items, int n, hipStream_t s);   // n up to BATCH_MAX
int dense_products_fwd(const mst_layer* L, const void* X, float* Y, int T, mst_dtype act, hipStream_t s, bool full);
int dense_products_bwd_input(const mst_layer* L, const void* dY, float* dX, int T, mst_dtype act, hipStream_t s, bool full,
                             float* split_ws = nullptr, int64_t split_ws_floats = 0);
int dense_products_bwd_weight(const mst_layer* L, const void* dY, const void* X, float* dW, int T,
                              mst_dtype act, const Workspace& ws, hipStream_t s, bool full);
int ensure_dense_copy(mst_layer* L, hipStream_t s, bool* refreshed);
// heavy rows of the forward product; see heavy.hip
int heavy_rows_enable(int on);
int heavy_rows_mode();
int heavy_mark(const mst_layer* L, const Workspace& ws, int Rpad, hipStream_t s);     // clears counts of the row view
int heavy_fill(const mst_layer* L, hipStream_t s);
int heavy_fwd(const mst_layer* L, const void* X, float* Y, int T, mst_dtype act, hipStream_t s);

}  // namespace mst
