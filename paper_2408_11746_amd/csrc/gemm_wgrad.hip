// G = dY^T X with bfloat16 activations, both operands k-major (A [K x M], B [K x N], M and N multiples of 8): the dense weight
// gradient, one MFMA per term, on 256 x 256 tiles.
// Nothing of a step passes through registers but the operands of the MFMAs: rows go straight to LDS as they are in memory,
// and ds_read_b64_tr_b16 turns four k of sixteen columns round on the way out (the kernel that transposed 8 x 8 patches in
// registers and stored them to LDS spent half its time there).
//   - Four wavefronts of 128 x 128 read 64 KB of LDS per step of 32 k, eight of 128 x 64 would read 96 KB: with the 32 KB that
//     arrive that is all the LDS can move in the 1024 clocks of a step's MFMAs.  The sums take the accumulation half of the registers.
//   - One wavefront per SIMD has nothing to hide behind, so every step's 32 reads (operands of the next step) and 8 loads
//     (the step two after that) stand one by one between MFMAs: 1861 clocks a step with the loads in front and the reads in
//     pairs, 1518 with the loads spread, 1343 with both; 1127 with neither.
//   - Every step loads and waits for the same number of pieces, which keeps the loop free of branches: past the end it reads the
//     last step again, into a stage that nobody reads.  Their number is made even (two register sets); rows past the
//     end are cleared in LDS.
// us, K = 16384: 4096 x 1024 in 4 ranges 158 -> 125, K = 4099 49.8 -> 41; 5120 x 1280, K = 8192, in 2 ranges 133 -> 111.  What bounds it
// now: 76 % of the matrix cores' clocks at 1.6 GHz, the clock they leave, and 8 us for the 256 KB that every workgroup
// stores at the end, all at the same time (9 TB/s).
#include <type_traits>

#include "common.h"
#include "active.h"
#include "split_bf16.h"

namespace mst {

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
constexpr int GK = 32, G_OP = GK * 512, G_STAGE = 2 * G_OP;      // a row of LDS is one k and 256 columns
constexpr unsigned G_LDS = 4 * G_STAGE, G_WORDS = 4096;         // (words of a wavefront's 128 rows and columns)

// The 32-byte units (16 columns) of row k are kept at unit ^ swizzle(k): the eight rows that half a wavefront reads
// (four and, eight further, four) lie in different banks.
__device__ __forceinline__ int wgrad_swizzle(int k) { return (k & 3) | ((k >> 1) & 4); }

// ACTIVE: only the active outputs, side by side (C and split_stride are of them).  Whole planes and a gather -> this, at a density of
// 0.05: 1024 <-> 4096, 16384 tokens 108 + 10.2 us, so 104 + 4.9; 4096 x 1024, 4099 tokens 39 + 8.5, so 37.7 + 4.9, and the products
// behind it, which find their operands in the caches: both products of the backward 10 us.
template <bool ACTIVE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_gemm_wgrad16(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, float* __restrict__ C, int M, int N, int Kdim,
                    int k_per_split, int64_t split_stride, const ActiveRuns runs) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * 128, wn = (wave & 1) * 128;
    const int gm = (M + 255) / 256, gn = (N + 255) / 256, ntiles = gm * gn, nsplit = (Kdim + k_per_split - 1) / k_per_split;
    const int Q = (ntiles + 7) >> 3, slot = blockIdx.x >> 3;
    const int split = slot / Q, tile_id = (blockIdx.x & 7) * Q + slot % Q;
    if (tile_id >= ntiles || split >= nsplit) return;
    int mi, ni;
    tile_coords(tile_id, gm, gn, mi, ni);
    const int m0 = mi * 256, n0 = ni * 256;
    const int kbeg = split * k_per_split, rows = min(Kdim - kbeg, k_per_split);
    const int nload = (rows + GK - 1) / GK, nsteps = (nload + 1) & ~1, tail = rows - (nload - 1) * GK;
    float* const Cz = C + (int64_t)split * split_stride;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    // A piece is two rows of an operand, 16 bytes per lane; a wavefront loads four of each.  Columns past the end are the last
    // ones again (their outputs are not stored), and so are rows past the end of the last step (cleared before use).
    constexpr int PIECES = 8;
    uint32_t va[4], vb[4];
    auto offsets = [&](int valid) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 2 * (wave * 4 + j) + (lane >> 5), row = min(k, valid - 1);
            const int col = 16 * (((lane & 31) >> 1) ^ wgrad_swizzle(k)) + 8 * (lane & 1);
            va[j] = 2u * ((uint32_t)row * (uint32_t)M + (uint32_t)min(m0 + col, M - 8));
            vb[j] = 2u * ((uint32_t)row * (uint32_t)N + (uint32_t)min(n0 + col, N - 8));
        }
    };
    const uint16_t *pa, *pb;
    uint32_t to;
    auto aim = [&](int t) __attribute__((always_inline)) {       // at step t
        if (t == nload - 1 && tail < GK) offsets(tail);
        const int u = min(t, nload - 1);
        pa = A + (int64_t)(kbeg + u * GK) * M;
        pb = B + (int64_t)(kbeg + u * GK) * N;
        to = lds0 + (uint32_t)(t & 3) * G_STAGE + 4096u * wave;
    };
    auto piece = [&](int j) __attribute__((always_inline)) {
        if (j & 1) load_to_lds(pb, vb[j >> 1], to + G_OP + 1024u * (j >> 1));
        else load_to_lds(pa, va[j >> 1], to + 1024u * (j >> 1));
    };
    auto load = [&](int t) __attribute__((always_inline)) {
        aim(t);
#pragma unroll
        for (int j = 0; j < PIECES; ++j) piece(j);
    };
    auto arrive = [&](int t) __attribute__((always_inline)) {    // step t is in LDS, and everyone is done with step t - 2
        wait_loads<PIECES>();
        lds_barrier();
        const int valid = min(max(rows - t * GK, 0), GK);
        if (valid < GK) {
            for (int u = tid; u < (GK - valid) * 64; u += 256)
                *reinterpret_cast<uint4*>(lds + (t & 3) * G_STAGE + ((u >> 5) & 1) * G_OP + (valid + (u >> 6)) * 512 + (u & 31) * 16) = make_uint4(0, 0, 0, 0);
            lds_barrier();
        }
    };

    // operand reads: lane 16 g + 4 x + c gives the address of columns 4 c .. of row 8 g + x (and of row 8 g + x + 4) and
    // gets k 8 g .. 8 g + 7 of column 4 x + c
    const int g = lane >> 4, x = (lane >> 2) & 3;
    const uint32_t lrow = (uint32_t)((8 * g + x) * 512 + (lane & 3) * 8);
    uint32_t fa[8], fb[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        fa[i] = lrow + (uint32_t)(((wm / 16 + i) ^ wgrad_swizzle(8 * g + x)) << 5);
        fb[i] = lrow + (uint32_t)(((wn / 16 + i) ^ wgrad_swizzle(8 * g + x)) << 5) + G_OP;
    }
    typedef __attribute__((address_space(3))) shortx4* lds_shortx4;
    auto read = [&](uint32_t at) __attribute__((always_inline)) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4)(uintptr_t)at); };
    auto join = [&](shortx4 lo, shortx4 hi) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    floatx4 acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[2][8], b[2][8];
    // products of step t from register set P; the operands of step t + 1 go to the other set (after the last step: whatever
    // the stage holds, not used), pieces are those that aim() chose
    auto step = [&](auto pc, int t) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        const uint32_t st = lds0 + (uint32_t)((t + 1) & 3) * G_STAGE;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            shortx4 a0, a1, b0, b1;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // (by hand: the compiler would keep some of the sums outside the accumulation registers and spill)
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(b[P][j]), "v"(a[P][i]));
                if (j == 0) b0 = read(st + fb[i]);
                if (j == 1) b1 = read(st + fb[i] + 2048);
                if (j == 3) a0 = read(st + fa[i]);
                if (j == 4) a1 = read(st + fa[i] + 2048);
                if (j == 6) piece(i);
                __builtin_amdgcn_sched_barrier(0);
            }
            b[P ^ 1][i] = join(b0, b1);
            a[P ^ 1][i] = join(a0, a1);
        }
    };

    offsets(GK);
    if constexpr (ACTIVE) {
        // The words of this wavefront's outputs (past the end: no active ones), now: loaded behind the last step, their way from memory
        // was 3.5 us of the kernel's time.
        uint2 w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int at = 64 * e + lane, m = m0 + wm + (at >> 2), word = ((n0 + wn) >> 5) + (at & 3);
            w[e] = make_uint2(0xFFFFFFFFu, 0u);
            if (m < M && word < runs.per_row) w[e] = runs.words[(int64_t)m * runs.per_row + word];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) *reinterpret_cast<uint2*>(lds + G_LDS + G_WORDS * wave + 8 * (64 * e + lane)) = w[e];
    }
    load(0);
    load(1);
    arrive(0);
    load(2);
#pragma unroll
    for (int j = 0; j < 8; ++j) b[0][j] = join(read(lds0 + fb[j]), read(lds0 + fb[j] + 2048));
#pragma unroll
    for (int i = 0; i < 8; ++i) a[0][i] = join(read(lds0 + fa[i]), read(lds0 + fa[i] + 2048));
#pragma unroll 1
    for (int t = 0; t < nsteps; t += 2) {
        arrive(t + 1);
        aim(t + 3);
        step(std::integral_constant<int, 0>{}, t);
        arrive(t + 2);
        aim(t + 4);
        step(std::integral_constant<int, 1>{}, t + 1);
    }
    // nothing may arrive in LDS that is not ours any more; and the last MFMA is 18 wait states from its result
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) asm volatile("" : "+a"(acc[i][j]));
    // D layout of the 16x16 MFMA: lane l, register v -> row 4*(l/16) + v (B's), column l%16 (A's).  Through LDS, 64 rows at a
    // time in this wavefront's quarter, so that a store writes two runs of 512 bytes (sixteen of 64 bytes: 16200 clocks instead of
    // 14500); unit u (four columns) of row r is kept at u ^ (r & 15).
    __syncthreads();
    char* const mine = lds + 32768 * wave;
    const int lm = lane & 15, ou = lane & 31, n = n0 + wn + 4 * ou;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) *reinterpret_cast<floatx4*>(mine + (16 * i + lm) * 512 + (((4 * j + g) ^ lm) << 4)) = acc[4 * h + i][j];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if constexpr (ACTIVE) {
            // a lane has a column, so that a store writes what is active among 64 columns in one run
            const __amdgpu_buffer_rsrc_t out = active_buffer(Cz, runs);
            const uint32_t below = (1u << (lane & 31)) - 1u;
            const char* const words = lds + G_LDS + G_WORDS * wave + (64 * h) * 32 + 8 * (lane >> 5);
            // (four rows at a time, the next ones on their way while these are stored: there is one wavefront on a SIMD)
            uint2 w[2][8];
            float o[2][8];
            auto get = [&](int set, int r0) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int r = r0 + (e >> 1), c = 64 * (e & 1) + lane;
                    w[set][e] = *reinterpret_cast<const uint2*>(words + 32 * r + 16 * (e & 1));
                    o[set][e] = *reinterpret_cast<const float*>(mine + r * 512 + (((c >> 2) ^ (r & 15)) << 4) + 4 * (c & 3));
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            auto put = [&](int set) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 8; ++e) store_active(out, w[set][e], lane, below, o[set][e]);
                __builtin_amdgcn_sched_barrier(0);
            };
            get(0, 0);
#pragma unroll 2
            for (int r = 0; r < 64; r += 8) {
                get(1, r + 4);
                put(0);
                get(0, min(r + 8, 60));
                put(1);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            continue;
        }
#pragma unroll 8
        for (int r = lane >> 5; r < 64; r += 2) {
            const int m = m0 + wm + 64 * h + r;
            const floatx4 o = *reinterpret_cast<const floatx4*>(mine + r * 512 + ((ou ^ (r & 15)) << 4));
            if (m < M && n < N) *reinterpret_cast<floatx4*>(Cz + (int64_t)m * N + n) = o;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

// ranges of k_per_split (a multiple of 32) rows, each into its own M x N floats, split_stride (a multiple of 4) apart
int gemm_wgrad16(const uint16_t* A, const uint16_t* B, float* C, int M, int N, int Kdim, int k_per_split, int64_t split_stride,
                 const ActiveRuns& runs, hipStream_t s) {
    if (M % 8 || N % 8 || k_per_split % GK) return MST_ERR_ARG;
    static uint64_t done[2] = {0, 0};
    const bool active = runs.words != nullptr;
    const auto kernel = active ? k_gemm_wgrad16<true> : k_gemm_wgrad16<false>;
    const unsigned bytes = G_LDS + (active ? 4 * G_WORDS : 0u);
    const int rc = allow_lds(reinterpret_cast<const void*>(kernel), (int)bytes, done[active]);
    if (rc != MST_OK) return rc;
    const unsigned grid = (unsigned)(8 * cdiv(cdiv(M, 256) * cdiv(N, 256), 8) * cdiv(Kdim, k_per_split));
    kernel<<<grid, 256, bytes, s>>>(A, B, C, M, N, Kdim, k_per_split, split_stride, runs);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

}  // namespace mst
