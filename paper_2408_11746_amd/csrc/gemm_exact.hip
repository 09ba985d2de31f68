// Dense products of any shape at full fp32 precision on the bf16 matrix cores.
//
// Every fp32 operand element is cut, while it is staged, into three bfloat16 values hi + mid + lo of
// eight significant bits each, each the nearest to what is left: x = hi + mid + lo exactly (Henry, Tang and
// Heinecke 2019, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations"; below
// 2^-110 the last part falls under bfloat16's smallest value).  A product is
// hi.hi + hi.mid + mid.hi + mid.mid + hi.lo + lo.hi with fp32 accumulation; what is dropped is at most 2^-24 of it,
// in either direction.  A bfloat16 operand is one value, so bfloat16 x fp32 takes three products per term, all exact.
// Root mean square error of Y at 129 x 4099 -> 387 in units of 2^-24 sum |x w|, fp32 matrix instructions / 64 tile /
// 128 tile: normal operands 0.47 / 0.29 / 0.41, all positive ones 16.0 / 8.1 / 10.0 (mean -0.2 / -0.7 / -1.4).
// With truncated parts, which cost the same instructions, the dropped products all point to zero and are up to
// eight times as large: 65.7 / 194 on the positive operands, nearly all of it the mean.
// A value within 2^-9 of the largest finite one rounds to an infinity: its outputs come out as NaN and are
// formed again (fp32_sum).
//
// C[M x N] = sum_k A'[k][m] B'[k][n]; each operand k-major (element (k, m) at src[k*ld + m]) or m-major
// (src[m*ld + k]).  Serves the shapes whose tiles are not whole (an activation batch of any length, a
// layer of any size): they used to run on v_mfma_f32_32x32x2f32 at 100 TFLOP/s.  Six
// v_mfma_f32_32x32x16_bf16 take the place of eight of those at a sixteenth of the time each.
//
// k_gemm_exact: workgroup tile TM x TM, TM = 128 or 64, 256 threads = four wavefronts of (TM/2) x (TM/2); k steps of
// 4096 / TM, so that a plane of an operand's tile is 8 KB and a workgroup's LDS 48 KB (32 KB with a
// bfloat16 operand): two (three) workgroups share a CU and one's staging runs beside another's MFMAs.
// Loads are buffer loads from the tile's corner with exact ends: rows past the matrix read as zeros
// without an access, a 16-byte load needs dword alignment only, so no leading dimension is special.
// What lies past the end of a row is the next row; it lands in outputs that are not stored,
// or, along k, is cleared in the last step.  Bound: the matrix cores (six products per term; a large
// bf16 product runs at 1294 TFLOP/s on this card, that is 215 of these); the 128 tile pulls 1/6 of the
// operand bytes per MFMA of a plain bf16 kernel.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "active.h"
#include "split_bf16.h"

namespace mst {

typedef uint32_t ex_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t ex_u32x2 __attribute__((ext_vector_type(2)));

// LDS position of unit u (eight k) of row m in a plane of rows of 32 k (64 bytes) or 64 k (128 bytes).  Sixteen lanes read, and eight lanes
// store, without meeting in a bank: rows 0, 4, 8, 12 lie side by side, and the units of rows that are a multiple of 128 bytes apart
// are exchanged differently for each of them (k-major stores take every other row; before the last term of the exchange, and with
// m-major stores of consecutive rows, a third of the LDS cycles were conflicts).
template <int TM>
__device__ inline uint32_t ex_unit(int m, int u) {
    if (TM == 64) return (uint32_t)(m * 128 + ((u ^ ((m >> 1) & 7)) << 4));      // (stores of rows two apart, or of one row)
    const int rho = (m & ~15) | ((m & 3) << 2) | ((m >> 2) & 3);
    return (uint32_t)(rho * 64 + (((u ^ (rho >> 2) ^ (rho >> 4) ^ (rho >> 1 & 1)) & 3) << 4));
}

// a pair of fp32 values as three words of two bfloat16 each.  The parts are rounded to nearest, so the lower
// ones have either sign and half the size that truncation leaves: what the dropped products lose has no direction.
// The third part is exact: 24 bits less 8 and a sign, twice.
__device__ inline void cut_pair(float x0, float x1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    hi = cvt_pk_bf16(x0, x1);
    const float b0 = x0 - __uint_as_float(hi << 16), b1 = x1 - __uint_as_float(hi & 0xFFFF0000u);
    mid = cvt_pk_bf16(b0, b1);
    const float c0 = b0 - __uint_as_float(mid << 16), c1 = b1 - __uint_as_float(mid & 0xFFFF0000u);
    lo = __builtin_amdgcn_perm(__float_as_uint(c1), __float_as_uint(c0), 0x07060302u);
}

// The lower parts of an infinite value are inf - inf = NaN (those of a finite one whose first part rounds to an
// infinity the infinity of the other sign and NaN), so a sum with such an operand comes out as NaN where fp32
// products give a number or an infinity.  An output that is NaN is therefore formed again by fp32
// multiply-adds, up to the first term that makes it NaN by itself; no other output pays more than a compare.
template <typename TA, bool A_KMAJOR, typename TB, bool B_KMAJOR>
__device__ __forceinline__ float fp32_sum(const TA* __restrict__ A, int64_t lda, const TB* __restrict__ B, int64_t ldb, int m, int n,
                                          int kbeg, int kend) {
    auto value = [](auto x) {
        if constexpr (sizeof(x) == 2) return __uint_as_float((uint32_t)x << 16);
        else return x;
    };
    float sum = 0.f;
#pragma unroll 1
    for (int k = kbeg; k < kend && sum == sum; ++k)
        sum = fmaf(value(A[A_KMAJOR ? (int64_t)k * lda + m : (int64_t)m * lda + k]),
                   value(B[B_KMAJOR ? (int64_t)k * ldb + n : (int64_t)n * ldb + k]), sum);
    return sum;
}

// One operand's registers between global memory and LDS.  A thread (p = 0 .. 255) stages two pieces per
// step, a piece being one 16-byte unit (eight k of one row) in every plane: k-major the patch of eight k x
// two rows, m-major two units.
template <bool BF16, bool KMAJOR, int TM>
struct ExOperand {
    static constexpr int BK = 4096 / TM, UNITS = BK / 8, PLANES = BF16 ? 1 : 3;
    typedef typename std::conditional<BF16, uint16_t, float>::type T;
    float f[BF16 ? 1 : 16];      // piece j, k kk: k-major f[2 kk + j], m-major f[8 j + kk]
    ex_u32x4 h[BF16 ? 2 : 1];

    // Which row and unit thread p stages as its piece j.  (m-major, 128 tile: eight lanes store 128 consecutive bytes, the four units of two
    // rows that lie together.)
    __device__ static __forceinline__ int row(int p, int j) {
        if constexpr (KMAJOR) return 2 * (p % (TM / 2)) + j;
        else if constexpr (TM == 64) return (j * 256 + p) / UNITS;
        else return 64 * j + 16 * (p >> 6) + 4 * (p >> 2 & 3) + (p >> 4 & 3);
    }
    __device__ static __forceinline__ int unit(int p) { return KMAJOR ? p / (TM / 2) : p % UNITS; }

    // rows (k-major: k, m-major: m) of the tile past the end are cut off by the descriptor
    __device__ __forceinline__ void fetch(const T* __restrict__ src, int64_t ld, int k0, int m0, int kend, int Mdim, int p) {
        const int64_t corner = KMAJOR ? (int64_t)k0 * ld + m0 : (int64_t)m0 * ld + k0;
        const int64_t left = KMAJOR ? (int64_t)min(kend - k0, BK) * ld - m0 : (int64_t)min(Mdim - m0, TM) * ld - k0;   // elements
        const uint32_t bytes = (uint32_t)((left * (int64_t)sizeof(T) + 3) & ~3ll);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src + corner), 0, (int)bytes, 0x00020000);
        const uint32_t pitch = (uint32_t)ld * (uint32_t)sizeof(T);
        if constexpr (KMAJOR) {
            static_assert(!BF16, "a bfloat16 operand is m-major");
            const uint32_t o = (uint32_t)(8 * unit(p)) * pitch + (uint32_t)(4 * row(p, 0));
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const ex_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(o + kk * pitch), 0, 0);
                f[2 * kk] = __uint_as_float(v.x);
                f[2 * kk + 1] = __uint_as_float(v.y);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t o = (uint32_t)row(p, j) * pitch + (uint32_t)(8 * unit(p)) * (uint32_t)sizeof(T);
                if constexpr (BF16) {
                    if ((ld & 1) == 0) {
                        h[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o, 0, 0);
                    } else {                                              // odd rows start in the middle of a dword
                        const uint32_t oa = o & ~3u, sh = (o & 2u) << 3;
                        const ex_u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)oa, 0, 0);
                        const uint32_t e = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(oa + 16), 0, 0);
                        h[j].x = __builtin_amdgcn_alignbit(w.y, w.x, sh);
                        h[j].y = __builtin_amdgcn_alignbit(w.z, w.y, sh);
                        h[j].z = __builtin_amdgcn_alignbit(w.w, w.z, sh);
                        h[j].w = __builtin_amdgcn_alignbit(e, w.w, sh);
                    }
                } else {
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const ex_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(o + 16 * half), 0, 0);
#pragma unroll
                        for (int d = 0; d < 4; ++d) f[8 * j + 4 * half + d] = __uint_as_float(v[d]);
                    }
                }
            }
        }
    }
    // m-major rows go on past kend into the next row: cleared in the last step
    __device__ __forceinline__ void clear_tail(int k0, int kend, int p) {
        if constexpr (!KMAJOR) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int valid = kend - (k0 + 8 * unit(p));      // k of this unit that exist
                if constexpr (BF16) {
#pragma unroll
                    for (int d = 0; d < 4; ++d)
                        h[j][d] = valid >= 2 * d + 2 ? h[j][d] : valid == 2 * d + 1 ? h[j][d] & 0xFFFFu : 0u;
                } else {
#pragma unroll
                    for (int d = 0; d < 8; ++d) f[8 * j + d] = d < valid ? f[8 * j + d] : 0.f;
                }
            }
        }
    }
    __device__ __forceinline__ void stage(char* lds, int p) const {
        constexpr int PLANE = TM * BK * 2;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t a = ex_unit<TM>(row(p, j), unit(p));
            if constexpr (BF16) {
                *reinterpret_cast<ex_u32x4*>(lds + a) = h[j];
            } else {
                uint32_t hi[4], mid[4], lo[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    if constexpr (KMAJOR) cut_pair(f[4 * d + j], f[4 * d + 2 + j], hi[d], mid[d], lo[d]);
                    else cut_pair(f[8 * j + 2 * d], f[8 * j + 2 * d + 1], hi[d], mid[d], lo[d]);
                }
                *reinterpret_cast<uint4*>(lds + a) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                *reinterpret_cast<uint4*>(lds + PLANE + a) = make_uint4(mid[0], mid[1], mid[2], mid[3]);
                *reinterpret_cast<uint4*>(lds + 2 * PLANE + a) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            }
        }
    }
};

// Tile numbers run in bands of eight tile rows, column by column inside a band (the tiles an XCD works on
// at a time share operand panels in its L2); XCD x takes a contiguous share, one k range after the other.
// PER_CU: workgroups on a CU that the registers are for (plan_exact's choice; 0: as many as the LDS holds).  With both operands k-major always
// three, two of them held apart by their LDS: the code for two takes three registers more (170) and is, alone on its CU, 9 % slower (dense
// gradients of 1048 x 792, 385 tokens, to 5000 x 4000, one k range; half of the 80 shapes are 10 % slower with it).
// ACTIVE: only the active outputs, side by side (C and split_stride are of them).  Whole outputs and a gather -> this: 4000 x 1000 at a density of
// 0.2, 5001 tokens 215 us, so 208, 1000 tokens 54.2, so 49.4; 5000 x 4000 at 0.9, 700 tokens 180, so 149.
template <bool A16, bool A_KMAJOR, bool B_KMAJOR, int TM, int PER_CU, bool ACTIVE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PER_CU ? PER_CU : A_KMAJOR ? 3 : 2, PER_CU ? PER_CU : 3)))
void k_gemm_exact(const void* __restrict__ Av, int64_t lda, const float* __restrict__ B, int64_t ldb, float* __restrict__ C,
                  int M, int N, int Kdim, int k_per_split, int64_t split_stride, const ActiveRuns runs) {
    static_assert(!ACTIVE || TM == 128);
    typedef ExOperand<A16, A_KMAJOR, TM> OpA;
    typedef ExOperand<false, B_KMAJOR, TM> OpB;
    constexpr int BK = 4096 / TM, PLANE = 8192, MI = TM / 64;
    extern __shared__ __attribute__((aligned(16))) char ex_lds[];
    char* const la = ex_lds;
    char* const lb = la + OpA::PLANES * PLANE;
    const int gm = (M + TM - 1) / TM, gn = (N + TM - 1) / TM, ntiles = gm * gn;
    const int nsplit = (Kdim + k_per_split - 1) / k_per_split, Q = (ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int split = slot / Q, tile_id = xcd * Q + slot % Q;
    if (tile_id >= ntiles || split >= nsplit) return;
    const int band = tile_id / (8 * gn), rem = tile_id - band * 8 * gn, hgt = min(8, gm - 8 * band);
    const int m0 = (8 * band + rem % hgt) * TM, n0 = (rem / hgt) * TM;
    const int kbeg = split * k_per_split, kend = min(Kdim, kbeg + k_per_split);
    float* const Cz = C + (int64_t)split * split_stride;
    const typename OpA::T* const A = static_cast<const typename OpA::T*>(Av);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * (TM / 2);
    floatx16 acc[MI][MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // one tile per wavefront: two chains of products, an MFMA on the result of the one before waits for it
    constexpr int CHAINS = MI == 1 ? 2 : 1;
    floatx16 other;
#pragma unroll
    for (int v = 0; v < 16; ++v) other[v] = 0.f;
    OpA ra;
    OpB rb;
    auto fetch = [&](int k0) __attribute__((always_inline)) {
        ra.fetch(A, lda, k0, m0, kend, M, tid);
        rb.fetch(B, ldb, k0, n0, kend, N, tid);
    };
    const int lk = lane >> 5, lm = lane & 31;
    // plane pairs of the products, smallest terms first
    constexpr int NP = A16 ? 3 : 6;
    constexpr int pa[6] = {A16 ? 0 : 2, A16 ? 0 : 0, A16 ? 0 : 1, 1, 0, 0};
    constexpr int pb[6] = {A16 ? 2 : 0, A16 ? 1 : 2, A16 ? 0 : 1, 0, 1, 0};
    auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 a[OpA::PLANES][MI], b[OpB::PLANES][MI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const uint32_t ua = ex_unit<TM>(wm + 32 * i + lm, 2 * ks + lk), ub = ex_unit<TM>(wn + 32 * i + lm, 2 * ks + lk);
#pragma unroll
                for (int z = 0; z < OpA::PLANES; ++z) a[z][i] = *reinterpret_cast<const bf16x8*>(la + z * PLANE + ua);
#pragma unroll
                for (int z = 0; z < OpB::PLANES; ++z) b[z][i] = *reinterpret_cast<const bf16x8*>(lb + z * PLANE + ub);
            }
#pragma unroll
            for (int t = 0; t < NP; ++t)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < MI; ++j) {
                        floatx16& c = CHAINS > 1 && (t & 1) ? other : acc[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa[t]][i], b[pb[t]][j], c, 0, 0, 0);
                    }
        }
    };
    auto stage = [&]() __attribute__((always_inline)) {
        ra.stage(la, tid);
        rb.stage(lb, tid);
    };
    int k0 = kbeg;
    char* const words = lb + OpB::PLANES * PLANE + 1024 * wave;      // of this wavefront's 64 rows and columns; past the end: no active ones
    if constexpr (ACTIVE) {
        const int m = m0 + wm + lane, word = (n0 + wn) >> 5;
        uint2 w[2] = {make_uint2(0xFFFFFFFFu, 0u), make_uint2(0xFFFFFFFFu, 0u)};
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (m < M && word + j < runs.per_row) w[j] = runs.words[(int64_t)m * runs.per_row + word + j];
        *reinterpret_cast<uint4*>(words + 16 * lane) = make_uint4(w[0].x, w[0].y, w[1].x, w[1].y);
    }
    fetch(k0);
    for (; k0 + BK < kend; k0 += BK) {
        __syncthreads();
        stage();
        __syncthreads();
        fetch(k0 + BK);
        multiply();
    }
    __syncthreads();
    ra.clear_tail(k0, kend, tid);
    rb.clear_tail(k0, kend, tid);
    stage();
    __syncthreads();
    multiply();
    if constexpr (CHAINS > 1)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][0][v] += other[v];
    // D layout of the 32x32 MFMA: lane l, register v -> row 8*(v/4) + 4*(l/32) + v%4, column l%32
    bool nan = false;
    if constexpr (ACTIVE) {
        const __amdgpu_buffer_rsrc_t out = active_buffer(Cz, runs);
        const uint32_t below = (1u << lm) - 1u;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint4 w = *reinterpret_cast<const uint4*>(words + 16 * (32 * i + 8 * (v >> 2) + 4 * lk + (v & 3)));
                store_active(out, make_uint2(w.x, w.y), lane, below, acc[i][0][v]);
                store_active(out, make_uint2(w.z, w.w), lane, below, acc[i][MI - 1][v]);
                nan |= acc[i][0][v] != acc[i][0][v] || acc[i][MI - 1][v] != acc[i][MI - 1][v];
            }
        if (nan) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
            for (int x = 0; x < MI * MI * 16; ++x) {
                const int r = (x / (16 * MI)) * 32 + 8 * ((x >> 2) & 3) + 4 * lk + (x & 3), j = (x >> 4) % MI;
                const uint32_t at = active_offset(*reinterpret_cast<const uint2*>(words + 16 * r + 8 * j), (uint32_t)lm, below);
                if (at >= runs.bytes) continue;
                float* const c = Cz + (at >> 2);
                if (*c != *c) *c = fp32_sum<typename OpA::T, A_KMAJOR, float, B_KMAJOR>(A, lda, B, ldb, m0 + wm + r, n0 + wn + 32 * j + lm, kbeg, kend);
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + wm + i * 32 + 8 * (v >> 2) + 4 * lk + (v & 3);
                const int n = n0 + wn + j * 32 + lm;
                if (m < M && n < N) Cz[(int64_t)m * N + n] = acc[i][j][v];
                nan |= acc[i][j][v] != acc[i][j][v];
            }
    if (nan) {
#pragma unroll 1
        for (int x = 0; x < MI * MI * 16; ++x) {
            const int m = m0 + wm + (x / (16 * MI)) * 32 + 8 * ((x >> 2) & 3) + 4 * lk + (x & 3);
            const int n = n0 + wn + ((x >> 4) % MI) * 32 + lm;
            if (m >= M || n >= N) continue;
            float* const c = Cz + (int64_t)m * N + n;
            if (*c != *c) *c = fp32_sum<typename OpA::T, A_KMAJOR, float, B_KMAJOR>(A, lda, B, ldb, m, n, kbeg, kend);
        }
    }
}

// ---- Small outputs: one workgroup per 32 x 32 (MI = 1) or 64 x 64 (MI = 2) output tile, all its
// wavefronts on the same tile, each with k steps of its own.  Operands go from global memory straight to
// the registers the matrix instructions read (lane = row, 16 or 8 consecutive k), no LDS and no barrier until
// the partial tiles are added in wavefront order at the end.  An output of a few dozen tiles is a chain
// of k steps that nothing else hides, and here a CU has 16 (8) steps on the way instead of one or three.
// Every wavefront converts its own operands, so the vector ALU (MI = 1: about 90 instructions beside six
// MFMAs per 16 k) bounds it where there are tiles for all CUs.
//
// Rows of the tile a lane holds: m-major lm and 32 + lm; k-major 2 lm and 2 lm + 1, so that both come with
// one load per k.
template <bool BF16, bool KMAJOR, int MI, int KS>
struct StreamOperand {                               // KS / 2 consecutive k of MI rows per lane
    static constexpr int NF = KS / 2, PLANES = BF16 ? 1 : 3;
    // bfloat16: dwords from the one that holds the first element; k-major MI = 1 would waste half of each
    static constexpr int NH = !BF16 ? 1 : KMAJOR ? 2 * NF : MI * (NF / 2 + 1);
    typedef typename std::conditional<BF16, uint16_t, float>::type T;
    static_assert(!(BF16 && KMAJOR) || MI == 2, "");
    float f[BF16 ? 1 : MI * NF];                      // row i, k kk: f[i NF + kk]
    uint32_t h[NH];
    uint32_t sh[BF16 && !KMAJOR ? MI : 1];

    __device__ static __forceinline__ int row(int i, int lm) { return KMAJOR && MI == 2 ? 2 * lm + i : 32 * i + lm; }

    // rows past the matrix (m-major) and k from kend on (k-major) are cut off by the descriptor
    __device__ __forceinline__ void fetch(const T* __restrict__ src, int64_t ld, int k0, int m0, int kend, int Mdim, int lm, int lk) {
        const int64_t corner = KMAJOR ? (int64_t)k0 * ld + m0 : (int64_t)m0 * ld + k0;
        const int64_t left = k0 >= kend ? 0 : KMAJOR ? (int64_t)min(kend - k0, KS) * ld - m0 : (int64_t)min(Mdim - m0, 32 * MI) * ld - k0;
        const uint32_t bytes = left <= 0 ? 0u : (uint32_t)((left * (int64_t)sizeof(T) + 3) & ~3ll);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src + (bytes ? corner : 0)), 0, (int)bytes, 0x00020000);
        const uint32_t pitch = (uint32_t)ld * (uint32_t)sizeof(T);
        if constexpr (KMAJOR) {
            uint32_t o = (uint32_t)(NF * lk) * pitch + (uint32_t)(MI * lm) * (uint32_t)sizeof(T);
            asm volatile("" : "+v"(o));               // (NF offsets kept across the loop would not fit the registers)
#pragma unroll
            for (int kk = 0; kk < NF; ++kk, o += pitch) {
                if constexpr (BF16) {                 // (rows of an odd length: every other one starts in the middle of a dword)
                    const ex_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(o & ~3u), 0, 0);
                    h[2 * kk] = v.x;
                    h[2 * kk + 1] = v.y;
                } else if constexpr (MI == 2) {
                    const ex_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, 0, 0);
                    f[kk] = __uint_as_float(v.x);
                    f[NF + kk] = __uint_as_float(v.y);
                } else {
                    f[kk] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)o, 0, 0));
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const uint32_t o = (uint32_t)(32 * i + lm) * pitch + (uint32_t)(NF * lk) * (uint32_t)sizeof(T);
                if constexpr (BF16) {
                    sh[i] = (o & 2u) << 3;
#pragma unroll
                    for (int u = 0; u < NF / 8; ++u) {
                        const ex_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)((o & ~3u) + 16 * u), 0, 0);
#pragma unroll
                        for (int d = 0; d < 4; ++d) h[i * (NF / 2 + 1) + 4 * u + d] = v[d];
                    }
                    h[i * (NF / 2 + 1) + NF / 2] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)((o & ~3u) + 2 * NF), 0, 0);
                } else {
#pragma unroll
                    for (int u = 0; u < NF / 4; ++u) {
                        const ex_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(o + 16 * u), 0, 0);
#pragma unroll
                        for (int d = 0; d < 4; ++d) f[i * NF + 4 * u + d] = __uint_as_float(v[d]);
                    }
                }
            }
        }
    }
    // bfloat16: pairs into place, h[i (NF / 2) + d] the pair of k 2d, 2d + 1 of row i.  In the last step
    // (`tail`) k from kend on are cleared: m-major rows go on into the next row there, and the last dword of
    // a k-major operand may hold the first element of row kend.
    __device__ __forceinline__ void settle(bool tail, int k0, int kend, int64_t ld, int lk) {
        const int valid = kend - (k0 + NF * lk);      // k of this lane that exist
        if constexpr (BF16 && KMAJOR) {
            const uint32_t s = (uint32_t)(ld & 1) << 4;
#pragma unroll
            for (int d = 0; d < NF / 2; ++d) {        // (k0 and NF lk are even)
                uint32_t e = h[4 * d], o = __builtin_amdgcn_alignbit(h[4 * d + 3], h[4 * d + 2], s);
                if (tail) {
                    e = 2 * d < valid ? e : 0u;
                    o = 2 * d + 1 < valid ? o : 0u;
                }
                h[2 * d] = __builtin_amdgcn_perm(o, e, 0x05040100u);
                h[2 * d + 1] = __builtin_amdgcn_perm(o, e, 0x07060302u);
            }
        } else if constexpr (BF16) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int d = 0; d < NF / 2; ++d) {
                    const int x = i * (NF / 2 + 1) + d;
                    h[x] = __builtin_amdgcn_alignbit(h[x + 1], h[x], sh[i]);
                    if (tail) h[x] = valid >= 2 * d + 2 ? h[x] : valid == 2 * d + 1 ? h[x] & 0xFFFFu : 0u;
                }
        } else if constexpr (!KMAJOR) {
            if (tail)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int d = 0; d < NF; ++d) f[i * NF + d] = d < valid ? f[i * NF + d] : 0.f;
        }
    }
    // planes of the u-th eight k of row i
    __device__ __forceinline__ void planes(int i, int u, bf16x8 (&p)[PLANES]) const {
        if constexpr (BF16) {
            ex_u32x4 w;
#pragma unroll
            for (int d = 0; d < 4; ++d) w[d] = KMAJOR ? h[2 * (4 * u + d) + i] : h[i * (NF / 2 + 1) + 4 * u + d];
            p[0] = __builtin_bit_cast(bf16x8, w);
        } else {
            ex_u32x4 w[3];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t hi, mid, lo;
                cut_pair(f[i * NF + 8 * u + 2 * d], f[i * NF + 8 * u + 2 * d + 1], hi, mid, lo);
                w[0][d] = hi; w[1][d] = mid; w[2][d] = lo;
            }
#pragma unroll
            for (int z = 0; z < 3; ++z) p[z] = __builtin_bit_cast(bf16x8, w[z]);
        }
    }
};

constexpr unsigned STREAM_LDS_32 = 16 * 32 * 32 * 4, STREAM_LDS_64 = 8 * 64 * 64 * 4;    // a partial tile per wavefront
template <bool A16, bool A_KMAJOR, bool B16, bool B_KMAJOR, int MI>
__global__ __launch_bounds__(MI == 1 ? 1024 : 512)
void k_gemm_stream(const void* __restrict__ Av, int64_t lda, const void* __restrict__ Bv, int64_t ldb, float* __restrict__ C,
                   int M, int N, int Kdim, int k_per_split, int64_t split_stride) {
    constexpr int KS = MI == 1 ? 32 : 16, NW = MI == 1 ? 16 : 8, TM = 32 * MI;
    typedef StreamOperand<A16, A_KMAJOR, MI, KS> OpA;
    typedef StreamOperand<B16, B_KMAJOR, MI, KS> OpB;
    extern __shared__ __attribute__((aligned(16))) char ex_lds[];
    const int gm = (M + TM - 1) / TM, gn = (N + TM - 1) / TM, ntiles = gm * gn;
    const int nsplit = (Kdim + k_per_split - 1) / k_per_split, Q = (ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int split = slot / Q, tile_id = xcd * Q + slot % Q;
    if (tile_id >= ntiles || split >= nsplit) return;
    const int band = tile_id / (8 * gn), rem = tile_id - band * 8 * gn, hgt = min(8, gm - 8 * band);
    const int m0 = (8 * band + rem % hgt) * TM, n0 = (rem / hgt) * TM;
    const int kbeg = split * k_per_split, kend = min(Kdim, kbeg + k_per_split);
    float* const Cz = C + (int64_t)split * split_stride;
    const typename OpA::T* const A = static_cast<const typename OpA::T*>(Av);
    const typename OpB::T* const B = static_cast<const typename OpB::T*>(Bv);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lk = lane >> 5, lm = lane & 31;

    floatx16 acc[MI][MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // plane pairs, smallest terms first
    constexpr int NP = A16 && B16 ? 1 : A16 ? 3 : 6;
    constexpr int pa[6] = {A16 ? 0 : 2, A16 ? 0 : 0, A16 ? 0 : 1, 1, 0, 0};
    constexpr int pb[6] = {B16 ? 0 : A16 ? 2 : 0, A16 ? 1 : 2, A16 ? 0 : 1, 0, 1, 0};
    OpA ra[2];
    OpB rb[2];
    auto fetch = [&](OpA& a, OpB& b, int k0) __attribute__((always_inline)) {
        a.fetch(A, lda, k0, m0, kend, M, lm, lk);
        b.fetch(B, ldb, k0, n0, kend, N, lm, lk);
    };
    auto multiply = [&](OpA& a, OpB& b, int k0) __attribute__((always_inline)) {
        if (k0 + KS > kend) {
            a.settle(true, k0, kend, lda, lk);
            b.settle(true, k0, kend, ldb, lk);
        } else {
            a.settle(false, k0, kend, lda, lk);
            b.settle(false, k0, kend, ldb, lk);
        }
#pragma unroll
        for (int u = 0; u < KS / 16; ++u) {
            bf16x8 fa[MI][OpA::PLANES], fb[MI][OpB::PLANES];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                a.planes(i, u, fa[i]);
                b.planes(i, u, fb[i]);
            }
#pragma unroll
            for (int t = 0; t < NP; ++t)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < MI; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][pa[t]], fb[j][pb[t]], acc[i][j], 0, 0, 0);
        }
    };
    // step r of this wavefront starts at kbeg + (r NW + wave) KS; steps past kend are zeros
    const int stride = KS * NW;
    int k0 = kbeg + wave * KS;
    fetch(ra[0], rb[0], k0);
    while (k0 < kend) {
        fetch(ra[1], rb[1], k0 + stride);
        multiply(ra[0], rb[0], k0);
        fetch(ra[0], rb[0], k0 + 2 * stride);
        multiply(ra[1], rb[1], k0 + stride);
        k0 += 2 * stride;
    }
    // D layout of the 32x32 MFMA: lane l, register v -> row 8*(v/4) + 4*(l/32) + v%4, column l%32
    float* const part = reinterpret_cast<float*>(ex_lds);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                part[(wave * TM + OpA::row(i, 8 * (v >> 2) + 4 * lk + (v & 3))) * TM + OpB::row(j, lm)] = acc[i][j][v];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < TM * TM / (64 * NW); ++e) {
        const int x = e * 64 * NW + tid, m = m0 + x / TM, n = n0 + x % TM;
        float sum = part[x];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += part[w * TM * TM + x];
        if (m < M && n < N) {
            if constexpr (!(A16 && B16))
                if (sum != sum) sum = fp32_sum<typename OpA::T, A_KMAJOR, typename OpB::T, B_KMAJOR>(A, lda, B, ldb, m, n, kbeg, kend);
            Cz[(int64_t)m * N + n] = sum;
        }
    }
}

// Kernel, workgroup tile and number of k ranges together, as for the split kernels: modelled time = rounds
// one XCD needs for its share of the tiles x time of a workgroup, plus a launch and the traffic of the
// partial outputs.  Places of an XCD: 64 or 96 workgroups of 128 x 128, 96 of 64 x 64, 32 of the streaming
// kernel; with no more workgroups than CUs each has one to itself and is faster.  Microseconds fitted to timings
// of 130 products, 1 to 40 GFLOP, on MI355X (8-14 % rms error).
// Three 128 x 128 workgroups of fp32 operands on a CU take 1.45 times as long as two (115 shapes, sd 4 to 7 %), so which of the two is
// ahead is a matter of how the tiles fill the rounds: Y of 1000 -> 4000, 5001 tokens (1280 tiles), 240 us with
// two and 212 with three, of 1203 -> 801, 16001 tokens (882 tiles), 191 and 212.  (bfloat16 A: three always, as its constants were fitted.)
// With both operands k-major 1.51 times, and less by a twentieth where a second round follows the first, whose workgroups do not
// end together (104 outputs of 10^6 and more, one to eight ranges; 1.56 and nothing off took one range where several with a second round were
// ahead: 2304 x 3840, 3001 tokens, 342 us with one range, 283 with five).
struct ExactPlan {
    int tile;
    bool stream;
    int nsplit;
    double us;
    int places;
};
static int g_exact_tile = 0;                          // test hook: 0 automatic, 64 or 128, streaming: 32 or 96 (64 x 64)
static ExactPlan plan_exact(bool three, bool tn, int M, int N, int Kdim, bool a16, int64_t max_split, bool summed) {
    struct Kind {
        int hook, tile;
        bool stream;
        int places, lone_places, bk;
        // fp32, bfloat16 A: a k step with all places taken, with a CU to itself; start-up and output of a workgroup
        // (streaming: a k of all steps; microseconds); launch
        double full[2], lone[2], start[2], launch[2];
    };
    static const Kind kinds[] = {{128, 128, false, 64, 32, 32, {2.71, 1.64}, {1.78, 1.08}, {1.4, 1.2}, {2.6, 4.0}},
                                 {128, 128, false, 96, 32, 32, {3.92, 0.0}, {1.78, 0.0}, {1.4, 0.0}, {2.6, 0.0}},
                                 {64, 64, false, 96, 32, 64, {2.63, 1.65}, {1.47, 0.97}, {0.5, 0.7}, {3.3, 3.6}},
                                 {32, 32, true, 32, 0, 128, {0.0052, 0.0046}, {0.0046, 0.0040}, {3.1, 2.6}, {2.9, 3.1}},
                                 {96, 64, true, 32, 0, 128, {0.0131, 0.0117}, {0.0108, 0.0106}, {3.7, 2.6}, {2.8, 3.1}}};
    static const int cand[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
    ExactPlan best{0, false, 1, 0.0, 0};
    for (const Kind& kd : kinds) {
        if (g_exact_tile && kd.hook != g_exact_tile) continue;
        const int64_t Q = cdiv(cdiv(M, kd.tile) * cdiv(N, kd.tile), 8);
        if ((a16 || !three) && kd.full[1] == 0.0) continue;
        const bool tn_three = tn && kd.tile == 128 && kd.places == 96;
        const double full = kd.full[a16] * (tn_three ? 1.045 : 1.0), lone = kd.lone[a16];
        for (int ns : cand) {
            if (ns > 1 && (ns > max_split || Kdim / ns < 256)) break;
            const double work = xcd_rounds(Q * ns, kd.places, kd.lone_places, full, lone) * (tn_three && Q * ns > kd.places ? 0.944 : 1.0);
            double cost = kd.launch[a16] + (kd.stream ? work * (double)cdiv(Kdim, ns) + (double)cdiv(Q * ns, kd.places) * kd.start[a16]
                                                      : work * ((double)cdiv(cdiv(Kdim, ns), kd.bk) + kd.start[a16]));
            if (ns > 1) cost += 3.0 + 1.0e-6 * (double)M * (double)N * (summed ? ns + 1.0 : 0.25 * ns);
            if (best.tile == 0 || cost < best.us) best = ExactPlan{kd.tile, kd.stream, ns, cost, kd.places};
        }
    }
    return best;
}

// For the choice between these kernels and others, whose lines were drawn with these times: as if two 128 x 128 workgroups on a CU were the only
// way.  (Of 8000 products 128 to 8192 wide 6 % are modelled more than 5 % too long by that, one 40 %.)
double gemm_exact_us(mst_dtype a_dt, int M, int N, int Kdim, int64_t max_split, bool summed) {
    return plan_exact(false, false, M, N, Kdim, a_dt == MST_BF16, max_split, summed).us;
}

int gemm_exact_tile(int tile) {
    g_exact_tile = tile;
    return MST_OK;
}

template <bool A16, bool AK, bool BKM>
static int launch_exact(const void* A, int64_t lda, const float* B, int64_t ldb, float* C, int M, int N, int Kdim,
                        float* split_ws, int64_t split_ws_floats, int* nparts, hipStream_t s, ActiveOut* active = nullptr) {
    const int64_t mn = (int64_t)M * N;
    const ExactPlan plan = plan_exact(true, AK, M, N, Kdim, A16, split_ws ? split_ws_floats / mn : 1, nparts == nullptr);
    const int kps = (int)(cdiv(cdiv(Kdim, plan.nsplit), 128) * 128);
    const int nsplit = (int)cdiv(Kdim, kps);
    const unsigned grid = (unsigned)(8 * cdiv(cdiv(M, plan.tile) * cdiv(N, plan.tile), 8) * nsplit);
    float* const dst = nsplit > 1 ? split_ws : C;
    constexpr unsigned lds = (ExOperand<A16, AK, 64>::PLANES + 3) * 8192;
    if (plan.stream && plan.tile == 32) {
        k_gemm_stream<A16, AK, false, BKM, 1><<<grid, 1024, STREAM_LDS_32, s>>>(A, lda, B, ldb, dst, M, N, Kdim, kps, mn);
    } else if (plan.stream) {
        static uint64_t done = 0;
        const int rc = allow_lds(reinterpret_cast<const void*>(&k_gemm_stream<A16, AK, false, BKM, 2>), STREAM_LDS_64, done);
        if (rc != MST_OK) return rc;
        k_gemm_stream<A16, AK, false, BKM, 2><<<grid, 512, STREAM_LDS_64, s>>>(A, lda, B, ldb, dst, M, N, Kdim, kps, mn);
    } else if (plan.tile == 128) {
        constexpr bool CAN = AK && BKM && !A16;
        int64_t stride = mn;
        ActiveRuns runs{};
        if constexpr (CAN) {
            const int rc = active_runs(active, s, runs, stride);
            if (rc != MST_OK) return rc;
        }
        const bool only = runs.words != nullptr;
        float* const to = only && nsplit == 1 ? active->dW : dst;
        if constexpr (A16) {
            k_gemm_exact<A16, AK, BKM, 128, 0, false><<<grid, 256, lds, s>>>(A, lda, B, ldb, to, M, N, Kdim, kps, stride, runs);
        } else {
            const auto three = only ? k_gemm_exact<A16, AK, BKM, 128, 3, CAN> : k_gemm_exact<A16, AK, BKM, 128, 3, false>;
            if (plan.places == 96) three<<<grid, 256, lds + (only ? 4096u : 0u), s>>>(A, lda, B, ldb, to, M, N, Kdim, kps, stride, runs);
            else if constexpr (AK) three<<<grid, 256, 56u << 10, s>>>(A, lda, B, ldb, to, M, N, Kdim, kps, stride, runs);     // (the LDS of three)
            else k_gemm_exact<A16, AK, BKM, 128, 2, false><<<grid, 256, 56u << 10, s>>>(A, lda, B, ldb, to, M, N, Kdim, kps, stride, runs);
        }
    } else {
        k_gemm_exact<A16, AK, BKM, 64, 0, false><<<grid, 256, lds, s>>>(A, lda, B, ldb, dst, M, N, Kdim, kps, mn, ActiveRuns{});
    }
    MST_LAUNCH_CHECK();
    if (nparts) {
        *nparts = nsplit;
        return MST_OK;
    }
    return nsplit > 1 ? sum_split_planes(split_ws, mn, nsplit, C, mn, s) : MST_OK;
}

// C = A^T B, both bfloat16 and k-major, on 64 x 64 tiles; k_per_split a multiple of 64
int gemm_stream_tn_bf16(const uint16_t* A, const uint16_t* B, float* C, int M, int N, int Kdim, int k_per_split, int64_t split_stride,
                        hipStream_t s) {
    static uint64_t done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(&k_gemm_stream<true, true, true, true, 2>), STREAM_LDS_64, done);
    if (rc != MST_OK) return rc;
    const unsigned grid = (unsigned)(8 * cdiv(cdiv(M, 64) * cdiv(N, 64), 8) * cdiv(Kdim, k_per_split));
    k_gemm_stream<true, true, true, true, 2><<<grid, 512, STREAM_LDS_64, s>>>(A, M, B, N, C, M, N, Kdim, k_per_split, split_stride);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

int gemm_exact(GemmKind kind, const void* A, mst_dtype a_dt, const float* B, float* C, int M, int N, int Kdim,
               float* split_ws, int64_t split_ws_floats, hipStream_t s, int* nparts, ActiveOut* active) {
    const bool a16 = a_dt == MST_BF16;
    if (kind == GEMM_TN) return a16 ? MST_ERR_ARG : launch_exact<false, true, true>(A, M, B, N, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s, active);
    if (kind == GEMM_NT)
        return a16 ? launch_exact<true, false, false>(A, Kdim, B, Kdim, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s)
                   : launch_exact<false, false, false>(A, Kdim, B, Kdim, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s);
    return a16 ? launch_exact<true, false, true>(A, Kdim, B, N, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s)
               : launch_exact<false, false, true>(A, Kdim, B, N, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s);
}

}  // namespace mst
