// Dense products of any shape at full fp32 precision on the bf16 matrix cores.
//
// Every fp32 operand element is cut, while it is staged, into three bfloat16 values hi + mid + lo of
// eight significant bits each: x = hi + mid + lo exactly (truncation: no rounding, no overflow).  A
// product is hi.hi + hi.mid + mid.hi + mid.mid + hi.lo + lo.hi with fp32 accumulation; what is dropped
// is below 2^-24 of it, less than the rounding of one fp32 product.  A bfloat16 operand is one
// value, so bfloat16 x fp32 takes three products per term, all exact.
//
// C[M x N] = sum_k A'[k][m] B'[k][n]; each operand k-major (element (k, m) at src[k*ld + m]) or m-major
// (src[m*ld + k]).  Serves the shapes whose tiles are not whole (an activation batch of any length, a
// layer of any size): they used to run on v_mfma_f32_32x32x2f32 at 100 TFLOP/s.  Six
// v_mfma_f32_32x32x16_bf16 take the place of eight of those at a sixteenth of the time each.
//
// Workgroup tile TM x TM, TM = 128 or 64, 256 threads = four wavefronts of (TM/2) x (TM/2); k steps of
// 4096 / TM, so that a plane of an operand's tile is 8 KB and a workgroup's LDS 48 KB (32 KB with a
// bfloat16 operand): two (three) workgroups share a CU and one's staging runs beside another's MFMAs.
// Loads are buffer loads from the tile's corner with exact ends: rows past the matrix read as zeros
// without an access, a 16-byte load needs dword alignment only, so no leading dimension is special.
// What lies past the end of a row is the next row (finite); it lands in outputs that are not stored,
// or, along k, is cleared in the last step.  Bound: the matrix cores (six products per term; a large
// bf16 product runs at 1294 TFLOP/s on this card, that is 215 of these); the 128 tile pulls 1/6 of the
// operand bytes per MFMA of a plain bf16 kernel.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "split_bf16.h"

namespace mst {

typedef uint32_t ex_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t ex_u32x2 __attribute__((ext_vector_type(2)));

// LDS position of unit u (eight k) of row m in a plane of rows of 32 k (64 bytes) or 64 k (128 bytes)
template <int TM>
__device__ inline uint32_t ex_unit(int m, int u) {
    if (TM == 64) return bf_unit(m, u);
    const int rho = (m & ~15) | ((m & 3) << 2) | ((m >> 2) & 3);
    return (uint32_t)(rho * 64 + (((u ^ (rho >> 2) ^ (rho >> 4)) & 3) << 4));
}

// a pair of fp32 values as three words of two bfloat16 each
__device__ inline void cut_pair(float x0, float x1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    constexpr uint32_t UPPER = 0x07060302u;
    const uint32_t a0 = __float_as_uint(x0), a1 = __float_as_uint(x1);
    hi = __builtin_amdgcn_perm(a1, a0, UPPER);
    const uint32_t b0 = __float_as_uint(x0 - __uint_as_float(a0 & 0xFFFF0000u)), b1 = __float_as_uint(x1 - __uint_as_float(a1 & 0xFFFF0000u));
    mid = __builtin_amdgcn_perm(b1, b0, UPPER);
    const float c0 = __uint_as_float(b0) - __uint_as_float(b0 & 0xFFFF0000u), c1 = __uint_as_float(b1) - __uint_as_float(b1 & 0xFFFF0000u);
    lo = __builtin_amdgcn_perm(__float_as_uint(c1), __float_as_uint(c0), UPPER);
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

    // rows (k-major: k, m-major: m) of the tile past the end are cut off by the descriptor
    __device__ __forceinline__ void fetch(const T* __restrict__ src, int64_t ld, int k0, int m0, int kend, int Mdim, int p) {
        const int64_t corner = KMAJOR ? (int64_t)k0 * ld + m0 : (int64_t)m0 * ld + k0;
        const int64_t left = KMAJOR ? (int64_t)min(kend - k0, BK) * ld - m0 : (int64_t)min(Mdim - m0, TM) * ld - k0;   // elements
        const uint32_t bytes = (uint32_t)((left * (int64_t)sizeof(T) + 3) & ~3ll);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src + corner), 0, (int)bytes, 0x00020000);
        const uint32_t pitch = (uint32_t)ld * (uint32_t)sizeof(T);
        if constexpr (KMAJOR) {
            static_assert(!BF16, "a bfloat16 operand is m-major");
            const uint32_t o = (uint32_t)(8 * (p / (TM / 2))) * pitch + (uint32_t)(8 * (p % (TM / 2)));
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const ex_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(o + kk * pitch), 0, 0);
                f[2 * kk] = __uint_as_float(v.x);
                f[2 * kk + 1] = __uint_as_float(v.y);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int idx = j * 256 + p, m = idx / UNITS, u = idx % UNITS;
                const uint32_t o = (uint32_t)m * pitch + (uint32_t)(8 * u) * (uint32_t)sizeof(T);
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
                const int valid = kend - (k0 + 8 * ((j * 256 + p) % UNITS));      // k of this unit that exist
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
            uint32_t a;
            if constexpr (KMAJOR) a = ex_unit<TM>(2 * (p % (TM / 2)) + j, p / (TM / 2));
            else a = ex_unit<TM>((j * 256 + p) / UNITS, (j * 256 + p) % UNITS);
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
//
// KG: groups of four wavefronts that share one output tile and take its k steps in turn, each with LDS
// planes of its own; their sums are added in order at the end.  With one group a step costs at least
// the latency of its loads (1.3 us however few products it has), so where there are fewer tiles than CUs
// three groups of a 64 x 64 tile fill a CU's LDS and have three steps on the way.
template <bool A16, bool A_KMAJOR, bool B_KMAJOR, int TM, int KG>
__global__ __launch_bounds__(256 * KG) __attribute__((amdgpu_waves_per_eu(2, 3)))
void k_gemm_exact(const void* __restrict__ Av, int64_t lda, const float* __restrict__ B, int64_t ldb, float* __restrict__ C,
                  int M, int N, int Kdim, int k_per_split, int64_t split_stride) {
    typedef ExOperand<A16, A_KMAJOR, TM> OpA;
    typedef ExOperand<false, B_KMAJOR, TM> OpB;
    constexpr int BK = 4096 / TM, PLANE = 8192, MI = TM / 64;
    constexpr int GROUP_LDS = (OpA::PLANES + OpB::PLANES) * PLANE;
    extern __shared__ __attribute__((aligned(16))) char ex_lds[];
    const int group = KG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) : 0;
    char* const la = ex_lds + group * GROUP_LDS;
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

    const int tid = threadIdx.x & 255, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
    // rounds of one step per group; only in the last one a group may have no step, or one that ends at kend
    const int rounds = (kend - kbeg + BK * KG - 1) / (BK * KG);
    int k0 = kbeg + group * BK;
    if (KG == 1 || k0 < kend) fetch(k0);
    for (int r = 1; r < rounds; ++r) {
        __syncthreads();
        stage();
        __syncthreads();
        k0 += BK * KG;
        if (KG == 1 || k0 < kend) fetch(k0);
        multiply();
    }
    __syncthreads();
    if (KG == 1 || k0 < kend) {
        ra.clear_tail(k0, kend, tid);
        rb.clear_tail(k0, kend, tid);
        stage();
    }
    __syncthreads();
    if (KG == 1 || k0 < kend) multiply();
    if constexpr (CHAINS > 1)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][0][v] += other[v];
    if constexpr (KG > 1) {
        static_assert(MI == 1, "one MFMA tile per wavefront");
        float* const sums = reinterpret_cast<float*>(ex_lds);
        __syncthreads();
        if (group > 0)
#pragma unroll
            for (int v = 0; v < 16; ++v) sums[((group - 1) * 16 + v) * 256 + tid] = acc[0][0][v];
        __syncthreads();
        if (group > 0) return;
#pragma unroll
        for (int z = 0; z < KG - 1; ++z)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[0][0][v] += sums[(z * 16 + v) * 256 + tid];
    }
    // D layout of the 32x32 MFMA: lane l, register v -> row 8*(v/4) + 4*(l/32) + v%4, column l%32
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + wm + i * 32 + 8 * (v >> 2) + 4 * lk + (v & 3);
                const int n = n0 + wn + j * 32 + lm;
                if (m < M && n < N) Cz[(int64_t)m * N + n] = acc[i][j][v];
            }
}

// Workgroup tile, wavefront groups and number of k ranges together, as for the split kernels: modelled
// time = rounds one XCD needs for its share of the tiles x time of a workgroup (k steps, start-up and output
// counted in steps), plus the traffic of the partial outputs.  Places of an XCD: 64 workgroups of
// 128 x 128, 96 of 64 x 64 (32 with three groups).  Microseconds of a step with all places taken
// and with a CU to itself, from timings at ten shapes on MI355X.
struct ExactPlan {
    int tile, groups, nsplit;
};
static int g_exact_tile = 0;                          // test hook: 0 automatic, 64, 128, or 192: 64 with three groups
static ExactPlan plan_exact(int M, int N, int Kdim, bool a16, int64_t max_split, bool summed) {
    struct Kind {
        int tile, groups, places, lone_places;
        double start;                                 // start-up and output of a workgroup, in steps
        double full[2], lone[2];                      // fp32, bfloat16 A
    };
    static const Kind kinds[] = {{128, 1, 64, 32, 4.0, {2.6, 1.4}, {1.87, 1.0}},
                                 {64, 1, 96, 32, 4.0, {2.65, 1.4}, {1.45, 0.95}},
                                 {64, 3, 32, 32, 3.0, {2.3, 1.65}, {2.3, 1.65}}};
    static const int cand[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
    ExactPlan best{0, 1, 1};
    double best_cost = 0.0;
    for (const Kind& kd : kinds) {
        if (g_exact_tile && kd.tile * kd.groups != g_exact_tile) continue;
        const int bk = 4096 / kd.tile;
        const int64_t Q = cdiv(cdiv(M, kd.tile) * cdiv(N, kd.tile), 8);
        for (int ns : cand) {
            if (ns > 1 && (ns > max_split || Kdim / ns < 256)) continue;
            const double steps = (double)cdiv(cdiv(cdiv(Kdim, ns), bk), kd.groups);
            const int64_t n = Q * ns, rest = n % kd.places;
            if (kd.groups > 1 && n > kd.places && !g_exact_tile) continue;    // more than a round of tiles: one group each
            const double full = kd.full[a16], lone = kd.lone[a16];
            // (a last round that leaves places empty is shorter: the workgroups of a CU share its matrix cores)
            const double last = rest == 0 ? 0.0 : rest <= kd.lone_places ? lone
                : lone + (full - lone) * (double)(rest - kd.lone_places) / (double)(kd.places - kd.lone_places);
            double cost = ((double)(n / kd.places) * full + last) * (steps + kd.start);
            if (ns > 1) cost += 3.0 + 1.0e-6 * (double)M * (double)N * (summed ? ns + 1.0 : 0.25 * ns);
            if (best.tile == 0 || cost < best_cost) {
                best_cost = cost;
                best = ExactPlan{kd.tile, kd.groups, ns};
            }
        }
    }
    return best;
}

int gemm_exact_tile(int tile) {
    g_exact_tile = tile;
    return MST_OK;
}

template <bool A16, bool AK, bool BKM>
static int launch_exact(const void* A, int64_t lda, const float* B, int64_t ldb, float* C, int M, int N, int Kdim,
                        float* split_ws, int64_t split_ws_floats, int* nparts, hipStream_t s) {
    const int64_t mn = (int64_t)M * N;
    const ExactPlan plan = plan_exact(M, N, Kdim, A16, split_ws ? split_ws_floats / mn : 1, nparts == nullptr);
    const int bk = 4096 / plan.tile;
    const int kps = (int)(cdiv(cdiv(Kdim, plan.nsplit), bk) * bk);
    const int nsplit = (int)cdiv(Kdim, kps);
    const unsigned grid = (unsigned)(8 * cdiv(cdiv(M, plan.tile) * cdiv(N, plan.tile), 8) * nsplit);
    float* const dst = nsplit > 1 ? split_ws : C;
    constexpr unsigned lds = (ExOperand<A16, AK, 64>::PLANES + 3) * 8192;
    if (plan.tile == 128) {
        k_gemm_exact<A16, AK, BKM, 128, 1><<<grid, 256, lds, s>>>(A, lda, B, ldb, dst, M, N, Kdim, kps, mn);
    } else if (plan.groups == 1) {
        k_gemm_exact<A16, AK, BKM, 64, 1><<<grid, 256, lds, s>>>(A, lda, B, ldb, dst, M, N, Kdim, kps, mn);
    } else {
        static uint64_t done = 0;
        const int rc = allow_lds(reinterpret_cast<const void*>(&k_gemm_exact<A16, AK, BKM, 64, 3>), 3 * lds, done);
        if (rc != MST_OK) return rc;
        k_gemm_exact<A16, AK, BKM, 64, 3><<<grid, 768, 3 * lds, s>>>(A, lda, B, ldb, dst, M, N, Kdim, kps, mn);
    }
    MST_LAUNCH_CHECK();
    if (nparts) {
        *nparts = nsplit;
        return MST_OK;
    }
    return nsplit > 1 ? sum_split_planes(split_ws, mn, nsplit, C, mn, s) : MST_OK;
}

int gemm_exact(GemmKind kind, const void* A, mst_dtype a_dt, const float* B, float* C, int M, int N, int Kdim,
               float* split_ws, int64_t split_ws_floats, hipStream_t s, int* nparts) {
    const bool a16 = a_dt == MST_BF16;
    if (kind == GEMM_TN) return a16 ? MST_ERR_ARG : launch_exact<false, true, true>(A, M, B, N, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s);
    if (kind == GEMM_NT)
        return a16 ? launch_exact<true, false, false>(A, Kdim, B, Kdim, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s)
                   : launch_exact<false, false, false>(A, Kdim, B, Kdim, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s);
    return a16 ? launch_exact<true, false, true>(A, Kdim, B, N, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s)
               : launch_exact<false, false, true>(A, Kdim, B, N, C, M, N, Kdim, split_ws, split_ws_floats, nparts, s);
}

}  // namespace mst
