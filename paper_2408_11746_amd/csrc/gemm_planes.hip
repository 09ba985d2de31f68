// Y = X Wd^T and dX = dY Wd of whole 256 x 256 tiles with bfloat16 activations and weights that are split already: a layer
// keeps the two bfloat16 parts of its dense weights (W = hi + lo, the parts of split_bf16.h) beside the fp32 copy, once for
// either product, in the order in which a workgroup wants them in LDS.  Nothing of a step passes through registers: both
// operands go straight to LDS (global_load_lds_dwordx4, 16 bytes per lane), a term is a.lo + a.hi, two MFMAs.
// The kernel that split W anew in every workgroup (one conversion per 256 outputs of a weight, loads and LDS stores through
// registers) gave the same bits and was bound by that staging: T = 16384 at density 0.05, 1024 -> 4096: Y 296 -> 234 us, dX 309
// -> 233; 4096 -> 1024: Y 265 -> 197, dX 277 -> 198; the GPT-2-medium block's step 2089 -> 1795 us.
// What bounds it now: a step of 32 k takes 2650 clocks where its products need 2048, at 1.8 GHz (the clock that the matrix
// cores leave), and the 256 KB of outputs of every workgroup 6.5 us that nothing else of its CU fills.
// The same for fp32 activations (X still split while it is staged) was tried and is not used: 3 % faster at 1280 -> 5120,
// half dense, nothing at 768 -> 3072 and 10 %, where making the planes after every change of the weights costs more.
//
// Planes of the rows r of S (S = Wd for Y, Wd^T for dX), contraction index k: 128 bytes per row and 32 k, first the hi
// parts, then the lo parts.
#include "common.h"
#include "split_bf16.h"

namespace mst {

constexpr int PK = 32;                                // k of a step; an LDS row is 64 bytes
constexpr int P_PLANE = 256 * 64, P_STAGE = 3 * P_PLANE;
constexpr unsigned P_LDS = 3 * P_STAGE;               // three stages of [A, B hi, B lo]

// LDS position of unit u (eight k) of row m inside a plane; see ex_unit in gemm_exact.hip
__device__ __forceinline__ uint32_t plane_unit(int m, int u) {
    const int rho = (m & ~15) | ((m & 3) << 2) | ((m >> 2) & 3);
    return (uint32_t)(rho * 64 + (((u ^ (rho >> 2) ^ (rho >> 4)) & 3) << 4));
}
// Eight wavefronts (2 x 4) of 128 x 64; the loads of a step are issued two steps ahead, one barrier per step.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_planes(const uint16_t* __restrict__ A, const uint16_t* __restrict__ P, float* __restrict__ C, int M, int N, int Kdim) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 2) * 128, wn = (wave & 3) * 64;
    // XCD x takes a contiguous share of the tiles
    const int gm = M / 256, gn = N / 256, ntiles = gm * gn, Q = (ntiles + 7) >> 3;
    const int tile_id = (blockIdx.x & 7) * Q + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= Q || tile_id >= ntiles) return;
    int mi, ni;
    tile_coords(tile_id, gm, gn, mi, ni);
    const int m0 = mi * 256, n0 = ni * 256, nsteps = Kdim / PK;

    // A wavefront's instruction fills 16 rows of a plane, two groups of 16 per wavefront and plane.  Lane l writes the place of
    // row `row` of the sixteen and of position l & 3, so it reads the unit that belongs there.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const int rho = lane >> 2, row = ((rho & 3) << 2) | (rho >> 2);
    const char* const pa = reinterpret_cast<const char*>(A + (int64_t)m0 * Kdim);
    const char* const pb = reinterpret_cast<const char*>(P) + (int64_t)n0 * Kdim * 4;
    uint32_t va[2], vb[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int g = 2 * wave + j;
        const uint32_t u = ((lane & 3) ^ (rho >> 2) ^ g) & 3;
        va[j] = (uint32_t)(16 * g + row) * (uint32_t)(2 * Kdim) + 16u * u;
        vb[j] = (uint32_t)(16 * g + row) * (uint32_t)(4 * Kdim) + 16u * u;
    }
    constexpr int EACH = 6;                           // loads of a wavefront per step
    auto load = [&](int t, uint32_t stage) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t at = lds0 + stage + 1024u * (2 * wave + j);
            load_to_lds(pa + 64 * (int64_t)t, va[j], at);
            load_to_lds(pb + 128 * (int64_t)t, vb[j], at + P_PLANE);
            load_to_lds(pb + 128 * (int64_t)t + 64, vb[j], at + 2 * P_PLANE);
        }
    };
    floatx16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // operand reads: lane = row of a tile of 32 rows and a unit; tile i of the wavefront 2048 bytes on, its swizzle by the
    // parity of its number
    const int lr = lane & 31, lu = lane >> 5;
    uint32_t fo[2][2];
#pragma unroll
    for (int x = 0; x < 4; ++x) fo[x >> 1][x & 1] = plane_unit(32 * (x & 1) + lr, 2 * (x >> 1) + lu) - 2048u * (x & 1);
    load(0, 0);
    if (nsteps > 1) load(1, P_STAGE);
    uint32_t cur = 0, next = 2 * P_STAGE;             // the stage in use, the one two steps on
#pragma unroll 1
    for (int t = 0; t < nsteps; ++t) {
        if (t + 1 < nsteps) wait_loads<EACH>();       // (those of the next step may still be on the way)
        else wait_loads<0>();
        lds_barrier();
        if (t + 2 < nsteps) load(t + 2, next);        // into the stage that the step before has read
        const char* const a_ = lds + cur + wm * 64;
        const char* const b_ = lds + cur + P_PLANE + wn * 64;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 a[4], b[2][2];                     // b: [part][tile]
#pragma unroll
            for (int j = 0; j < 2; ++j) b[1][j] = *reinterpret_cast<const bf16x8*>(b_ + P_PLANE + fo[ks][j] + 2048 * j);
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const bf16x8*>(a_ + fo[ks][i & 1] + 2048 * i);
#pragma unroll
            for (int j = 0; j < 2; ++j) b[0][j] = *reinterpret_cast<const bf16x8*>(b_ + fo[ks][j] + 2048 * j);
#pragma unroll
            for (int z = 1; z >= 0; --z)              // a.lo, then a.hi
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[z][j], a[i], acc[i][j], 0, 0, 0);
        }
        const uint32_t was = cur;
        cur = cur == 2 * P_STAGE ? 0 : cur + P_STAGE;
        next = was;
    }
    // D layout of the 32x32 MFMA: lane l, register v -> row 8*(v/4) + 4*(l/32) + v%4 (B's), column l%32 (A's)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float* const c = C + (int64_t)(m0 + wm + 32 * i + lr) * N + n0 + wn + 4 * lu;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 o;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = acc[i][j][4 * q + v];
                *reinterpret_cast<floatx4*>(c + 32 * j + 8 * q) = o;
            }
    }
}

// C [M x N] = A [M x K] S^T, S given by its planes; M, N multiples of 256, K of 32
int gemm_planes(const uint16_t* A, const uint16_t* P, float* C, int M, int N, int Kdim, hipStream_t s) {
    if (!P || M % 256 || N % 256 || Kdim % PK) return MST_ERR_ARG;
    static uint64_t done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(&k_gemm_planes), P_LDS, done);
    if (rc != MST_OK) return rc;
    k_gemm_planes<<<(unsigned)(8 * cdiv((int64_t)(M / 256) * (N / 256), 8)), 512, P_LDS, s>>>(A, P, C, M, N, Kdim);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

// ---- the planes of Wd [O x I] for Y (rows o) and for dX (rows i), O and I multiples of 32: a workgroup reads a tile of
// 64 x 64 once.  Bound by the 12 bytes per position.
__global__ __launch_bounds__(256) void k_make_planes(const float* __restrict__ W, int O, int I, uint16_t* __restrict__ Py, uint16_t* __restrict__ Px) {
    __shared__ float t[64][65];
    const int tid = threadIdx.x, i0 = blockIdx.x * 64, o0 = blockIdx.y * 64;
    const int c4 = 4 * (tid & 15), r16 = tid >> 4;
    auto store = [&](uint16_t* P, int row, int k, int K, float x0, float x1, float x2, float x3) __attribute__((always_inline)) {
        uint32_t h0, l0, h1, l1;
        split_pair(x0, x1, h0, l0);
        split_pair(x2, x3, h1, l1);
        uint16_t* const q = P + ((int64_t)row * (K / 32) + k / 32) * 64 + (k & 31);
        *reinterpret_cast<uint2*>(q) = make_uint2(h0, h1);
        *reinterpret_cast<uint2*>(q + 32) = make_uint2(l0, l1);
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = o0 + 16 * r + r16, i = i0 + c4;
        if (o >= O || i >= I) continue;
        const float4 v = *reinterpret_cast<const float4*>(W + (int64_t)o * I + i);
        store(Py, o, i, I, v.x, v.y, v.z, v.w);
        t[16 * r + r16][c4] = v.x;
        t[16 * r + r16][c4 + 1] = v.y;
        t[16 * r + r16][c4 + 2] = v.z;
        t[16 * r + r16][c4 + 3] = v.w;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + 16 * r + r16, o = o0 + c4, x = 16 * r + r16;
        if (i < I && o < O) store(Px, i, o, O, t[c4][x], t[c4 + 1][x], t[c4 + 2][x], t[c4 + 3][x]);
    }
}

int make_planes(const mst_layer* L, hipStream_t s) {
    k_make_planes<<<dim3((unsigned)cdiv(L->I, 64), (unsigned)cdiv(L->O, 64)), 256, 0, s>>>(L->Wd, L->O, L->I, L->planes_y, L->planes_x);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

}  // namespace mst
