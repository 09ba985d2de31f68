// Dense fp32 products of any shape at full precision on the fp16 matrix cores, for outputs of many tiles.
//
// A row of an operand (all its k) gets a scale, a power of two, and every scaled value y is kept as two fp16 values,
// hi = fp16(y) and lo = fp16(y - hi), both rounded to nearest: 11 + 11 significant bits and lo's sign hold fp32's 24
// but for half of an fp32 ulp in the root mean square.  A product is lo.hi + hi.lo + hi.hi with fp32 accumulation
// (lo.lo is at most 2^-24 of it and has no direction): three matrix instructions where the three bfloat16 parts of
// gemm_exact.hip take six.  The splitting of an operand into scaled fp16 parts follows Ootomo and Yokota 2022, "Recovering
// single precision accuracy from Tensor Cores while surpassing the FP32 theoretical peak performance".
// Root mean square error of Y at 8192 x 1280 -> 5120 in units of 2^-24 sum |x w|: 256 tile 0.29, 128 tile 0.17;
// six products on a 128 tile (what served these shapes before) 0.41, two bfloat16 parts 3.3.
//
// Scales.  fp16 keeps lo in full only down to 2^-1 of a scaled value and ends at 2^16, so a row is scaled to where its
// values are: of the first step whose tiles are not zero throughout, each of the row's four units of eight k has
// a largest magnitude, and the smallest of these that is not zero goes to [2^6, 2^7).  (The smallest of the four: a single
// outlier does not set the scale.)  A value 2^-9 of that loses nothing, smaller ones an absolute 2^-25 of the scaled range.
// A step with a scaled value of 65000 or more, or where three of four patches of a wavefront have shrunk below 2^-2, ends
// the fast loop: that step and those after it take the values as three bfloat16 parts, which have fp32's range, six products
// per term (about the time of the kernel this one replaces).  Infinities and NaN end up as outputs that are not finite; those
// are formed again by fp32 multiply-adds, as in gemm_exact.hip.
//
// What bounds it: with random operands in all of them the matrix instructions pull the clock down to 1.6 GHz; in clocks a
// 32-k step of the 256 tile takes 4300 where its 192 products per SIMD need 3072.  900 of the rest are the staging (seven
// vector instructions per pair of values beside matrix instructions that keep the vector ALU out for 10 of their 16
// clocks), 270 the LDS reads.  5001 x 1000 -> 4000: Y 268 us with six products, 182 on this 256 tile and 205 on the 128 tile;
// dX (80 tiles of 256) 309, 280, 220; dense gradient 249, 158, 216.  A training step of this layer, half dense: 701 -> 564 us.
#include <algorithm>

#include "common.h"
#include "split_bf16.h"

namespace mst {

typedef uint32_t gh_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t gh_u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int HK = 32;                                // k of a step: an LDS row is 64 bytes, four units of eight k
constexpr float HALF_TOP = 65000.f, HALF_LOW = 0.25f;

// LDS position of unit u of row m inside a plane: the two low bit pairs of m swapped inside its group of 16, the unit
// swizzled.  Operand reads of 16 or 32 consecutive rows and the stores of both layouts then cover all banks once.
__device__ __forceinline__ uint32_t half_unit(int m, int u) {
    const int rho = (m & ~15) | ((m & 3) << 2) | ((m >> 2) & 3);
    return (uint32_t)(rho * 64 + (((u ^ (rho >> 2) ^ (rho >> 4)) & 3) << 4));
}

__device__ __forceinline__ void half_pair(float y0, float y1, uint32_t& hi, uint32_t& lo) {
    const f16x2 h = __builtin_convertvector((floatx2){y0, y1}, f16x2);
    const f16x2 l = __builtin_convertvector((floatx2){y0 - (float)h.x, y1 - (float)h.y}, f16x2);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

// One operand's registers between global memory and LDS: ROWS rows x 32 k of a tile, staged by THREADS threads p.  A
// piece is one unit (eight k of one row) in both planes; a thread stages NP of them, all with the same k: k-major the
// patch of eight k x NP consecutive rows, m-major NP rows THREADS / 4 apart.
template <bool KMAJOR, int ROWS, int THREADS>
struct HalfOperand {
    static constexpr int NP = ROWS * 4 / THREADS, PLANE = ROWS * 64, PATCHES = ROWS / NP;
    static_assert(NP == 2 || NP == 4, "");
    float f[8 * NP];
    float scale[NP];
    uint32_t hw[4], lw[4];

    __device__ __forceinline__ float& at(int j, int d) { return KMAJOR ? f[NP * d + j] : f[8 * j + d]; }
    __device__ static __forceinline__ int row(int p, int j) {
        if (KMAJOR) return NP * (p % PATCHES) + j;
        return THREADS / 4 * j + 16 * (p >> 6) + 4 * ((p >> 2) & 3) + ((p >> 4) & 3);
    }
    __device__ static __forceinline__ int unit(int p) { return KMAJOR ? p / PATCHES : p & 3; }

    // rows (k-major: k, m-major: m) of the tile past the end are cut off by the descriptor; a step past the end reads zeros.
    // What lies past the end of a row is the next row: it lands in outputs that are not stored, or, along k, is cleared.
    __device__ __forceinline__ void fetch(const float* __restrict__ src, int64_t ld, int k0, int o0, int kend, int dim, int p) {
        const bool any = k0 < kend;
        const int64_t corner = KMAJOR ? (int64_t)k0 * ld + o0 : (int64_t)o0 * ld + k0;
        const int64_t left = KMAJOR ? (int64_t)min(kend - k0, HK) * ld - o0 : (int64_t)min(dim - o0, ROWS) * ld - k0;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(src + (any ? corner : 0)), 0, any ? (int)(4 * left) : 0, 0x00020000);
        const uint32_t pitch = 4u * (uint32_t)ld;
        uint32_t o = KMAJOR ? 8u * (uint32_t)unit(p) * pitch + 4u * (uint32_t)row(p, 0) : (uint32_t)row(p, 0) * pitch + 32u * (uint32_t)unit(p);
        asm volatile("" : "+v"(o));                   // (every load's offset kept across the loop would not fit the registers)
        if constexpr (KMAJOR) {
#pragma unroll
            for (int d = 0; d < 8; ++d, o += pitch) {
                if constexpr (NP == 4) {
                    const gh_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o, 0, 0);
#pragma unroll
                    for (int x = 0; x < 4; ++x) f[4 * d + x] = __uint_as_float(v[x]);
                } else {
                    const gh_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, 0, 0);
                    f[2 * d] = __uint_as_float(v.x);
                    f[2 * d + 1] = __uint_as_float(v.y);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < NP; ++j, o += THREADS / 4 * pitch)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const gh_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(o + 16 * q), 0, 0);
#pragma unroll
                    for (int x = 0; x < 4; ++x) f[8 * j + 4 * q + x] = __uint_as_float(v[x]);
                }
        }
    }
    __device__ __forceinline__ void clear_tail(int k0, int kend, int p) {
        if constexpr (!KMAJOR) {
            const int valid = kend - k0 - 8 * unit(p);
#pragma unroll
            for (int j = 0; j < NP; ++j)
#pragma unroll
                for (int d = 0; d < 8; ++d) f[8 * j + d] = d < valid ? f[8 * j + d] : 0.f;
        }
    }
    // per unit and row the largest magnitude as bits (those of a NaN above all); mx [4][ROWS]
    __device__ __forceinline__ void maxima(uint32_t* mx, int p) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            uint32_t m = 0;
#pragma unroll
            for (int d = 0; d < 8; ++d) m = max(m, __float_as_uint(at(j, d)) & 0x7FFFFFFFu);
            mx[ROWS * unit(p) + row(p, j)] = m;
        }
    }
    __device__ __forceinline__ void take_scales(const int* e, int p) {
#pragma unroll
        for (int j = 0; j < NP; ++j) scale[j] = ldexpf(1.f, e[row(p, j)]);
    }
    __device__ static __forceinline__ uint32_t address(int p, int j) { return half_unit(row(p, j), unit(p)); }
    // pair q of piece j; its units leave after the fourth.  top: the largest scaled magnitude
    __device__ __forceinline__ void put_pair(char* lds, uint32_t a, int j, int q, float& top) {
        const float y0 = at(j, 2 * q) * scale[j], y1 = at(j, 2 * q + 1) * scale[j];
        top = fmaxf(fmaxf(__builtin_fabsf(y0), __builtin_fabsf(y1)), top);
        half_pair(y0, y1, hw[q], lw[q]);
        if (q == 3) {
            *reinterpret_cast<uint4*>(lds + a) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
            *reinterpret_cast<uint4*>(lds + PLANE + a) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
        }
    }
    // the first and (part 0) the third or (1) the second of three bfloat16 parts
    __device__ __forceinline__ void put_wide(char* lds, int p, int part) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            uint32_t a[4], b[4], c[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) cut_pair(at(j, 2 * q) * scale[j], at(j, 2 * q + 1) * scale[j], a[q], b[q], c[q]);
            const uint32_t u = address(p, j);
            *reinterpret_cast<uint4*>(lds + u) = make_uint4(a[0], a[1], a[2], a[3]);
            *reinterpret_cast<uint4*>(lds + PLANE + u) = part ? make_uint4(b[0], b[1], b[2], b[3]) : make_uint4(c[0], c[1], c[2], c[3]);
        }
    }
};

// what a row's scale goes by: the smallest of its four units' largest magnitudes that is not zero
template <int ROWS>
__device__ __forceinline__ uint32_t row_size(const uint32_t* mx, int r) {
    uint32_t m = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t x = mx[ROWS * u + r];
        m = x > 0 && (m == 0 || x < m) ? x : m;
    }
    return m;
}
// exponent of the scale of a row of that size; a row that is zero so far goes by the largest of its tile
__device__ __forceinline__ int scale_exponent(uint32_t size, int largest) {
    const uint32_t of = size > 0 ? size : (uint32_t)largest;
    return of > 0 ? min(126, 133 - (int)(of >> 23)) : 0;
}
// a staged tile is out of the range of its scales (uniform decisions are made after the next barrier, from LDS)
__device__ __forceinline__ bool out_of_range(float top) {
    return top >= HALF_TOP || __popcll(__ballot(top > 0.f && top < HALF_LOW)) >= 48;
}

// Output of a wavefront whose outputs that are not finite are formed again
template <bool AK, bool BKM>
__device__ __forceinline__ void form_again(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, float* c,
                                           int m, int n, int kbeg, int kend) {
    if (!(__builtin_fabsf(*c) < __builtin_inff())) *c = fp32_sum<float, AK, float, BKM>(A, lda, B, ldb, m, n, kbeg, kend);
}
// Where N is no multiple of four a wavefront's outputs leave by way of LDS, 32 rows x COLS at a time, so that a store writes a run
// of 256 bytes: element by element every lane of an accumulator would write to a row of its own.  2379 x 2025, k = 512,
// 128 x 128 tiles: 49 -> 39 us (2379 x 2024, four outputs per lane and store: 35, and no less through LDS).
// Unit u (four columns) of row r is kept at u ^ (r & 15); only this wavefront uses the area.
template <int COLS>
__device__ __forceinline__ uint32_t out_unit(int r, int u) { return (uint32_t)(r * (COLS * 4) + ((u ^ (r & 15)) << 4)); }
__device__ __forceinline__ void wave_lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <int COLS>
__device__ __forceinline__ void store_rows(const char* area, float* __restrict__ C, int m0, int n0, int M, int N, int lane) {
    wave_lds_done();
#pragma unroll 8
    for (int x = 0; x < 32 * COLS / 64; ++x) {
        const int r = x / (COLS / 64), c = x % (COLS / 64) * 64 + lane;
        if (m0 + r < M && n0 + c < N) C[(int64_t)(m0 + r) * N + n0 + c] = *reinterpret_cast<const float*>(area + out_unit<COLS>(r, c >> 2) + 4 * (c & 3));
    }
    wave_lds_done();
}

// Workgroup -> (tile, k range): XCD x takes a contiguous share of the tiles, one k range after the other; tiles in bands of
// `band` tile rows, column by column inside a band, so that the tiles an XCD works on at a time share operand panels in its L2
__device__ __forceinline__ bool half_tile(int TM, int band, int M, int N, int Kdim, int k_per_split, int& m0, int& n0, int& split) {
    const int gm = (M + TM - 1) / TM, gn = (N + TM - 1) / TM, ntiles = gm * gn;
    const int nsplit = (Kdim + k_per_split - 1) / k_per_split, Q = (ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int tile_id = xcd * Q + slot % Q;
    split = slot / Q;
    if (tile_id >= ntiles || split >= nsplit) return false;
    const int bd = tile_id / (band * gn), rem = tile_id - bd * band * gn, hgt = min(band, gm - bd * band);
    m0 = (bd * band + rem % hgt) * TM;
    n0 = (rem / hgt) * TM;
    return true;
}

// ---- 256 x 256 tiles: eight wavefronts (4 x 2) of 64 x 128, two LDS stages of 64 KB, one barrier per step.  The
// products are v_mfma_f32_16x16x32_f16 (16 rows of W or X each way; with random operands in all of them they run at 1735
// TFLOP/s from LDS where the 32x32x16 form reaches 1530), rows of B as the rows of the result: a lane then holds
// four consecutive outputs.  The next tile's conversions and LDS stores are slipped between the products of the second half
// of a step.  Operands of one layout: threads 0..255 stage A, the others B; otherwise every thread stages two pieces
// of each.
constexpr int H256_PLANE = 256 * 64, H256_STAGE = 4 * H256_PLANE;
constexpr unsigned H256_LDS = 2 * H256_STAGE + 512 * 4 + 16;

template <bool AK, bool BKM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_half256(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, float* __restrict__ C,
                    int M, int N, int Kdim, int k_per_split, int64_t split_stride) {
    constexpr bool MIXED = AK != BKM;
    typedef HalfOperand<AK, 256, MIXED ? 512 : 256> OpA;
    typedef HalfOperand<BKM, 256, MIXED ? 512 : 256> OpB;
    extern __shared__ __attribute__((aligned(16))) char gh_lds[];      // two stages [A hi, A lo, B hi, B lo], tables
    int* const expo = reinterpret_cast<int*>(gh_lds + 2 * H256_STAGE);  // [512] exponents of the scales, A's rows and B's
    int* const flags = expo + 512;                                      // [0..1] a step out of range, [2..3] largest of A, B
    int m0, n0, split;
    if (!half_tile(256, 4, M, N, Kdim, k_per_split, m0, n0, split)) return;
    const int kbeg = split * k_per_split, kend = min(Kdim, kbeg + k_per_split), nsteps = (kend - kbeg + HK - 1) / HK;
    float* const Cz = C + (int64_t)split * split_stride;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 128;
    const int h = __builtin_amdgcn_readfirstlane(tid >> 8);            // equal layouts: the operand this thread stages

    OpA ra;                                           // (equal layouts: either operand's)
    OpB rb;
    auto mine = [&](int tid) __attribute__((always_inline)) { return MIXED ? tid : tid & 255; };
    auto fetch = [&](int t, int p) __attribute__((always_inline)) {
        const int k0 = kbeg + t * HK;
        if constexpr (MIXED) {
            ra.fetch(A, lda, k0, m0, kend, M, p);
            rb.fetch(B, ldb, k0, n0, kend, N, p);
        } else {
            ra.fetch(h == 0 ? A : B, h == 0 ? lda : ldb, k0, h == 0 ? m0 : n0, kend, h == 0 ? M : N, p);
        }
    };
    auto clear_tail = [&](int t, int p) __attribute__((always_inline)) {
        const int k0 = kbeg + t * HK;
        if (k0 + HK <= kend) return;
        ra.clear_tail(k0, kend, p);
        if constexpr (MIXED) rb.clear_tail(k0, kend, p);
    };
    uint32_t at[4];                                   // LDS addresses of this thread's four pieces inside a stage
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if constexpr (MIXED) at[j] = j < 2 ? OpA::address(tid, j) : 2 * H256_PLANE + OpB::address(tid, j - 2);
        else at[j] = 2 * H256_PLANE * h + OpA::address(tid & 255, j);
    }
    float top = 0.f;
    auto put_pair = [&](char* stage, int x) __attribute__((always_inline)) {       // pair x & 3 of piece x >> 2
        const int j = x >> 2;
        if constexpr (MIXED) {
            if (j < 2) ra.put_pair(stage, at[j], j, x & 3, top);
            else rb.put_pair(stage, at[j], j - 2, x & 3, top);
        } else {
            ra.put_pair(stage, at[j], j, x & 3, top);
        }
    };
    auto report = [&](int t) __attribute__((always_inline)) {
        if (out_of_range(top)) flags[t & 1] = t;
        top = 0.f;
    };
    floatx4 acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
    // operand reads: lane = row of a tile of 16 rows and a unit; tile x of the wavefront 1024 bytes on, its swizzle by x & 3
    uint32_t fo[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) fo[x] = half_unit(16 * x + (lane & 15), lane >> 4) - 1024u * x;

    auto step = [&](char* cur, char* nxt) __attribute__((always_inline)) {
        const char* const pa = cur + wm * 64;
        const char* const pb = cur + 2 * H256_PLANE + wn * 64;
        f16x8 a[2][4], b[2][2];                       // a: [part][tile]; b: [column parity][part], the next column's come while this one's are used
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[0][i] = *reinterpret_cast<const f16x8*>(pa + fo[i] + 1024 * i);
            a[1][i] = *reinterpret_cast<const f16x8*>(pa + H256_PLANE + fo[i] + 1024 * i);
        }
        auto column = [&](int j) __attribute__((always_inline)) {
            b[j & 1][0] = *reinterpret_cast<const f16x8*>(pb + fo[j & 3] + 1024 * j);
            b[j & 1][1] = *reinterpret_cast<const f16x8*>(pb + H256_PLANE + fo[j & 3] + 1024 * j);
        };
        column(0);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j < 7) column(j + 1);
#pragma unroll
            for (int e = 0; e < 12; ++e) {
                const int pr = e >> 2, i = e & 3;     // lo.hi, hi.lo, hi.hi
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b[j & 1][pr == 1], a[pr == 0][i], acc[i][j], 0, 0, 0);
                if (j >= 4 && e % 3 == 2) put_pair(nxt, 4 * (j - 4) + e / 3);
                if (e % 3 == 2) __builtin_amdgcn_sched_barrier(0x24);
            }
        }
    };

    // scales, from the first step whose tiles are not zero throughout
    if (tid < 2) flags[tid] = -1;
    int t = 0;
    uint32_t* const mx = reinterpret_cast<uint32_t*>(gh_lds);          // [A, B][4][256]
#pragma unroll 1
    while (true) {
        fetch(t, mine(tid));
        clear_tail(t, mine(tid));
        __syncthreads();
        if (tid < 2) flags[2 + tid] = 0;
        if constexpr (MIXED) {
            ra.maxima(mx, tid);
            rb.maxima(mx + 1024, tid);
        } else {
            ra.maxima(mx + 1024 * h, tid & 255);
        }
        __syncthreads();
        const uint32_t size = row_size<256>(mx + 1024 * h, tid & 255);
        if (size > 0) atomicMax(&flags[2 + h], (int)size);
        __syncthreads();
        if (t == nsteps - 1 || (flags[2] != 0 && flags[3] != 0)) {
            expo[tid] = scale_exponent(size, flags[2 + h]);
            break;
        }
        ++t;
    }
    __syncthreads();
    if constexpr (MIXED) {
        ra.take_scales(expo, tid);
        rb.take_scales(expo + 256, tid);
    } else {
        ra.take_scales(expo + 256 * h, tid & 255);
    }
    if (t > 0) {
        fetch(0, mine(tid));
        clear_tail(0, mine(tid));
    }
#pragma unroll
    for (int x = 0; x < 16; ++x) put_pair(gh_lds, x);
    report(0);
    fetch(1, mine(tid));
    __syncthreads();
    // where the run of fast steps ends for now
    auto last_good = [&](int t) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(flags[t & 1]) == t ? t : nsteps; };
    int stop = last_good(0);
#pragma unroll 1
    for (t = 0; t < stop; ++t) {                      // (the last step stages a tile of zeros)
        if (t == nsteps - 2) clear_tail(t + 1, mine(tid));
        step(gh_lds + (t & 1) * H256_STAGE, gh_lds + (~t & 1) * H256_STAGE);
        report(t + 1);
        fetch(t + 2, mine(tid));
        __syncthreads();
        stop = last_good(t + 1);
    }
    // (the accumulators change hands here: otherwise the compiler copies all of them in every step of the loop above)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(acc[i][j]));
    int own = tid;
    asm volatile("" : "+v"(own));                     // nothing below stays in registers across the loop above
    const int lr = own & 15, lu = (own >> 4) & 3;
#pragma unroll 1
    for (; t < nsteps; ++t) {                         // three bfloat16 parts
        fetch(t, mine(own));
        clear_tail(t, mine(own));
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            __syncthreads();
            if constexpr (MIXED) {
                ra.put_wide(gh_lds, own, pass);
                rb.put_wide(gh_lds + 2 * H256_PLANE, own, pass);
            } else {
                ra.put_wide(gh_lds + 2 * H256_PLANE * h, own & 255, pass);
            }
            __syncthreads();
#pragma unroll 1
            for (int pr = pass ? 0 : 1; pr < (pass ? 4 : 3); ++pr) {   // hi and lo: lo.hi, hi.lo; hi and mid: mid.mid, mid.hi, hi.mid, hi.hi
                const char* const pa = gh_lds + (pr < 2 ? H256_PLANE : 0);
                const char* const pb = gh_lds + 2 * H256_PLANE + ((pr & 1) ? 0 : H256_PLANE);
                bf16x8 a[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const bf16x8*>(pa + half_unit(wm + 16 * i + lr, lu));
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bf16x8 b = *reinterpret_cast<const bf16x8*>(pb + half_unit(wn + 16 * j + lr, lu));
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[i], acc[i][j], 0, 0, 0);
                }
            }
        }
    }
    // D layout of the 16x16 MFMA: lane l, register v -> row 4*(l/16) + v (B's), column l%16 (A's)
    bool bad = false;
    const bool rows_aligned = (N & 3) == 0;
    char* const area = gh_lds + 16384 * (own >> 6);
    __syncthreads();                                  // (everyone is done with the operands there)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + wm + 16 * i + lr, ea = expo[wm + 16 * i + lr];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = n0 + wn + 16 * j + 4 * lu;
            floatx4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                bad |= !(__builtin_fabsf(acc[i][j][v]) < __builtin_inff());
                o[v] = ldexpf(acc[i][j][v], -ea - expo[256 + wn + 16 * j + 4 * lu + v]);
            }
            if (!rows_aligned) *reinterpret_cast<floatx4*>(area + out_unit<128>(16 * (i & 1) + lr, 4 * j + lu)) = o;
            else if (m < M && n < N) *reinterpret_cast<floatx4*>(Cz + (int64_t)m * N + n) = o;
        }
        if ((i & 1) && !rows_aligned) store_rows<128>(area, Cz, m0 + wm + 16 * (i - 1), n0 + wn, M, N, own & 63);
    }
    if (bad) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (other lanes have stored this lane's outputs)
#pragma unroll 1
        for (int x = 0; x < 128; ++x) {
            const int m = m0 + wm + 16 * (x >> 5) + lr, n = n0 + wn + 16 * ((x >> 2) & 7) + 4 * lu + (x & 3);
            if (m < M && n < N) form_again<AK, BKM>(A, lda, B, ldb, Cz + (int64_t)m * N + n, m, n, kbeg, kend);
        }
    }
}

// ---- 128 x 128 tiles, for outputs that 256 x 256 leave CUs idle: four wavefronts of 64 x 64 on one LDS stage of 32 KB; two
// workgroups share a CU and one's staging runs beside another's products.  lo.hi and hi.lo have accumulators
// of their own, so the sum of hi.hi is rounded once per 16 k (error 0.17 where one chain of three products has 0.29,
// for 5 % of the time).
constexpr int H128_PLANE = 128 * 64;
constexpr unsigned H128_LDS = 4 * H128_PLANE + 256 * 4 + 16;

template <bool AK, bool BKM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3)))
void k_gemm_half128(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, float* __restrict__ C,
                    int M, int N, int Kdim, int k_per_split, int64_t split_stride) {
    typedef HalfOperand<AK, 128, 256> OpA;
    typedef HalfOperand<BKM, 128, 256> OpB;
    extern __shared__ __attribute__((aligned(16))) char gh_lds[];      // A hi, A lo, B hi, B lo, tables
    char* const la = gh_lds;
    char* const lb = gh_lds + 2 * H128_PLANE;
    int* const expo = reinterpret_cast<int*>(gh_lds + 4 * H128_PLANE);  // [256], as above
    int* const flags = expo + 256;
    int m0, n0, split;
    if (!half_tile(128, 8, M, N, Kdim, k_per_split, m0, n0, split)) return;
    const int kbeg = split * k_per_split, kend = min(Kdim, kbeg + k_per_split), nsteps = (kend - kbeg + HK - 1) / HK;
    float* const Cz = C + (int64_t)split * split_stride;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;

    OpA ra;
    OpB rb;
    auto fetch = [&](int t, int p) __attribute__((always_inline)) {
        ra.fetch(A, lda, kbeg + t * HK, m0, kend, M, p);
        rb.fetch(B, ldb, kbeg + t * HK, n0, kend, N, p);
    };
    auto clear_tail = [&](int t, int p) __attribute__((always_inline)) {
        const int k0 = kbeg + t * HK;
        if (k0 + HK <= kend) return;
        ra.clear_tail(k0, kend, p);
        rb.clear_tail(k0, kend, p);
    };
    floatx16 acc[2][2], cross[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = cross[i][j][v] = 0.f;

    if (tid < 2) flags[tid] = -1;
    int t = 0;
    uint32_t* const mx = reinterpret_cast<uint32_t*>(gh_lds);          // [A, B][4][128]
    const int side = tid >> 7;
#pragma unroll 1
    while (true) {
        fetch(t, tid);
        clear_tail(t, tid);
        __syncthreads();
        if (tid < 2) flags[2 + tid] = 0;
        ra.maxima(mx, tid);
        rb.maxima(mx + 512, tid);
        __syncthreads();
        const uint32_t size = row_size<128>(mx + 512 * side, tid & 127);
        if (size > 0) atomicMax(&flags[2 + side], (int)size);
        __syncthreads();
        if (t == nsteps - 1 || (flags[2] != 0 && flags[3] != 0)) {
            expo[tid] = scale_exponent(size, flags[2 + side]);
            break;
        }
        ++t;
    }
    __syncthreads();
    ra.take_scales(expo, tid);
    rb.take_scales(expo + 128, tid);
    if (t > 0) {
        fetch(0, tid);
        clear_tail(0, tid);
    }
    auto stage = [&](int t) __attribute__((always_inline)) {
        float top = 0.f;
#pragma unroll
        for (int x = 0; x < 8; ++x) ra.put_pair(la, OpA::address(tid, x >> 2), x >> 2, x & 3, top);
#pragma unroll
        for (int x = 0; x < 8; ++x) rb.put_pair(lb, OpB::address(tid, x >> 2), x >> 2, x & 3, top);
        if (out_of_range(top)) flags[t & 1] = t;
    };
    const int lane = tid & 63;
    auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            f16x8 a[2][2], b[2][2];                   // [part][tile]
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t ua = half_unit(wm + 32 * i + (lane & 31), 2 * ks + (lane >> 5)), ub = half_unit(wn + 32 * i + (lane & 31), 2 * ks + (lane >> 5));
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    a[z][i] = *reinterpret_cast<const f16x8*>(la + z * H128_PLANE + ua);
                    b[z][i] = *reinterpret_cast<const f16x8*>(lb + z * H128_PLANE + ub);
                }
            }
#pragma unroll
            for (int pr = 0; pr < 3; ++pr)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        floatx16& c = pr < 2 ? cross[i][j] : acc[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[pr == 1][j], a[pr == 0][i], c, 0, 0, 0);
                    }
        }
    };
    stage(0);
    __syncthreads();
    auto last_good = [&](int t) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(flags[t & 1]) == t ? t : nsteps; };
    int stop = last_good(0);
#pragma unroll 1
    for (t = 0; t < stop; ++t) {
        fetch(t + 1, tid);
        multiply();
        __syncthreads();
        clear_tail(t + 1, tid);
        stage(t + 1);
        __syncthreads();
        stop = last_good(t + 1);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            acc[i][j] += cross[i][j];
            asm volatile("" : "+v"(acc[i][j]));
        }
    int own = tid;
    asm volatile("" : "+v"(own));
    const int lr = own & 31, lu = (own >> 5) & 1;
#pragma unroll 1
    for (; t < nsteps; ++t) {                         // three bfloat16 parts
        fetch(t, own);
        clear_tail(t, own);
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            __syncthreads();
            ra.put_wide(la, own, pass);
            rb.put_wide(lb, own, pass);
            __syncthreads();
#pragma unroll 1
            for (int pr = pass ? 0 : 1; pr < (pass ? 4 : 3); ++pr) {
                const char* const pa = la + (pr < 2 ? H128_PLANE : 0);
                const char* const pb = lb + ((pr & 1) ? 0 : H128_PLANE);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    bf16x8 a[2], b[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        a[i] = *reinterpret_cast<const bf16x8*>(pa + half_unit(wm + 32 * i + lr, 2 * ks + lu));
                        b[i] = *reinterpret_cast<const bf16x8*>(pb + half_unit(wn + 32 * i + lr, 2 * ks + lu));
                    }
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
                }
            }
        }
    }
    // D layout of the 32x32 MFMA: lane l, register v -> row 8*(v/4) + 4*(l/32) + v%4 (B's), column l%32 (A's)
    bool bad = false;
    const bool rows_aligned = (N & 3) == 0;
    char* const area = gh_lds + 8192 * (own >> 6);
    __syncthreads();                                  // (everyone is done with the operands there)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = m0 + wm + 32 * i + lr, ea = expo[wm + 32 * i + lr];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int nl = wn + 32 * j + 8 * q + 4 * lu;
                floatx4 o;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float c = acc[i][j][4 * q + v];
                    bad |= !(__builtin_fabsf(c) < __builtin_inff());
                    o[v] = ldexpf(c, -ea - expo[128 + nl + v]);
                }
                if (!rows_aligned) *reinterpret_cast<floatx4*>(area + out_unit<64>(lr, 8 * j + 2 * q + lu)) = o;
                else if (m < M && n0 + nl < N) *reinterpret_cast<floatx4*>(Cz + (int64_t)m * N + n0 + nl) = o;
            }
        if (!rows_aligned) store_rows<64>(area, Cz, m0 + wm + 32 * i, n0 + wn, M, N, own & 63);
    }
    if (bad) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (other lanes have stored this lane's outputs)
#pragma unroll 1
        for (int x = 0; x < 64; ++x) {
            const int m = m0 + wm + 32 * (x >> 5) + lr, n = n0 + wn + 32 * ((x >> 4) & 1) + 8 * ((x >> 2) & 3) + 4 * lu + (x & 3);
            if (m < M && n < N) form_again<AK, BKM>(A, lda, B, ldb, Cz + (int64_t)m * N + n, m, n, kbeg, kend);
        }
    }
}

template <bool AK, bool BKM>
static int launch_half(int tile, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int M, int N, int Kdim,
                       int k_per_split, int64_t split_stride, hipStream_t s) {
    const unsigned grid = (unsigned)(8 * cdiv(cdiv(M, tile) * cdiv(N, tile), 8) * cdiv(Kdim, k_per_split));
    if (tile == 256) {
        static uint64_t done = 0;
        const int rc = allow_lds(reinterpret_cast<const void*>(&k_gemm_half256<AK, BKM>), H256_LDS, done);
        if (rc != MST_OK) return rc;
        k_gemm_half256<AK, BKM><<<grid, 512, H256_LDS, s>>>(A, lda, B, ldb, C, M, N, Kdim, k_per_split, split_stride);
    } else {
        k_gemm_half128<AK, BKM><<<grid, 256, H128_LDS, s>>>(A, lda, B, ldb, C, M, N, Kdim, k_per_split, split_stride);
    }
    MST_LAUNCH_CHECK();
    return MST_OK;
}

int gemm_half(GemmKind kind, int tile, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int M, int N, int Kdim,
              int k_per_split, int64_t split_stride, hipStream_t s) {
    if (kind == GEMM_TN) return launch_half<true, true>(tile, A, lda, B, ldb, C, M, N, Kdim, k_per_split, split_stride, s);
    if (kind == GEMM_NT) return launch_half<false, false>(tile, A, lda, B, ldb, C, M, N, Kdim, k_per_split, split_stride, s);
    return launch_half<false, true>(tile, A, lda, B, ldb, C, M, N, Kdim, k_per_split, split_stride, s);
}

}  // namespace mst
