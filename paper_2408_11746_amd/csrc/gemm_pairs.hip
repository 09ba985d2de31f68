// Y = X Wd^T and dX = dY Wd at densities of about a tenth and below on the sparse matrix instructions
// (v_smfmac_f32_32x32x32_bf16): of every four consecutive k a row of the weights holds two values and two 2-bit
// selectors, and the instruction covers 32 k in the 32 clocks in which the dense one covers 16.  Operands, parts and products are
// those of the dense kernels (two bfloat16 parts per fp32 operand: lo.hi, hi.lo, hi.hi; bfloat16 activations: lo, hi).
//
// A row with three entries among four k does not fit.  At density 0.1 that is one quad in 270, somewhere in 61 % of the tiles
// of 32 rows x 32 k, and a second pass over those would take back most of the gain.  So the quads are chosen:  the
// activations go to LDS by dwords (two k, as bfloat16) anyway, and for every band of 256 rows and step of 64 k the 32 dwords are
// paired up so that the fewest rows overflow (k_match_pairs: greedy, then exchanges between two quads).  Up to density 0.08 that
// leaves nothing, at 0.10 one step in ten with a few overflowing rows, at 0.12 five in six.  What is left goes to a second step of the
// same 64 k with the third and fourth entries, walked after the others by the wavefronts that have any: every mask is exact.
//
// A workgroup: one band x 128 tokens (fp32) or 256, 192, 128 tokens (bfloat16), eight wavefronts of 64 rows x half the tokens;
// two LDS stages of 64 k, one barrier per step.
//   - Everything passes through registers, packed weights too: an operand is loaded one or two steps before its way to LDS,
//     each piece right behind the store that freed its registers, between the products (loads in front of the step held the
//     matrix cores up for 1000 clocks; straight to LDS, all loads of a step had to arrive within it: 1280 <- 5120, 0.1, 8192 tokens,
//     cold activations 270 us, so 248).
//   - The operands of a step's last products are in registers when the wavefronts meet, so the first ones of the next step are
//     read beside them (Y of 1280 -> 5120, 0.05: 203 -> 189 us).
// Measured (us, before = the dense kernels; 8192 tokens, fp32, 0.10): Y of 1280 -> 5120 281 -> 196, dX of it 304 -> 223; Y of 768 ->
// 3072 114 -> 90, dX of it 123 -> 92.  16384 tokens, bfloat16, 0.05: Y of 1024 -> 4096 234 -> 144, dX 198 -> 118.
// What bounds it: the matrix cores take 18 ns an instruction with the whole chip on them (1.75 GHz), 0.86 of the 1.4 us of a
// step of fp32 and 1.15 of the 1.95 of bfloat16; the conversions and stores of the activations between the products (10 %), and the
// outputs of all workgroups at once (7 to 9 us a round) are the most of the rest.
#include <type_traits>
#include <utility>

#include "common.h"
#include "split_bf16.h"

namespace mst {

typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef uint32_t pk_u32x4 __attribute__((ext_vector_type(4)));

constexpr int PB_ROWS = 256, PB_TILES = PB_ROWS / 32;          // rows of a band, MFMA tiles of them
constexpr int PW_TILE = 2048, PW_SUB = PB_TILES * PW_TILE + PB_TILES * 128;   // [tile][hi 1 KB, lo 1 KB], [tile][64 lanes] selectors
constexpr int PK_STEP = 64, PK_PAIRS = PK_STEP / 2, PK_BLOCK = 2 * PW_SUB;    // k of a step, packed bytes of a step

PairsView pairs_view(void* mem, int R, int K) {
    PairsView v;
    v.R = R;
    v.K = K;
    v.nk = (int)cdiv(K, PK_STEP);
    v.bands = (int)cdiv(R, PB_ROWS);
    const int64_t n = (int64_t)v.bands * v.nk;
    char* b = static_cast<char*>(mem);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return b ? b + o : nullptr; };
    v.slots = (uint8_t*)take((size_t)n * PK_PAIRS);
    v.flags = (uint32_t*)take((size_t)n * 4);
    v.over = (uint8_t*)take((size_t)n);
    v.count = (uint32_t*)take(8);
    v.blocks = take((size_t)n * 2 * PK_BLOCK);
    v.bytes = off;
    return v;
}

// ------------------------------------------------------------------ which dwords share a quad
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    // (lanes without a source keep their own value)
#define MST_MIN_DPP(CTRL, ROWS) x = min(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROWS, 0xf, false))
    MST_MIN_DPP(0x111, 0xf);                          // row_shr:1, 2, 4, 8
    MST_MIN_DPP(0x112, 0xf);
    MST_MIN_DPP(0x114, 0xf);
    MST_MIN_DPP(0x118, 0xf);
    MST_MIN_DPP(0x142, 0xa);                          // row_bcast:15 into rows 1 and 3
    MST_MIN_DPP(0x143, 0xc);                          // row_bcast:31 into rows 2 and 3
#undef MST_MIN_DPP
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// Block = (view, band, step); y first.  Bound by latencies: the mask's lines (all of a thread's loads go out together; eight pairs of them at a
// time and counts looked up lane by lane: 28 us at 5120 x 1280, so 22), then the search of one wavefront.
__global__ __launch_bounds__(256) void k_match_pairs(const uint8_t* __restrict__ mask, int I, const PairsView y, const PairsView x) {
    constexpr int NP = PK_PAIRS, NQ = NP / 2;
    __shared__ unsigned long long g1[NP][4], g2[NP][4];
    __shared__ uint16_t cost[NP][NP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool rows = blockIdx.x < (unsigned)(y.bands * y.nk);
    const PairsView& v = rows ? y : x;
    const unsigned at = rows ? blockIdx.x : blockIdx.x - (unsigned)(y.bands * y.nk);
    const int band = (int)(at / (unsigned)v.nk), kb = (int)(at - (unsigned)band * (unsigned)v.nk);
    const int r = band * PB_ROWS + tid, k0 = kb * PK_STEP;
    const bool in = r < v.R;
    // rows (bits of four words) with one, with two entries in a pair
    auto pair = [&](int p, bool a, bool b) {
        const unsigned long long one = __ballot(a || b), two = __ballot(a && b);
        if (lane == 0) { g1[p][wave] = one; g2[p][wave] = two; }
    };
    if (rows) {
        const uint8_t* m = mask + (int64_t)(in ? r : 0) * I + k0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 u = *reinterpret_cast<const uint4*>(m + 16 * q);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const uint32_t h = w[p >> 1] >> (16 * (p & 1));
                pair(8 * q + p, in && (h & 0xFFu) != 0, in && (h & 0xFF00u) != 0);
            }
        }
    } else {
        const uint8_t* m = mask + (int64_t)k0 * I + (in ? r : 0);
        uint8_t e[PK_STEP];                           // (all loads in flight before the first is looked at)
#pragma unroll
        for (int k = 0; k < PK_STEP; ++k) e[k] = m[(int64_t)k * I];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < NP; ++p) pair(p, in && e[2 * p] != 0, in && e[2 * p + 1] != 0);
    }
    // rows past the end: no weights (whatever is there reaches outputs that are not stored), selectors as of empty quads, no flags
    // (nothing else of the flags: a product that reads the same layer on another stream may be under way, and the packing behind this
    // launch writes what is there already)
    const int missing = (band + 1) * PB_ROWS - v.R;
    if (tid < 4 && 64 * tid >= PB_ROWS - missing) reinterpret_cast<uint8_t*>(v.flags + at)[tid] = 0;
    if (missing > 0)
        for (int e = tid; e < 4 * missing; e += 256) {       // [first, second step][32 k][missing rows]
            const int row = PB_ROWS - missing + e % missing, ss = e / missing;
            char* b = v.blocks + ((int64_t)band * 2 * v.nk + kb + (ss >> 1) * v.nk) * PK_BLOCK + (ss & 1) * PW_SUB + PB_TILES * PW_TILE;
            reinterpret_cast<uint16_t*>(b)[(row >> 5) * 64 + (row & 31)] = 0x4444u;
            reinterpret_cast<uint16_t*>(b)[(row >> 5) * 64 + 32 + (row & 31)] = 0x4444u;
        }
    __syncthreads();
    for (int e = tid; e < NP * NP; e += 256) {
        const int p = e / NP, q = e % NP;
        int c = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) c += __popcll((g2[p][w] & g1[q][w]) | (g1[p][w] & g2[q][w]));
        cost[p][q] = (uint16_t)c;
    }
    __syncthreads();
    if (wave != 0) return;
    // The cheapest pair of free dwords, sixteen times.  Lane: q = lane % 32, p = 2 j + lane / 32.
    uint32_t key[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
        const int p = 2 * j + (lane >> 5), q = lane & 31;
        key[j] = p < q ? (uint32_t)cost[p][q] << 16 | (uint32_t)p << 8 | (uint32_t)q : 0xFFFFFFFFu;
    }
    int total = 0, first = 0, second = 0;             // lane m (mod 16): quad m
    uint32_t used = 0;
    for (int m = 0; m < NQ; ++m) {
        uint32_t best = 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < NQ; ++j) best = min(best, (used >> (2 * j + (lane >> 5)) & 1u) ? 0xFFFFFFFFu : key[j]);
        if (used >> (lane & 31) & 1u) best = 0xFFFFFFFFu;
        best = wave_min(best);
        const uint32_t p = best >> 8 & 31u, q = best & 31u;
        total += (int)(best >> 16);
        used |= 1u << p | 1u << q;
        if ((lane & (NQ - 1)) == m) first = (int)p, second = (int)q;
    }
    // exchanges between two quads while one gains
    for (int round = 0; round < NQ && total > 0; ++round) {
        uint32_t best = 0xFFFFFFFFu;
        const int u = __shfl(first, lane >> 1 & (NQ - 1)), w = __shfl(second, lane >> 1 & (NQ - 1));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int e = 64 * j + lane, how = e & 1, a = (e >> 1) / NQ, b = (e >> 1) % NQ;
            const int p = __shfl(first, a), q = __shfl(second, a);
            const int gain = (int)cost[p][q] + cost[u][w] - (how ? (int)cost[p][w] + cost[q][u] : (int)cost[p][u] + cost[q][w]);
            if (a < b && gain > 0) best = min(best, (uint32_t)(0x7FFF - gain) << 16 | (uint32_t)e);
        }
        best = wave_min(best);
        if (best == 0xFFFFFFFFu) break;
        const int e = (int)(best & 0xFFFFu), how = e & 1, a = (e >> 1) / NQ, b = (e >> 1) % NQ, m = lane & (NQ - 1);
        const int qa = __builtin_amdgcn_readlane(second, a), ub = __builtin_amdgcn_readlane(first, b), wb = __builtin_amdgcn_readlane(second, b);
        if (m == a) second = how ? wb : ub;
        if (m == b) first = qa, second = how ? ub : wb;
        total -= 0x7FFF - (int)(best >> 16);
    }
    if (lane == 0) v.over[at] = total > 0 ? 1 : 0;
    // Where the quads go.  Four dwords that 32 lanes of the product's staging store together meet in no LDS bank if they are the four
    // dwords of 16 bytes, each of another such unit (see row0 there); which four go together differs with the activations' type.  So
    // each quad in turn takes the half of a unit, and its two dwords the order, that meet the fewest so far.  Lane g: dwords of
    // group g at each place of a unit; 0 <= g < 8 fp32 (line, half of its chunks, dword of a chunk), then bfloat16.  (Quads in the order
    // in which they were found, and rows that shared banks: 500 clocks of conflicts in a step of fp32, 815 of bfloat16; the products of
    // 1024 <-> 4096, 16384 tokens, bfloat16, 0.05: Y 150 -> 148.5 and dX 123 -> 120 us, fp32 within 1 %.)
    uint32_t met = 0;                                 // lane g: four counts of eight bits
    int taken[2] = {0, 0}, place = 0;                 // lane m: place of quad m's first dword
    for (int m = 0; m < NQ; ++m) {
        const int p = __builtin_amdgcn_readlane(first, m), q = __builtin_amdgcn_readlane(second, m);
        const int pf = (p >> 4) * 4 + (p >> 3 & 1) * 2 + (p & 1), pb = 8 + (p >> 4) * 4 + (p & 3);
        const int qf = (q >> 4) * 4 + (q >> 3 & 1) * 2 + (q & 1), qb = 8 + (q >> 4) * 4 + (q & 3);
        const uint32_t of_p = (uint32_t)(__builtin_amdgcn_readlane((int)met, pf) + __builtin_amdgcn_readlane((int)met, pb));
        const uint32_t of_q = (uint32_t)(__builtin_amdgcn_readlane((int)met, qf) + __builtin_amdgcn_readlane((int)met, qb));
        const uint32_t sum = of_p + ((of_q & 0x00FF00FFu) << 8 | (of_q >> 8 & 0x00FF00FFu));       // (q takes the place beside p's)
        uint32_t least = 0xFFFFFFFFu;
#pragma unroll
        for (uint32_t l = 0; l < 4; ++l)
            if (taken[l >> 1] < NQ / 2) least = min(least, (sum >> (8 * l) & 255u) << 2 | l);
        const int best = (int)(least & 3u), half = best >> 1, unit = half ? taken[1]++ : taken[0]++;
        met += (lane == pf || lane == pb ? 1u << (8 * best) : 0u) + (lane == qf || lane == qb ? 1u << (8 * (best ^ 1)) : 0u);
        if (lane == m) place = 4 * unit + best;
    }
    if (lane < NQ) {
        v.slots[(int64_t)at * NP + first] = (uint8_t)(4 * place);
        v.slots[(int64_t)at * NP + second] = (uint8_t)(4 * (place ^ 1));
    }
}

// ------------------------------------------------------------------ packing
// Block = 64 o x 64 i of the dense weights, read once for both views: two tiles of 32 rows of either, one step.  A wavefront
// packs a tile; lane = row and 16 k of every 32.  Bound by the 8.5 bytes per position that it reads and writes.
// first: the packing behind a choice of slots; block 0 counts the steps that go a second time (a launch of its own: four layers of a
// GPT-2-small block 19 us longer in the first pass on new masks).
__global__ __launch_bounds__(256) void k_pack_pairs(const float* __restrict__ W, int I, const PairsView y, const PairsView x, bool first) {
    constexpr int LD = PK_STEP + 1;
    __shared__ float tile[64 * LD];
    __shared__ uint8_t pair_s[2][PK_PAIRS];           // dword in a slot
    __shared__ uint32_t over_s[4];                    // tiles that need a second step
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int o0 = blockIdx.y * 64, i0 = blockIdx.x * 64;
    const bool of_x = wave >= 2;
    const PairsView& v = of_x ? x : y;
    const int r0 = of_x ? i0 : o0, band = r0 / PB_ROWS, kb = (of_x ? o0 : i0) / PK_STEP, t = (r0 % PB_ROWS) / 32 + (wave & 1);
    const int64_t bk = (int64_t)band * v.nk + kb;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int o = 16 * e + (tid >> 4), c = 4 * (tid & 15);
        const float4 w = *reinterpret_cast<const float4*>(W + (int64_t)(o0 + o) * I + i0 + c);
        float* p = tile + o * LD + c;
        p[0] = w.x; p[1] = w.y; p[2] = w.z; p[3] = w.w;
    }
    if ((wave & 1) == 0 && lane < PK_PAIRS) pair_s[wave >> 1][v.slots[bk * PK_PAIRS + lane] >> 2] = (uint8_t)lane;
    __syncthreads();
    const int row = 32 * (wave & 1) + (lane & 31), h = lane >> 5;
    // element (row, k) of this wavefront's view
    const float* const at = tile + (of_x ? row : row * LD);
    const int step = of_x ? LD : 1;
    const uint8_t* const ps = pair_s[wave >> 1];
    pk_u32x4 hi2[2], lo2[2];
    uint32_t ix2[2];
    bool over = false;
    char* const blk = v.blocks + ((int64_t)band * 2 * v.nk + kb) * PK_BLOCK;
    auto store = [&](char* b, pk_u32x4 hi, pk_u32x4 lo, uint32_t ix) {
        *reinterpret_cast<pk_u32x4*>(b + t * PW_TILE + lane * 16) = hi;
        *reinterpret_cast<pk_u32x4*>(b + t * PW_TILE + 1024 + lane * 16) = lo;
        *reinterpret_cast<uint16_t*>(b + PB_TILES * PW_TILE + t * 128 + lane * 2) = (uint16_t)ix;
    };
#pragma unroll
    for (int ss = 0; ss < 2; ++ss) {
        float f[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float* p = at + 2 * ps[16 * ss + 8 * h + i] * step;
            f[2 * i] = p[0];
            f[2 * i + 1] = p[step];
        }
        pk_u32x4 hi, lo;
        uint32_t ix = 0;
        ix2[ss] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float* g = f + 4 * q;
            uint32_t m = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) m |= (g[e] != 0.f ? 1u : 0u) << e;
            auto pick = [&](uint32_t i) { return i == 0 ? g[0] : i == 1 ? g[1] : i == 2 ? g[2] : g[3]; };
            // the two lowest entries of mm at ascending positions; a lone one beside a zero
            auto two = [&](uint32_t mm, float& a, float& b) {
                const uint32_t rest = mm & (mm - 1u);
                uint32_t p0 = mm ? (uint32_t)__ffs((int)mm) - 1u : 0u, p1 = rest ? (uint32_t)__ffs((int)rest) - 1u : 3u;
                a = mm ? pick(p0) : 0.f;
                b = rest ? pick(p1) : 0.f;
                if (p0 == 3u) { p0 = 0; b = a; a = 0.f; }
                return p0 | p1 << 2;
            };
            float a, b;
            uint32_t hh, ll;
            ix |= two(m, a, b) << (4 * q);
            split_pair(a, b, hh, ll);
            hi[q] = hh;
            lo[q] = ll;
            uint32_t m2 = m & (m - 1u);
            m2 &= m2 - 1u;
            over |= m2 != 0;
            ix2[ss] |= two(m2, a, b) << (4 * q);
            split_pair(a, b, hh, ll);
            hi2[ss][q] = hh;
            lo2[ss][q] = ll;
        }
        store(blk + ss * PW_SUB, hi, lo, ix);
    }
    const unsigned long long any = __ballot(over);
    if (lane == 0) over_s[wave] = any != 0ull;
    __syncthreads();
    // the two tiles go together
    const bool on = (over_s[wave] | over_s[wave ^ 1]) != 0;
    if (lane == 0 && (wave & 1) == 0) reinterpret_cast<uint8_t*>(v.flags + bk)[t >> 1] = on ? 1 : 0;
    if (first && blockIdx.x == 0 && blockIdx.y == 0) {            // (a wavefront each)
        const PairsView& of = wave == 0 ? y : x;
        if (wave < 2) {
            uint32_t c = 0;
            for (int e = lane; e < of.bands * of.nk; e += 64) c += of.over[e];
            for (int d = 32; d >= 1; d >>= 1) c += (uint32_t)__shfl_xor((int)c, d, 64);
            if (lane == 0) y.count[wave] = c;
        }
    }
    if (!on) return;
#pragma unroll
    for (int ss = 0; ss < 2; ++ss) store(blk + (int64_t)v.nk * PK_BLOCK + ss * PW_SUB, hi2[ss], lo2[ss], ix2[ss]);
}

// From the mask and the dense copy: the slots where the active set is a new one, and the blocks
int make_pairs(mst_layer* L, hipStream_t s) {
    const PairsView &y = L->pairs_y, &x = L->pairs_x;
    if (!L->pairs_matched) {
        k_match_pairs<<<(unsigned)(y.bands * y.nk + x.bands * x.nk), 256, 0, s>>>(L->mask, L->I, y, x);
        MST_LAUNCH_CHECK();
    }
    k_pack_pairs<<<dim3((unsigned)(L->I / 64), (unsigned)(L->O / 64)), 256, 0, s>>>(L->Wd, L->I, y, x, !L->pairs_matched);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

// ------------------------------------------------------------------ product
// Position of unit u (16 bytes: eight k) of row m inside a plane (64-byte rows)
__device__ __forceinline__ int pr_rho(int m) { return (m & ~15) | ((m & 3) << 2) | ((m >> 2) & 3); }
__device__ __forceinline__ uint32_t pr_unit(int m, int u) {
    const int rho = pr_rho(m);
    return (uint32_t)(rho * 64 + (((u ^ (rho >> 2) ^ (rho >> 4)) & 3) << 4));
}

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl(std::make_integer_sequence<int, N>{}, f); }

// NTK: tiles of 32 tokens of a wavefront; AHEAD: steps between the load of an operand and its way to LDS, a register set each
template <bool BF, int NTK, int AHEAD>
__device__ __forceinline__ void pairs_tile(const char* __restrict__ A, const PairsView& v, float* __restrict__ C, int T, int t0, int band, char* const lds) {
    constexpr int TOK = 64 * NTK, PLANE = TOK * 64, XST = (BF ? 2 : 4) * PLANE, STAGE = XST + PK_BLOCK;
    constexpr int LINES = BF ? 1 : 2, NX = NTK * LINES;           // 128-byte lines of a row in a step; 16-byte pieces of a thread
    uint16_t* const list = reinterpret_cast<uint16_t*>(lds + 2 * STAGE);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = v.nk;
    // steps of the second kind, in ascending order
    const uint32_t* const flags = v.flags + (int64_t)band * nk;
    int nsec = 0;
    for (int base = 0; base < nk; base += 64) {
        const bool on = base + lane < nk && flags[base + lane] != 0;
        const unsigned long long bal = __ballot(on);
        if (wave == 0 && on) list[nsec + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(base + lane);
        nsec += __popcll(bal);
    }
    nsec = __builtin_amdgcn_readfirstlane(nsec);
    __syncthreads();
    const int nv = nk + nsec;
    auto kblock = [&](int t) { return t < nk ? t : __builtin_amdgcn_readfirstlane((int)list[t - nk]); };

    // ---- staging: chunk of 16 bytes of row r0 + 64 it
    // (32 lanes: four chunks of eight rows whose positions in LDS, two in 128 bytes times four swizzles, put any dword of a
    // 64-byte row in eight different banks)
    const int chunk = (lane & 3) | (lane >> 5) << 2;
    const int row0 = (lane >> 2 & 7) + 8 * wave;
    const uint32_t pitch = (uint32_t)v.K * (BF ? 2u : 4u);
    const uint32_t rows = (uint32_t)min(T - t0, TOK);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(A + (int64_t)t0 * pitch), 0, (int)(rows * pitch), 0x00020000);
    const uint32_t xoff = (uint32_t)row0 * pitch + 16u * chunk;
    const uint32_t wbase = (uint32_t)pr_rho(row0) * 64u, wswz = (((uint32_t)pr_rho(row0) >> 2 ^ (uint32_t)pr_rho(row0) >> 4) & 3u) << 4;
    const char* const slots = reinterpret_cast<const char*>(v.slots) + (int64_t)band * nk * PK_PAIRS;
    const char* const wblk = v.blocks + (int64_t)band * 2 * nk * PK_BLOCK;

    // What a thread carries of a step: NX pieces of 16 bytes of the activations with the slots of their dwords, four pieces of
    // the packed weights and a dword of their selectors.  Operation n of a step: something goes to LDS, and what its
    // registers held is loaded AHEAD steps on.
    struct Carried {
        pk_u32x4 x[NX], w[4];
        uint32_t slot[LINES], sel;
    };
    struct Source {
        const char* w;
        int kb;
    };
    auto source = [&](int t) {
        t = min(t, nv - 1);                           // (past the end the last step again, into a stage that nobody reads)
        const int kb = kblock(t);
        return Source{wblk + (int64_t)(t < nk ? t : nk + kb) * PK_BLOCK, kb};
    };
    auto load_x = [&](Carried& f, const Source& src, int n) __attribute__((always_inline)) {
        f.x[n] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(xoff + (uint32_t)(64 * (n % NTK)) * pitch + 128u * (uint32_t)(src.kb * LINES + n / NTK)), 0, 0);
    };
    auto load_slot = [&](Carried& f, const Source& src, int line) __attribute__((always_inline)) {
        // (fp32: those of two chunks; a load of 16 bits would be widened, and waited for, where the loop closes)
        f.slot[line] = *reinterpret_cast<const uint32_t*>(slots + (int64_t)src.kb * PK_PAIRS + 16 * line + (BF ? 4 * chunk : 2 * (chunk & ~1)));
    };
    // (of a block [2][tiles, selectors]: 16 bytes at 1 KB (wave + 8 n) of the tiles, a dword of the selectors)
    const uint32_t wsel = (uint32_t)(PB_TILES * PW_TILE + (tid >> 8) * PW_SUB + 4 * (tid & 255));
    auto wpiece = [&](int n) { return (uint32_t)((n >> 1) * PW_SUB + 16 * (512 * (n & 1) + tid)); };
    auto load_w = [&](Carried& f, const Source& src, int n) __attribute__((always_inline)) {
        if (n < 4) f.w[n] = *reinterpret_cast<const pk_u32x4*>(src.w + wpiece(n));
        else f.sel = *reinterpret_cast<const uint32_t*>(src.w + wsel);
    };
    constexpr int HALF = (NTK + 1) / 2, NPUT = BF ? 4 * HALF : 4 * NTK, NOPS = NPUT + 5;
    auto operation = [&](Carried& f, uint32_t stage, const Source& next, auto nc) __attribute__((always_inline)) {
        constexpr int n = decltype(nc)::value;
        if constexpr (n >= NPUT) {
            constexpr int m = n - NPUT;
            if constexpr (m < 4) *reinterpret_cast<pk_u32x4*>(lds + stage + XST + wpiece(m)) = f.w[m];
            else *reinterpret_cast<uint32_t*>(lds + stage + XST + wsel) = f.sel;
            load_w(f, next, m);
        } else if constexpr (BF) {
            constexpr int e = n % 4, h = n / 4;               // dword e of pieces 2 h and 2 h + 1
            const uint32_t b = f.slot[0] >> (8 * e) & 255u;
            char* const p = lds + stage + wbase + 8192u * h + (b >> 6) * PLANE + ((b & 63u) ^ wswz);
            *reinterpret_cast<uint32_t*>(p) = f.x[2 * h][e];
            if (2 * h + 1 < NTK) *reinterpret_cast<uint32_t*>(p + 4096) = f.x[2 * h + 1 < NTK ? 2 * h + 1 : 0][e];
            if constexpr (e == 3) {
                load_x(f, next, 2 * h);
                if (2 * h + 1 < NTK) load_x(f, next, 2 * h + 1);
                if constexpr (h == HALF - 1) load_slot(f, next, 0);
            }
        } else {
            constexpr int e = n % 2, it = n / 2 % NTK, line = n / (2 * NTK);
            const uint32_t b = f.slot[line] >> (8 * e + 16 * (chunk & 1)) & 255u;
            const pk_u32x4& x = f.x[line * NTK + it];
            uint32_t hi, lo;
            split_pair(__uint_as_float(x[2 * e]), __uint_as_float(x[2 * e + 1]), hi, lo);
            char* const p = lds + stage + wbase + 4096u * it + (b >> 6) * (2 * PLANE) + ((b & 63u) ^ wswz);
            *reinterpret_cast<uint32_t*>(p) = hi;
            *reinterpret_cast<uint32_t*>(p + PLANE) = lo;
            if constexpr (e == 1) {
                load_x(f, next, line * NTK + it);
                if constexpr (it == NTK - 1) load_slot(f, next, line);
            }
        }
    };
    auto load_all = [&](Carried& f, const Source& src) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NX; ++n) load_x(f, src, n);
#pragma unroll
        for (int n = 0; n < LINES; ++n) load_slot(f, src, n);
#pragma unroll
        for (int n = 0; n < 5; ++n) load_w(f, src, n);
    };

    // ---- products: wavefront = 64 rows of the band x 32 NTK tokens
    const int wr = wave >> 1, wt = (wave & 1) * 32 * NTK;
    const int ln = lane & 31, lh = lane >> 5;
    uint32_t fx[2][2];                                // [unit 0 + lh, 2 + lh][parity of the tile]
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int par = 0; par < 2; ++par) fx[u][par] = pr_unit(32 * par + ln, 2 * u + lh) - 2048u * par;
    floatx16 acc[2][NTK];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NTK; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

    auto frag_x = [&](uint32_t stage, int plane, int j) __attribute__((always_inline)) {
        const int tile = (wt >> 5) + j;
        const char* p = lds + stage + plane * PLANE + 2048 * tile;
        // (NTK odd: the parity of the wavefront's first tile differs)
        const bf16x8 lo = *reinterpret_cast<const bf16x8*>(p + ((tile & 1) ? fx[0][1] : fx[0][0]));
        const bf16x8 hi = *reinterpret_cast<const bf16x8*>(p + ((tile & 1) ? fx[1][1] : fx[1][0]));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
    };
    constexpr int NZ = BF ? 2 : 3, NB = 2 * NTK;      // a block: the NZ products of 32 k with one token tile, for two row tiles
    bf16x8 w[2][2][2];                                // [set][part][row tile]
    int ix[2][2];
    bf16x16 x[2][BF ? 1 : 2];
    auto read_w = [&](auto set, uint32_t stage, int ss) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        const char* wp = lds + stage + XST + ss * PW_SUB;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int z = 0; z < 2; ++z) w[S][z][i] = *reinterpret_cast<const bf16x8*>(wp + (2 * wr + i) * PW_TILE + 1024 * z + 16 * lane);
            ix[S][i] = *reinterpret_cast<const uint16_t*>(wp + PB_TILES * PW_TILE + (2 * wr + i) * 128 + 2 * lane);
        }
    };
    auto read_x = [&](auto set, uint32_t stage, int b) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        if (BF) {
            x[S][0] = frag_x(stage, b / NTK, b % NTK);
        } else {
            x[S][0] = frag_x(stage, 2 * (b / NTK), b % NTK);
            x[S][BF ? 0 : 1] = frag_x(stage, 2 * (b / NTK) + 1, b % NTK);
        }
    };
    // block b of a step (weights in set b / NTK, activations in set b % 2; NB is even): `between` its products something else
    auto block = [&](auto bc, auto between) __attribute__((always_inline)) {
        constexpr int b = decltype(bc)::value, j = b % NTK, W = b / NTK, X = b & 1;
        static_for<2 * NZ>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value, z = m >> 1, i = m & 1;
            if constexpr (BF) acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(w[W][1 - z][i], x[X][0], acc[i][j], ix[W][i], 0, 0);
            else acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(w[W][z == 0 ? 1 : 0][i], x[X][z == 1 ? 1 : 0], acc[i][j], ix[W][i], 0, 0);
            between(mc);
            __builtin_amdgcn_sched_barrier(0x124);
        });
    };
    using zero = std::integral_constant<int, 0>;
    using one_ = std::integral_constant<int, 1>;

    Carried carried[AHEAD];
    load_all(carried[0], source(0));
    static_for<NOPS>([&](auto nc) __attribute__((always_inline)) { operation(carried[0], 0, source(1), nc); });
    if constexpr (AHEAD == 2) load_all(carried[AHEAD - 1], source(2));
    lds_barrier();
    read_w(zero{}, 0, 0);
    read_x(zero{}, 0, 0);
    // step t on stage cur, whose first operands are in registers: f holds step t + 1.  The operands of the last block are in
    // registers when everyone meets, so the first ones of the next step are read beside its products.
    // SECOND: the steps of the second kind (and a last odd one of the first), few, some of them without products for this
    // wavefront's rows.
    auto step = [&](int t, Carried& f, uint32_t cur, auto odd, auto second) __attribute__((always_inline)) {
        constexpr int ODD = decltype(odd)::value, SECOND = decltype(second)::value, NM = (NB - 1) * 2 * NZ;
        const uint32_t nxt = STAGE - cur;
        const bool mul = !SECOND || t < nk || (t < nv && (__builtin_amdgcn_readfirstlane((int)flags[kblock(t)]) >> (8 * wr) & 255) != 0);
        const Source next = source(t + 1 + AHEAD);
        if constexpr (SECOND) static_for<NOPS>([&](auto nc) __attribute__((always_inline)) { operation(f, nxt, next, nc); });
        if (mul) {
            static_for<NB - 1>([&](auto bc) __attribute__((always_inline)) {
                constexpr int b = decltype(bc)::value;
                __builtin_amdgcn_sched_barrier(0);
                read_x(std::integral_constant<int, (b + 1) & 1>{}, cur, b + 1);
                if constexpr (b == NTK - 1) read_w(one_{}, cur, 1);
                block(bc, [&](auto mc) __attribute__((always_inline)) {
                    constexpr int at = b * 2 * NZ + decltype(mc)::value;
                    if constexpr (!SECOND)
                        static_for<(at + 1) * NOPS / NM - at * NOPS / NM>([&](auto pc) __attribute__((always_inline)) {
                            operation(f, nxt, next, std::integral_constant<int, at * NOPS / NM + decltype(pc)::value>{});
                        });
                });
            });
        }
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
        read_w(zero{}, nxt, 0);
        read_x(zero{}, nxt, 0);
        if (mul) block(std::integral_constant<int, NB - 1>{}, [](auto) {});
    };
    int t = 0;
#pragma unroll 1
    for (; t + 2 <= nk; t += 2) {
        step(t, carried[0], 0, zero{}, zero{});
        step(t + 1, carried[AHEAD - 1], STAGE, one_{}, zero{});
    }
#pragma unroll 1
    for (; t < nv; t += 2) {
        step(t, carried[0], 0, zero{}, one_{});
        step(t + 1, carried[AHEAD - 1], STAGE, one_{}, one_{});
    }
    // D: lane l, register q -> row 8 (q / 4) + 4 (l / 32) + q % 4 of the band's tile, token l % 32.  The outputs leave through this
    // wavefront's part of LDS, 32 tokens x 64 rows at a time, in runs of 256 bytes past the L2 (768 -> 768, 8192 tokens: 30.2
    // us with stores of 16 bytes from the registers, 28.5 in runs, 26.4 in runs past the L2; from the registers past it 43).
    lds_barrier();
    const int R = v.R;
    char* const mine = lds + wave * 8192;
    const int r0 = band * PB_ROWS + 64 * wr;
#pragma unroll
    for (int j = 0; j < NTK; ++j) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = acc[i][j][4 * q + e];
                const int u = 8 * i + 2 * q + lh;
                *reinterpret_cast<floatx4*>(mine + ln * 256 + ((u ^ (ln & 15)) << 4)) = o;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const int tl = 4 * g + (lane >> 4), u = lane & 15;
            const floatx4 o = *reinterpret_cast<const floatx4*>(mine + tl * 256 + ((u ^ (tl & 15)) << 4));
            const int tt = t0 + wt + 32 * j + tl;
            if (tt < T && r0 + 4 * u < R) __builtin_nontemporal_store(o, reinterpret_cast<floatx4*>(C + (int64_t)tt * R + r0 + 4 * u));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

// `full` token tiles of 64 NTK tokens, the tokens behind them in tiles of 64 (TAIL)
template <bool BF, int NTK, int AHEAD, bool TAIL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_pairs(const char* __restrict__ A, const PairsView v, float* __restrict__ C, int T, int full) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int xcd = (int)(blockIdx.x & 7), at = (int)(blockIdx.x >> 3);
    const int nfull = full * v.bands, Q = (nfull + 7) >> 3;
    int mi, band;
    if (at < Q) {
        const int id = xcd * Q + at;
        if (id >= nfull) return;
        tile_coords(id, full, v.bands, mi, band);
        pairs_tile<BF, NTK, AHEAD>(A, v, C, T, mi * 64 * NTK, band, lds);
    } else if constexpr (TAIL) {
        const int t1 = full * 64 * NTK, rest = (T - t1 + 63) / 64, ntail = rest * v.bands, QT = (ntail + 7) >> 3;
        const int id = xcd * QT + at - Q;
        if (at - Q >= QT || id >= ntail) return;
        tile_coords(id, rest, v.bands, mi, band);
        pairs_tile<BF, 1, AHEAD>(A, v, C, T, t1 + mi * 64, band, lds);
    }
}

template <bool BF, int NTK, int AHEAD, bool TAIL>
static int launch_pairs(const void* A, const PairsView& v, float* C, int T, int full, hipStream_t s) {
    constexpr int STAGE = 64 * NTK * 64 * (BF ? 2 : 4) + PK_BLOCK;
    const unsigned bytes = 2 * STAGE + (unsigned)align_up(2 * (size_t)v.nk, 16);
    static uint64_t done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(&k_gemm_pairs<BF, NTK, AHEAD, TAIL>), 2 * STAGE + 4096, done);
    if (rc != MST_OK) return rc;
    const int64_t tail = full * 64 * NTK < T ? cdiv(T - full * 64 * NTK, 64) : 0;
    const int64_t per_xcd = cdiv((int64_t)full * v.bands, 8) + cdiv(tail * v.bands, 8);
    k_gemm_pairs<BF, NTK, AHEAD, TAIL><<<(unsigned)(8 * per_xcd), 512, bytes, s>>>(static_cast<const char*>(A), v, C, T, full);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

// What a step of the second kind takes against one of the first: nothing goes to LDS beside its products, and a wavefront without any
// waits for the others.
constexpr double SECOND_STEP_F32 = 1.4, SECOND_STEP_BF16 = 1.3;

// Microseconds of an fp32 product with `full` token tiles of 128, the rest in tiles of 64.  (Per step of 64 k: 1.41 with 128 tokens
// on every CU, 0.93 on a few, 0.81 and 0.70 with 64: the weights of a step cost the same for either.)
static double pairs_f32_us(int T, int R, int K, int full, double second) {
    const int64_t bands = cdiv(R, PB_ROWS), rest = std::max(0, T - 128 * full);
    const int64_t Q = cdiv(full * bands, 8), QT = cdiv(cdiv(rest, 64) * bands, 8);
    return (xcd_rounds(Q, 32, 8, 1.41, 0.93) + xcd_rounds(QT, 32, 8, 0.81, 0.70)) * (K / PK_STEP) * (1.0 + SECOND_STEP_F32 * second) +
           (double)cdiv(Q, 32) * 7.4 + (double)cdiv(QT, 32) * 4.6;
}

// Token tiles of 128 of an fp32 product.  A CU holds one workgroup, so 320 tiles are two rounds, the second one a quarter full:
// the tokens behind the last full round go in tiles of 64, twice as many CUs for them, where that is the shorter way (5120
// -> 1280, 8192 tokens: 212 -> 186 us; 3840 -> 1280: 161 -> 141; all of them where 128 would leave half of the CUs idle: 3072 -> 768,
// 2048 tokens: 57 -> 41).
static int pairs_full_tiles(int T, int R, int K) {
    const int all = (int)cdiv(T, 128);
    if (gemm_pairs_forced()) return T % 3 == 0 ? all : T % 3 == 1 ? 0 : all / 2;      // (pinned: every kind)
    const int bands = (int)cdiv(R, PB_ROWS), whole = (int)((int64_t)all * bands / 256 * 256 / bands);
    return pairs_f32_us(T, R, K, whole, 0.0) < pairs_f32_us(T, R, K, all, 0.0) ? whole : all;
}

// C [T x R] = A [T x K] S^T, S given by its packed pairs; tokens: of a workgroup's tile (fp32: pairs_full_tiles)
int gemm_pairs(const void* A, mst_dtype act, const PairsView& v, float* C, int T, int tokens, hipStream_t s) {
    if (v.R % 4 || v.K % PK_STEP) return MST_ERR_ARG;
    if (act == MST_F32) return launch_pairs<false, 2, 2, true>(A, v, C, T, pairs_full_tiles(T, v.R, v.K), s);
    const int full = (int)cdiv(T, tokens);
    return tokens == 128 ? launch_pairs<true, 2, 2, false>(A, v, C, T, full, s) : tokens == 192 ? launch_pairs<true, 3, 2, false>(A, v, C, T, full, s)
                                                                                : launch_pairs<true, 4, 1, false>(A, v, C, T, full, s);
}

// ------------------------------------------------------------------ choice
constexpr double PAIRS_LINE = 0.12;

// share of the steps of a uniformly random mask that need a second one
static double second_steps(double d) {
    if (d <= 0.08) return 0.0;
    if (d <= 0.10) return 5.0 * (d - 0.08);
    return std::min(1.0, 0.10 + 38.0 * (d - 0.10));
}

bool pairs_kept(const mst_layer* L) { return !L->pairs_missed && (L->pairs_recorded || L->pairs_unread < mst_layer::PAIRS_UNREAD); }

// How uneven the present mask is: the share of the steps of a band that go a second time, against that of a uniformly random mask.
// By the mask and not by the weights: those that an update has grown are zero until the next step.  Read back by the first
// product that reads the packed weights of a mask, which waits for it.
int measure_pairs(mst_layer* L, hipStream_t s) {
    uint32_t second[2] = {0, 0};
    MST_HIP(hipMemcpyAsync(second, L->pairs_y.count, 8, hipMemcpyDeviceToHost, s));
    MST_HIP(hipStreamSynchronize(s));
    const double uniform = second_steps((double)L->nnz / (double)L->N);
    for (int v = 0; v < 2; ++v) {
        const PairsView& view = v == 0 ? L->pairs_y : L->pairs_x;
        L->pairs_skew[v] = (float)((double)second[v] / ((double)view.bands * view.nk) - uniform);
    }
    L->pairs_measured = true;
    L->pairs_calls = 0;
    return MST_OK;
}

static double pairs_us(mst_dtype act, int T, int R, int K, int tokens, double second) {
    if (act == MST_F32) return pairs_f32_us(T, R, K, pairs_full_tiles(T, R, K), second);
    const int64_t Q = cdiv(cdiv(T, tokens) * cdiv(R, PB_ROWS), 8);
    double full, lone, ends;
    if (tokens == 256) full = 1.95, lone = 1.3, ends = 9.0;
    else if (tokens == 192) full = 1.5, lone = 0.95, ends = 7.0;
    else full = 1.2, lone = 0.8, ends = 5.0;
    return xcd_rounds(Q, 32, 8, full, lone) * (K / PK_STEP) * (1.0 + SECOND_STEP_BF16 * second) + (double)cdiv(Q, 32) * ends;
}

// Of the packing, with the choice of the pairs or without (measured 64 x 64 to 5120 x 5120, within 2 us).
double making_pairs_us(const mst_layer* L, bool match) { return 5.0 + 1.5e-6 * (double)L->N + (match ? 14.0 + 1.6e-6 * (double)L->N : 0.0); }

// Tokens of a tile, 0 where the dense kernels are ahead.  making_us: what this product spends on the packed weights before it reads them
// 3040 products on three cards (layers of 256 to 6000, 1024 to 16384 tokens, densities 0.03 to 0.12, a quarter with full rows): the modelled times
// are, of the measured ones, 0.93 to 1.02 by card in fp32 (sd 0.06, where few steps go a second time), of the dense kernels there 0.96 to
// 1.04 (0.10); in bfloat16 1.12 to 1.21, 1.05 to 1.13 and 1.13 to 1.21 (0.05) for 128, 192 and 256 tokens, dense 1.18 to 1.25 (0.07).  The choice
// loses 0.3 % against the best of all kernels, 21 % at the worst, and leaves 9 of 2062 fp32 and 2 of 978 bfloat16 products slower than the
// dense kernels by more than 3 % (12 % at the worst).  With second steps at 0.8 of a first one and first ones 7 % dearer in fp32: 94 and 33, 23 %.
int pairs_tokens(const mst_layer* L, bool y, mst_dtype act, int T, int64_t split_floats, double making_us) {
    const double d = (double)L->nnz / (double)L->N;
    if (!L->pairs_y.blocks) return 0;
    if (gemm_pairs_forced()) return act == MST_F32 ? 128 : 64 * (2 + T % 3);
    if (d > PAIRS_LINE) return 0;
    const int R = y ? L->O : L->I, K = y ? L->I : L->O;
    const double dense = gemm_two_parts_us(y ? GEMM_NT : GEMM_NN, act, T, R, K, std::max<int64_t>(1, split_floats / ((int64_t)T * R)));
    if (dense == 0.0) return 0;
    const double second = std::min(1.0, std::max(0.0, second_steps(d) + (double)L->pairs_skew[y ? 0 : 1]));
    double best = dense;
    int tokens = 0;
    for (int t : {128, 192, 256}) {
        if (act == MST_F32 && t != 128) break;
        const double us = pairs_us(act, T, R, K, t, second) + making_us;
        if (us < best) best = us, tokens = t;
    }
    return tokens;
}

// Would Y or dX (both of them) of a batch like the last one read them?
bool pairs_wanted(const mst_layer* L, bool both) {
    if (L->hint_T <= 0) return false;
    const mst_dtype act = (mst_dtype)L->hint_act;
    auto reads = [&](bool y) {
        const WalkJob job = y ? WALK_FWD : WALK_BWD_INPUT;
        return use_dense_path(L, job, act, L->hint_T) && !full_precision(L, job, act, L->hint_T) && pairs_tokens(L, y, act, L->hint_T, 0, 0.0) != 0;
    };
    return both ? reads(true) && reads(false) : reads(true) || reads(false);
}

}  // namespace mst
