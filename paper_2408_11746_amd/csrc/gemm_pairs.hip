// Y = X Wd^T and dX = dY Wd at densities of about a tenth and below on the sparse matrix instructions
// (v_smfmac_f32_32x32x32_bf16): of every four consecutive k a row of the weights holds two values and two 2-bit
// selectors, and the instruction covers 32 k in the 32 clocks in which the dense one covers 16.  Operands, parts and products are
// those of the dense kernels (two bfloat16 parts per fp32 operand: lo.hi, hi.lo, hi.hi; bfloat16 activations: lo, hi).
//
// A row with three entries among four k does not fit.  At density 0.1 that is one quad in 270, somewhere in 61 % of the tiles
// of 32 rows x 32 k, and a second pass over those would take back most of the gain.  So the quads are chosen:  the
// activations go to LDS by dwords (two k, as bfloat16) anyway, and for every band of 256 rows and step of 64 k the 32 dwords are
// paired up so that the fewest rows overflow (k_match_pairs: greedy, then exchanges between two quads).  Up to density 0.08 that
// leaves nothing, at 0.10 one step in ten with a few overflowing rows, at 0.12 five in six.  What is left, the third and fourth entries, is
// packed by itself ("second weights") and multiplied in the same step by the wavefronts that have any, over the activations that are in LDS
// anyway: every mask is exact.
//
// A tile: one band x 128 tokens (fp32; the tokens behind the last full round in tiles of 64) or 256, 192, 128 tokens (bfloat16), eight
// wavefronts of 64 rows x half the tokens.  A CU holds one workgroup, which forms tile after tile (numbers 32 apart on its XCD).
//   - The steps of a tile follow those of the one before: what is on its way belongs to the next tile already while the outputs
//     leave, so a tile has no start of its own (as workgroups of one tile each, loads, conversion and the place of the
//     next workgroup took 5 us of 29 at 768 -> 3072).
//   - The weights go straight to LDS, three stages of 32 KB: loaded while the step before the last one runs.  Through registers they
//     cost 34 of those and 250 clocks of a step; with two stages they had to arrive within a step.
//   - The activations are loaded two steps before their way to LDS, each piece right behind the store that freed its registers, converted
//     and stored between the products.  A slot of the table is what the address differs by, so an address costs one instruction.  Two
//     stages of 32 KB: with the weights' all of a CU's LDS; the selectors stay in registers, and the outputs leave through the stage of
//     weights that is free then, every wavefront's through the part of it that its own loads fill next.
//   - The operands of the last two blocks of products of a step are in registers when the wavefronts meet, so the reads for the next step
//     stand beside 12 products and the reads of a step are spread evenly over it.
//   - One barrier per step.  The loop has one way out: with a second one in the middle the compiler counted a step's loads
//     less in every wait, and the step took 4000 clocks.
// Measured (us; before = one workgroup per tile, weights through registers, second weights as steps of their own behind the others; 8192
// tokens, fp32, 0.10): Y of 1280 -> 5120 199 -> 172, dX of it 210 -> 197; Y of 768 -> 3072 78 -> 69, dX of it 80 -> 70.  16384 tokens,
// bfloat16, 0.05: Y of 1024 -> 4096 143 -> 138, dX 113.5 -> 113.
// What bounds it: Y of 1280 -> 5120 keeps the CUs busy for 75 million clocks (before 90), 54 % of them matrix instructions (45), dX for 78 (92),
// 52 % (44); the bfloat16 products for 62 (69) and 50 (52), 54 % (49) and 67 % (64), what is left mostly the 256 KB of outputs of a tile, all
// workgroups at once.  One product at a time runs at 1.8 to 2.0 GHz; one behind the other the same clocks take up to a quarter
// longer (176 to 217 us in one trace).  Workgroups that start at different times (up to 10 us apart) gained nothing
// in fp32 and 2 % in bfloat16, outputs past the L2 or through it are the same.
#include <cmath>
#include <type_traits>
#include <utility>

#include "common.h"
#include "active.h"
#include "split_bf16.h"

namespace mst {

typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef uint32_t pk_u32x4 __attribute__((ext_vector_type(4)));

constexpr int PB_ROWS = 256, PB_TILES = PB_ROWS / 32;          // rows of a band, MFMA tiles of them
constexpr int PK_STEP = 64, PK_PAIRS = PK_STEP / 2;            // k of a step
constexpr int PW_TILE = 2048, PW_SUB = PB_TILES * PW_TILE, PW_STEP = 2 * PW_SUB;   // packed bytes: [32 k][tile][hi 1 KB, lo 1 KB]
constexpr int PW_SEL = PB_TILES / 2 * 64 * 8;                   // selectors of a step: [two tiles][lane][tile], first 32 k in the low half

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
    v.slots = (uint16_t*)take((size_t)n * PK_PAIRS * 2);
    v.flags = (uint32_t*)take((size_t)n * 4);
    v.over = (uint8_t*)take((size_t)n);
    v.count = (uint32_t*)take(8);
    v.blocks = take((size_t)n * 2 * PW_STEP);
    v.sel = (uint32_t*)take((size_t)n * 2 * PW_SEL);
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
        for (int e = tid; e < 4 * missing; e += 256) {       // [first, second step][half of a lane's k][missing rows]
            const int row = PB_ROWS - missing + e % missing, ss = e / missing;
            uint32_t* const sel = v.sel + ((int64_t)band * 2 * v.nk + kb + (ss >> 1) * v.nk) * (PW_SEL / 4);
            sel[(row >> 6) * 128 + ((ss & 1) * 32 + (row & 31)) * 2 + (row >> 5 & 1)] = 0x44444444u;
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
        // (as the product's staging store wants it, see there)
        auto slot = [](int pl) { return (uint16_t)((pl & 15) << 2 | (pl >> 4) << 14); };
        v.slots[(int64_t)at * NP + first] = slot(place);
        v.slots[(int64_t)at * NP + second] = slot(place ^ 1);
    }
}

// ------------------------------------------------------------------ packing
// Block = 64 o x 64 i of the dense weights, read once for both views: two tiles of 32 rows of either, one step.  A wavefront
// packs a tile; lane = row and 16 k of every 32.  Bound by the 8.5 bytes per position that it reads and writes.
// first: the packing behind a choice of slots; block 0 counts the steps that go a second time (a launch of its own: four layers of a
// GPT-2-small block 19 us longer in the first pass on new masks).
// HANDED_OVER: the dense weights are out of date and are written as well, from the active values and the words that lead to them (a
// launch that writes them and this kernel behind it: 3072 x 768 at a density of 0.1 5.9 + 9.1 us, so 10.6; 1024 x 4096 at 0.05 6.3 + 11.1,
// so 12.4).
template <bool HANDED_OVER>
__global__ __launch_bounds__(256) void k_pack_pairs(float* __restrict__ W, int I, const PairsView y, const PairsView x, bool first,
                                                    float* __restrict__ vals, const ActiveRuns runs, int* __restrict__ dense_live) {
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
    float4 handed[4];
    if constexpr (HANDED_OVER) {
        const __amdgpu_buffer_rsrc_t from = active_buffer(vals, runs);
        const int c = 4 * (tid & 15);
        uint2 word[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) word[e] = runs.words[(int64_t)(o0 + 16 * e + (tid >> 4)) * runs.per_row + ((i0 + c) >> 5)];
        auto value = [&](int e, int q) __attribute__((always_inline)) {
            const uint32_t col = (uint32_t)(c & 31) + (uint32_t)q;
            return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(from, (int)active_offset(word[e], col, (1u << col) - 1u), 0, 0));
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) handed[e] = make_float4(value(e, 0), value(e, 1), value(e, 2), value(e, 3));
        if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *dense_live = 1;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int o = 16 * e + (tid >> 4), c = 4 * (tid & 15);
        float4* const at = reinterpret_cast<float4*>(W + (int64_t)(o0 + o) * I + i0 + c);
        float4 w;
        if constexpr (HANDED_OVER) *at = w = handed[e];
        else w = *at;
        float* p = tile + o * LD + c;
        p[0] = w.x; p[1] = w.y; p[2] = w.z; p[3] = w.w;
    }
    if ((wave & 1) == 0 && lane < PK_PAIRS) {
        const uint32_t f = v.slots[bk * PK_PAIRS + lane];
        pair_s[wave >> 1][(f >> 2 & 15) | (f >> 14) << 4] = (uint8_t)lane;
    }
    __syncthreads();
    const int row = 32 * (wave & 1) + (lane & 31), h = lane >> 5;
    // element (row, k) of this wavefront's view
    const float* const at = tile + (of_x ? row : row * LD);
    const int step = of_x ? LD : 1;
    const uint8_t* const ps = pair_s[wave >> 1];
    pk_u32x4 hi2[2], lo2[2];
    uint32_t ix1 = 0, ix2 = 0;                        // of both halves of the step
    bool over = false;
    const int64_t first_step = (int64_t)band * 2 * v.nk + kb;
    auto store = [&](int64_t at_step, int ss, pk_u32x4 hi, pk_u32x4 lo) {
        char* const b = v.blocks + at_step * PW_STEP + ss * PW_SUB + t * PW_TILE + lane * 16;
        *reinterpret_cast<pk_u32x4*>(b) = hi;
        *reinterpret_cast<pk_u32x4*>(b + 1024) = lo;
    };
    auto store_sel = [&](int64_t at_step, uint32_t ix) { v.sel[at_step * (PW_SEL / 4) + (t >> 1) * 128 + lane * 2 + (t & 1)] = ix; };
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
            ix1 |= two(m, a, b) << (4 * q + 16 * ss);
            split_pair(a, b, hh, ll);
            hi[q] = hh;
            lo[q] = ll;
            uint32_t m2 = m & (m - 1u);
            m2 &= m2 - 1u;
            over |= m2 != 0;
            ix2 |= two(m2, a, b) << (4 * q + 16 * ss);
            split_pair(a, b, hh, ll);
            hi2[ss][q] = hh;
            lo2[ss][q] = ll;
        }
        store(first_step, ss, hi, lo);
    }
    store_sel(first_step, ix1);
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
    for (int ss = 0; ss < 2; ++ss) store(first_step + v.nk, ss, hi2[ss], lo2[ss]);
    store_sel(first_step + v.nk, ix2);
}

// From the mask and the dense copy: the slots where the active set is a new one, and the blocks.  words: of the active set, where the
// dense copy has to take the values first
int make_pairs(mst_layer* L, hipStream_t s, const ActiveRuns* words) {
    const PairsView &y = L->pairs_y, &x = L->pairs_x;
    if (!L->pairs_matched) {
        k_match_pairs<<<(unsigned)(y.bands * y.nk + x.bands * x.nk), 256, 0, s>>>(L->mask, L->I, y, x);
        MST_LAUNCH_CHECK();
    }
    const auto pack = words ? k_pack_pairs<true> : k_pack_pairs<false>;
    pack<<<dim3((unsigned)(L->I / 64), (unsigned)(L->O / 64)), 256, 0, s>>>(L->Wd, L->I, y, x, !L->pairs_matched, L->vals, words ? *words : ActiveRuns{}, L->dense_live);
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

// LDS: two stages of the activations, three of the weights
constexpr int PX_STAGE = 32768, PX_SUB = 16384, PW_RING = 2 * PX_STAGE, PAIRS_LDS = PW_RING + 3 * PW_STEP;

// All of a workgroup's tiles of 64 NTK tokens x one band: numbers xcd Q + at, at = at0, at0 + 32, ...  The steps of one tile follow
// those of the one before without a break; between two of them the wavefronts store their outputs.
// NTK: tiles of 32 tokens of a wavefront
template <bool BF, int NTK>
__device__ __forceinline__ void pairs_tiles(const char* __restrict__ A, const PairsView& v, float* __restrict__ C, int T, int t_begin, int n_tok, int xcd, int Q, int at0,
                                            char* const lds) {
    constexpr int TOK = 64 * NTK, PLANE = TOK * 64;
    constexpr int LINES = BF ? 1 : 2, NX = NTK * LINES;           // 128-byte lines of a row in a step; 16-byte pieces of a thread
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = v.nk, ntiles = n_tok * v.bands;
    auto is_tile = [&](int at) { return at < Q && xcd * Q + at < ntiles; };
    if (!is_tile(at0)) return;
    const uint32_t pitch = (uint32_t)v.K * (BF ? 2u : 4u);

    // ---- where a step's operands are
    struct Source {
        int at, kb, t0, band;
        const char* w;                                // packed tiles of the step
        __amdgpu_buffer_rsrc_t rs;                    // the token tile's activations
    };
    auto tile_of = [&](int at, int& t0, int& band) {
        int mi;
        tile_coords(xcd * Q + at, n_tok, v.bands, mi, band);
        t0 = t_begin + mi * TOK;
    };
    auto aim = [&](Source& s, int at) {
        s.at = at;
        s.kb = 0;
        tile_of(at, s.t0, s.band);
        s.w = v.blocks + (int64_t)s.band * 2 * nk * PW_STEP;
        s.rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(A + (int64_t)s.t0 * pitch), 0, (int)((uint32_t)min(T - s.t0, TOK) * pitch), 0x00020000);
    };
    auto advance = [&](Source& s) {                   // (past the last step: that step again, into stages that nobody reads)
        if (s.kb + 1 < nk) { ++s.kb; s.w += PW_STEP; }
        else if (is_tile(s.at + 32)) aim(s, s.at + 32);
    };

    // ---- staging: chunk of 16 bytes of row row0 + 64 it
    // (32 lanes: four chunks of eight rows whose positions in LDS, two in 128 bytes times four swizzles, put any dword of a
    // 64-byte row in eight different banks)
    const int chunk = (lane & 3) | (lane >> 5) << 2;
    const int row0 = (lane >> 2 & 7) + 8 * wave;
    const uint32_t xoff = (uint32_t)row0 * pitch + 16u * chunk;
    // a slot is the dword's place in a row (64 bytes of 32 k) and, 16 KB on, which 32 k: it and the row's address have no bits in
    // common but those of the swizzle
    const uint32_t wbase = (uint32_t)pr_rho(row0) * 64u | (((uint32_t)pr_rho(row0) >> 2 ^ (uint32_t)pr_rho(row0) >> 4) & 3u) << 4;
    const uint32_t slot_off = BF ? 8u * chunk : 4u * chunk, sel_off = (uint32_t)(wave >> 1) * 512u + 8u * lane, w_off = 4096u * wave + 16u * lane;
    uint32_t no_lane;                                 // zero that the compiler takes for a lane's own (a scalar load would share the LDS reads' counter)
    asm("v_mov_b32 %0, 0" : "=v"(no_lane));
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    // What a thread carries of a step: NX pieces of 16 bytes of the activations with the slots of their dwords, its selectors and the flags of
    // the 64-row groups.  Operation n of a step: something goes to LDS, and what its registers held is loaded two steps on.
    struct Carried {
        pk_u32x4 x[NX];
        uint32_t slot[2], sel[2], flag;
    };
    auto load_x = [&](Carried& f, const Source& src, int n) __attribute__((always_inline)) {
        f.x[n] = __builtin_amdgcn_raw_buffer_load_b128(src.rs, (int)(xoff + (uint32_t)(64 * (n % NTK)) * pitch + 128u * (uint32_t)(src.kb * LINES + n / NTK)), 0, 0);
    };
    auto load_slot = [&](Carried& f, const Source& src, int line) __attribute__((always_inline)) {
        const char* p = reinterpret_cast<const char*>(v.slots) + ((int64_t)src.band * nk + src.kb) * (2 * PK_PAIRS) + 32 * line + slot_off;
        if constexpr (BF) {
            const uint2 u = *reinterpret_cast<const uint2*>(p);
            f.slot[0] = u.x;
            f.slot[1] = u.y;
        } else {
            f.slot[line] = *reinterpret_cast<const uint32_t*>(p);
        }
    };
    auto load_sel = [&](Carried& f, const Source& src) __attribute__((always_inline)) {
        const uint2 u = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(v.sel) + ((int64_t)src.band * 2 * nk + src.kb) * PW_SEL + sel_off);
        f.sel[0] = u.x;
        f.sel[1] = u.y;
        f.flag = v.flags[(int64_t)src.band * nk + src.kb + no_lane];
    };
    auto load_w = [&](const char* w, uint32_t ring, int n) __attribute__((always_inline)) { load_to_lds(w + 1024 * n, w_off, lds0 + PW_RING + ring + 4096u * wave + 1024u * n); };
    constexpr int NPUT = BF ? 4 * ((NTK + 1) / 2) : 4 * NTK;
    constexpr int LOADS = NX + LINES + 2, VM = LOADS + 4;         // of a step, and with the weights' four
    auto put = [&](Carried& f, uint32_t stage, const Source& next, auto nc) __attribute__((always_inline)) {
        constexpr int n = decltype(nc)::value;
        if constexpr (BF) {
            constexpr int e = n % 4, h = n / 4;               // dword e of pieces 2 h and 2 h + 1
            const uint32_t b = e & 1 ? f.slot[e >> 1] >> 16 : f.slot[e >> 1] & 0xFFFFu;
            char* const p = lds + ((wbase ^ b) + stage + 8192u * h);
            *reinterpret_cast<uint32_t*>(p) = f.x[2 * h][e];
            if (2 * h + 1 < NTK) *reinterpret_cast<uint32_t*>(p + 4096) = f.x[2 * h + 1 < NTK ? 2 * h + 1 : 0][e];
            if constexpr (e == 3) {
                load_x(f, next, 2 * h);
                if (2 * h + 1 < NTK) load_x(f, next, 2 * h + 1);
                if constexpr (h == (NTK + 1) / 2 - 1) load_slot(f, next, 0);
            }
        } else {
            constexpr int e = n % 2, it = n / 2 % NTK, line = n / (2 * NTK);
            const uint32_t b = e ? f.slot[line] >> 16 : f.slot[line] & 0xFFFFu;
            const pk_u32x4& x = f.x[line * NTK + it];
            uint32_t hi, lo;
            split_pair(__uint_as_float(x[2 * e]), __uint_as_float(x[2 * e + 1]), hi, lo);
            asm volatile("" : "+v"(hi), "+v"(lo));    // (in front of the load: one register for what is loaded and what was)
            char* const p = lds + ((wbase ^ b) + stage + 4096u * it);
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
        load_sel(f, src);
    };

    // ---- products: wavefront = 64 rows of the band x 32 NTK tokens.  A block: the NZ products of 32 k with one token tile, for two row
    // tiles.  The operands of block b + LEAD are read in front of block b, so the last LEAD blocks of a step stand behind the
    // barrier that its reads end at, beside the reads for the next one.
    const int wr = wave >> 1, wt = (wave & 1) * NTK;
    const int ln = lane & 31, lh = lane >> 5;
    constexpr int NZ = BF ? 2 : 3, NB = 2 * NTK, LEAD = NTK == 1 || NTK == 4 ? 1 : 2, S = LEAD == 1 ? 2 : NTK == 3 ? 3 : 4;
    uint32_t fx[2][2];                                // [unit 0 + lh, 2 + lh][parity of the tile]
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int par = 0; par < 2; ++par) fx[u][par] = pr_unit(32 * par + ln, 2 * u + lh) - 2048u * par + 2048u * wt;
    const bool odd_wt = NTK % 2 != 0 && (wt & 1) != 0;       // (NTK odd: the parity of the wavefront's first tile differs)
    const uint32_t wlane = PW_RING + 2u * wr * PW_TILE + 16u * lane;
    floatx16 acc[2][NTK];
    bf16x8 w[2][2][2];                                // [32 k][part][row tile]
    bf16x16 x[S][BF ? 1 : 2];
    uint32_t sel[2][2], flag[2];                      // [parity of the step][row tile]
    auto zero_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NTK; ++j)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
    };
    auto frag_x = [&](uint32_t at, int j) __attribute__((always_inline)) {
        const uint32_t a = ((j & 1) != 0) != odd_wt ? fx[0][1] : fx[0][0], b = ((j & 1) != 0) != odd_wt ? fx[1][1] : fx[1][0];
        const bf16x8 lo = *reinterpret_cast<const bf16x8*>(lds + (a + at + 2048u * j));
        const bf16x8 hi = *reinterpret_cast<const bf16x8*>(lds + (b + at + 2048u * j));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
    };
    auto fragments = [&](bf16x16 (&x)[BF ? 1 : 2], auto bc, uint32_t stage) __attribute__((always_inline)) {         // operands of block b
        constexpr int b = decltype(bc)::value;
        x[0] = frag_x(stage + PX_SUB * (b / NTK), b % NTK);
        if constexpr (!BF) x[1] = frag_x(stage + PX_SUB * (b / NTK) + PLANE, b % NTK);
    };
    auto read_x = [&](auto bc, uint32_t stage) __attribute__((always_inline)) { fragments(x[decltype(bc)::value % S], bc, stage); };
    auto read_w = [&](auto ssc, uint32_t ring) __attribute__((always_inline)) {
        constexpr int ss = decltype(ssc)::value;
        const char* const p = lds + (wlane + ring);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int z = 0; z < 2; ++z) w[ss][z][i] = *reinterpret_cast<const bf16x8*>(p + ss * PW_SUB + i * PW_TILE + 1024 * z);
    };
    // the products of block b; `between` them something else
    auto products = [&](auto bc, const bf16x8 (&w)[2][2][2], const bf16x16 (&x)[BF ? 1 : 2], const uint32_t (&ix)[2], auto between) __attribute__((always_inline)) {
        constexpr int b = decltype(bc)::value, j = b % NTK, W = b / NTK;
        static_for<2 * NZ>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value, z = m >> 1, i = m & 1;
            const int s = (int)(W ? ix[i] >> 16 : ix[i]);
            if constexpr (BF) acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(w[W][1 - z][i], x[0], acc[i][j], s, 0, 0);
            else acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(w[W][z == 0 ? 1 : 0][i], x[z == 1 ? 1 : 0], acc[i][j], s, 0, 0);
            between(mc);
            __builtin_amdgcn_sched_barrier(0x124);
        });
    };
    auto block = [&](auto bc, const uint32_t (&ix)[2], auto between) __attribute__((always_inline)) { products(bc, w, x[decltype(bc)::value % S], ix, between); };
    using zero = std::integral_constant<int, 0>;
    using one_ = std::integral_constant<int, 1>;

    // ---- the tile whose products are formed
    int c_at = at0, c_kb = 0, c_t0, c_band;
    tile_of(at0, c_t0, c_band);

    // D: lane l, register q -> row 8 (q / 4) + 4 (l / 32) + q % 4 of the band's tile, token l % 32.  The outputs leave through the
    // wavefront's own part of the weights' stage that is free, 16 tokens x 64 rows at a time, in runs of 256 bytes past the L2 (768 -> 768,
    // 8192 tokens: 30.2 us with stores of 16 bytes from the registers, 28.5 in runs, 26.4 in runs past the L2; from the registers past it 43).
    auto store_tile = [&](uint32_t ring) __attribute__((always_inline)) {
        const int R = v.R, r0 = c_band * PB_ROWS;
        uint32_t le = threadIdx.x & 63;               // (lane constants worked out again)
        asm volatile("" : "+v"(le));
        const uint32_t me = PW_RING + ring + 4096u * wave, tok = le & 15, half = le >> 5;
        const uint32_t row = 64u * wr + 4u * tok;     // of the band, as this lane stores it
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(C + (int64_t)c_t0 * R + r0, 0, (min(T - c_t0, TOK) * R - r0) * 4, 0x00020000);
        const uint32_t off = (int)row < R - r0 ? ((le >> 4) * (uint32_t)R + row) * 4u : 0x80000000u;       // (past the end: no access)
#pragma unroll
        for (int j = 0; j < NTK; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if ((le >> 4 & 1) == (uint32_t)h) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            floatx4 o;
#pragma unroll
                            for (int e = 0; e < 4; ++e) o[e] = acc[i][j][4 * q + e];
                            *reinterpret_cast<floatx4*>(lds + (me + tok * 256u + (((8u * i + 2u * q + half) ^ tok) << 4))) = o;
                        }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint32_t tl = 4u * g + (le >> 4);
                    const pk_u32x4 o = *reinterpret_cast<const pk_u32x4*>(lds + (me + tl * 256u + ((tok ^ tl) << 4)));
                    __builtin_amdgcn_raw_buffer_store_b128(o, out, (int)(off + (uint32_t)(32 * (wt + j) + 16 * h + 4 * g) * (uint32_t)R * 4u), 0, 2);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
    };

    // ---- step t on stage P = t % 2 and ring place t % 3.  In front of its barrier: its first NB - LEAD blocks, the second part of what brings
    // step t + 1 to LDS, the loads of step t + 2's weights.  Behind: its last blocks, the first reads of step t + 1 and
    // the first part of what brings step t + 2 to LDS.
    constexpr int PUT_BEHIND = NPUT * LEAD / NB, NFRONT = NPUT - PUT_BEHIND + 5;
    Carried carried[2];
    Source far, near;                                 // of the activations (two steps on) and the weights (one step on) of the step that goes to LDS
    uint32_t ring = 0;                                // place of step t
    auto next_place = [](uint32_t r) { return r == 2u * PW_STEP ? 0u : r + PW_STEP; };
    auto second_weights = [&](auto ssc, bf16x8 (&w)[2][2][2], uint32_t (&ix)[2]) __attribute__((always_inline)) {
        constexpr int ss = decltype(ssc)::value;
        uint32_t le = threadIdx.x & 63;
        asm volatile("" : "+v"(le));
        const int64_t at = (int64_t)c_band * 2 * nk + nk + c_kb;
        const char* const p = v.blocks + at * PW_STEP + 2 * wr * PW_TILE + 16 * le;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int z = 0; z < 2; ++z) w[ss][z][i] = *reinterpret_cast<const bf16x8*>(p + ss * PW_SUB + i * PW_TILE + 1024 * z);
        if constexpr (ss == 0) {
            const uint2 u = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(v.sel) + at * PW_SEL + 512 * wr + 8 * le);
            ix[0] = u.x;
            ix[1] = u.y;
        }
    };
    auto keep_sel = [&](Carried& f, int p) __attribute__((always_inline)) {
        asm volatile("v_mov_b32 %0, %3\n\tv_mov_b32 %1, %4\n\tv_readfirstlane_b32 %2, %5" : "=&v"(sel[p][0]), "=&v"(sel[p][1]), "=&s"(flag[p]) : "v"(f.sel[0]), "v"(f.sel[1]), "v"(f.flag));
    };
    auto step = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        constexpr uint32_t cur = P * PX_STAGE, nxt = PX_STAGE - cur;
        const uint32_t ring1 = next_place(ring), ring2 = next_place(ring1);
        constexpr int MF = (NB - LEAD) * 2 * NZ, MB = LEAD * 2 * NZ;
        Carried& f1 = carried[1 - P];
        Carried& f2 = carried[P];
        auto front = [&](auto nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value + PUT_BEHIND;
            if constexpr (n < NPUT) {
                put(f1, nxt, far, std::integral_constant<int, n>{});
            } else if constexpr (n < NPUT + 4) {
                load_w(near.w, ring2, n - NPUT);
            } else {
                keep_sel(f1, 1 - P);
                load_sel(f1, far);
            }
        };
        static_for<NB - LEAD>([&](auto bc) __attribute__((always_inline)) {
            constexpr int b = decltype(bc)::value;
            __builtin_amdgcn_sched_barrier(0);
            read_x(std::integral_constant<int, b + LEAD>{}, cur);
            if constexpr (b == NTK - LEAD) read_w(one_{}, ring);
            block(bc, sel[P], [&](auto mc) __attribute__((always_inline)) {
                constexpr int at = b * 2 * NZ + decltype(mc)::value;
                static_for<(at + 1) * NFRONT / MF - at * NFRONT / MF>([&](auto oc) __attribute__((always_inline)) {
                    front(std::integral_constant<int, at * NFRONT / MF + decltype(oc)::value>{});
                });
            });
        });
        near = far;
        advance(far);
        // rows with a third or fourth weight among four k: those weights over the same activations, by the wavefronts that have any
        if ((flag[P] >> (8 * wr) & 255u) != 0) {
            bf16x8 w2[2][2][2];
            uint32_t ix[2];
            __builtin_amdgcn_sched_barrier(0);
            second_weights(zero{}, w2, ix);
            if constexpr (NTK < 3) second_weights(one_{}, w2, ix);
            static_for<NB>([&](auto bc) __attribute__((always_inline)) {
                constexpr int b = decltype(bc)::value;
                if constexpr (NTK >= 3 && b == NTK) {         // (no room for both)
                    __builtin_amdgcn_sched_barrier(0);
                    second_weights(one_{}, w2, ix);
                }
                bf16x16 x2[BF ? 1 : 2];
                fragments(x2, bc, cur);
                products(bc, w2, x2, ix, [](auto) {});
            });
        }
        __builtin_amdgcn_sched_barrier(0);
        wait_loads<VM>();                             // the weights of step t + 1 (loaded in step t - 1) are in LDS
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
        auto behind = [&](auto nc) __attribute__((always_inline)) { put(f2, cur, far, nc); };
        auto reads = [&](auto dc) __attribute__((always_inline)) {
            constexpr int d = decltype(dc)::value;
            if constexpr (d == 0) read_w(zero{}, ring1);
            read_x(dc, nxt);
        };
        static_for<LEAD>([&](auto dc) __attribute__((always_inline)) {
            constexpr int d = decltype(dc)::value;
            __builtin_amdgcn_sched_barrier(0);
            reads(dc);
            block(std::integral_constant<int, NB - LEAD + d>{}, sel[P], [&](auto mc) __attribute__((always_inline)) {
                constexpr int at = d * 2 * NZ + decltype(mc)::value;
                static_for<(at + 1) * PUT_BEHIND / MB - at * PUT_BEHIND / MB>([&](auto oc) __attribute__((always_inline)) {
                    behind(std::integral_constant<int, at * PUT_BEHIND / MB + decltype(oc)::value>{});
                });
            });
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    // behind the last step of a tile: its outputs
    bool live = true;
    auto finish = [&]() __attribute__((always_inline)) {
        const uint32_t place = ring;
        ring = next_place(ring);
        if (++c_kb < nk) return;
        if (live) store_tile(place);
        live = live && is_tile(c_at + 32);
        c_kb = 0;
        if (live) {
            c_at += 32;
            tile_of(c_at, c_t0, c_band);
        }
        zero_sums();
    };

    aim(far, at0);
    load_all(carried[0], far);
#pragma unroll
    for (int n = 0; n < 4; ++n) load_w(far.w, 0, n);
    advance(far);
    load_all(carried[1], far);
#pragma unroll
    for (int n = 0; n < 4; ++n) load_w(far.w, PW_STEP, n);
    advance(far);
    zero_sums();
    static_for<NPUT>([&](auto nc) __attribute__((always_inline)) { put(carried[0], 0, far, nc); __builtin_amdgcn_sched_barrier(0); });
    keep_sel(carried[0], 0);
    load_sel(carried[0], far);
    near = far;                                       // (the weights of step 2)
    advance(far);
    static_for<PUT_BEHIND>([&](auto nc) __attribute__((always_inline)) { put(carried[1], PX_STAGE, far, nc); __builtin_amdgcn_sched_barrier(0); });
    wait_loads<LOADS>();                              // (what came behind the weights of step 1)
    lds_barrier();
    read_w(zero{}, 0);
    static_for<LEAD>([&](auto dc) __attribute__((always_inline)) { read_x(dc, 0); });
    // (one way out of the loop, so that the waits for what is carried round it count all of the loads between: an odd number of steps is
    // followed by one for nobody)
#pragma unroll 1
    do {
        step(zero{});
        finish();
        step(one_{});
        finish();
    } while (live);
    // nothing may arrive in LDS that is not ours any more
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
}

// `full` token tiles of 64 NTK tokens, the tokens behind them in tiles of 64 (TAIL).  Workgroup = (XCD, one of its 32 CUs).
template <bool BF, int NTK, bool TAIL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_pairs(const char* __restrict__ A, const PairsView v, float* __restrict__ C, int T, int full) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int xcd = (int)(blockIdx.x & 7), first = (int)(blockIdx.x >> 3);
    const int Q = (full * v.bands + 7) >> 3;
    pairs_tiles<BF, NTK>(A, v, C, T, 0, full, xcd, Q, first, lds);
    if constexpr (TAIL) {
        const int t1 = full * 64 * NTK, rest = (T - t1 + 63) / 64, QT = (rest * v.bands + 7) >> 3;
        // (the CUs that have a tile less begin)
        pairs_tiles<BF, 1>(A, v, C, T, t1, rest, xcd, QT, first >= Q % 32 ? first - Q % 32 : first - Q % 32 + 32, lds);
    }
}

template <bool BF, int NTK, bool TAIL>
static int launch_pairs(const void* A, const PairsView& v, float* C, int T, int full, hipStream_t s) {
    static uint64_t done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(&k_gemm_pairs<BF, NTK, TAIL>), PAIRS_LDS, done);
    if (rc != MST_OK) return rc;
    const int64_t tail = full * 64 * NTK < T ? cdiv(T - full * 64 * NTK, 64) : 0;
    const int64_t per_xcd = cdiv((int64_t)full * v.bands, 8) + cdiv(tail * v.bands, 8);
    k_gemm_pairs<BF, NTK, TAIL><<<(unsigned)(8 * std::min<int64_t>(32, per_xcd)), 512, PAIRS_LDS, s>>>(static_cast<const char*>(A), v, C, T, full);
    MST_LAUNCH_CHECK();
    return MST_OK;
}

// What the second weights add to the steps' time where a share `second` of them has any.  The groups of 64 rows are taken to be alike; the
// wavefronts of those without wait for the others, so a step with one such group is long by a third.  (Uniform masks, Y of 768 -> 3072, 8190
// tokens, fp32, densities 0.07, 0.10, 0.11, 0.12, 0.25: 71, 73, 81, 100, 133 us; bfloat16, 256 tokens: 55, 57, 64, 75, 89.)
// Every step with some is modelled as 2.5 steps, and more than it takes: with a full row in every 64 Y of 1280 -> 5120 takes 285 us (without
// 167), of 768 -> 3072 108 (75), of 1280 -> 1280 106 (62); the dense kernels 256, 96 and 69, which are right there.  With one in every 256 it
// takes 213, 82 and 84, and the first two of these stay on the dense kernels all the same.
static double second_part(double second, bool bf16) {
    const double group = 1.0 - std::sqrt(std::sqrt(1.0 - second));        // share of the steps in which a group has some
    return (bf16 ? 0.40 : 0.35) * second + 1.15 * group * group;
}

// Microseconds of an fp32 product with `full` token tiles of 128, the rest in tiles of 64.  (Per step of 64 k: 1.36 with 128 tokens
// on every CU, 0.92 on a few, 0.89 and 0.68 with 64: the weights of a step cost the same for either.  222 products of whole tiles, sd 5 %.)
static double pairs_f32_us(int T, int R, int K, int full, double second) {
    const int64_t bands = cdiv(R, PB_ROWS), rest = std::max(0, T - 128 * full), steps = K / PK_STEP;
    const int64_t Q = cdiv(full * bands, 8), QT = cdiv(cdiv(rest, 64) * bands, 8);
    return xcd_rounds(Q, 32, 8, 1.36, 0.92) * steps * (1.0 + second_part(second, false)) + xcd_rounds(QT, 32, 8, 0.89, 0.68) * steps * (1.0 + 2.0 * second_part(second, false)) +
           (Q > 0 ? 2.6 + cdiv(Q, 32) * 4.7 : 0.0) + (QT > 0 ? 3.4 + cdiv(QT, 32) * 1.5 : 0.0);
}

// Token tiles of 128 of an fp32 product.  320 tiles are two rounds of the CUs, the second one a quarter full:
// the tokens behind the last full round go in tiles of 64, twice as many CUs for them, where that is the shorter way (5120
// -> 1280, 8192 tokens: 212 -> 186 us; 3840 -> 1280: 161 -> 141; all of them where 128 would leave half of the CUs idle: 3072 -> 768,
// 2048 tokens: 57 -> 41, before a workgroup's tiles followed each other without a break).
static int pairs_full_tiles(int T, int R, int K) {
    const int all = (int)cdiv(T, 128);
    if (gemm_pairs_forced()) return T % 3 == 0 ? all : T % 3 == 1 ? 0 : all / 2;      // (pinned: every kind)
    const int bands = (int)cdiv(R, PB_ROWS), whole = (int)((int64_t)all * bands / 256 * 256 / bands);
    return pairs_f32_us(T, R, K, whole, 0.0) < pairs_f32_us(T, R, K, all, 0.0) ? whole : all;
}

// C [T x R] = A [T x K] S^T, S given by its packed pairs; tokens: of a workgroup's tile (fp32: pairs_full_tiles)
int gemm_pairs(const void* A, mst_dtype act, const PairsView& v, float* C, int T, int tokens, hipStream_t s) {
    if (v.R % 4 || v.K % PK_STEP) return MST_ERR_ARG;
    if (act == MST_F32) return launch_pairs<false, 2, true>(A, v, C, T, pairs_full_tiles(T, v.R, v.K), s);
    const int full = (int)cdiv(T, tokens);
    return tokens == 128 ? launch_pairs<true, 2, false>(A, v, C, T, full, s) : tokens == 192 ? launch_pairs<true, 3, false>(A, v, C, T, full, s)
                                                                                : launch_pairs<true, 4, false>(A, v, C, T, full, s);
}

// ------------------------------------------------------------------ choice
// Above, four steps in five have second weights and the products are within 10 % of the dense kernels on either side (Y of 1024 -> 4096, 16384
// tokens, fp32: 268 of 313 us at 0.11, 306 of 307 at 0.119).
constexpr double PAIRS_LINE = 0.118;

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
    if (tokens == 256) full = 1.78, lone = 1.25, ends = 11.5;
    else if (tokens == 192) full = 1.40, lone = 1.08, ends = 8.0;
    else full = 1.13, lone = 0.90, ends = 4.7;
    return 3.0 + xcd_rounds(Q, 32, 8, full, lone) * (K / PK_STEP) * (1.0 + second_part(second, true)) + (double)cdiv(Q, 32) * ends;
}

// Of the packing, with the choice of the pairs or without (measured 64 x 64 to 5120 x 5120, within 2 us).
double making_pairs_us(const mst_layer* L, bool match) { return 5.0 + 1.5e-6 * (double)L->N + (match ? 14.0 + 1.6e-6 * (double)L->N : 0.0); }

// Tokens of a tile, 0 where the dense kernels are ahead.  making_us: what this product spends on the packed weights before it reads them
// 468 products of whole tiles (layers of 256 to 5120, 2048 to 16384 tokens, densities 0.03 to 0.11): the modelled times are the measured ones
// in fp32 (sd 0.05) and 1.2 of them in bfloat16 (sd 0.03 to 0.04), as those of the dense kernels are there (0.96 to 1.04 and 1.18 to 1.25).
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
