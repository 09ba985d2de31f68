// The walk of an index view, the one kernel body behind the three products of the sparse path:
//
//   OUT        out[t, r] = sum_k A[t, k] S[r, k]          an SpMM: Y over the row view (S = W, A = X;
//                                                         App. "FLOP Calculation" Eq. (1)), dX over the
//                                                         col view (S = W^T, A = dY)
//   DW         p[e] = sum_t A[t, k_e] B[t, r_e]           an SDDMM: the weight gradient at the active
//                                                         positions, over either view (the product is
//                                                         symmetric in its dense operands)
//   OUT and DW both gradients of a layer from one walk of the col view (backward = 2 x forward)
//
// A workgroup of 16 wavefronts takes the whole LDS of a CU: a tile of 64 tokens x a chunk of up to 640
// contraction indices of A, transposed.  It owns Q row blocks of 128 rows; a wavefront walks one octet
// of eight rows of each of them.  A wavefront is eight lane groups of eight lanes; in one step each
// lane group multiplies ONE entry of its own row with the 64 tokens, eight per lane, read from LDS as
// two 16-byte halves.  Entries {offset, weight} come from global memory: a lane loads 16 bytes (one
// pair of its lane group) of a batch of four pairs, the next batch is in flight meanwhile, and the
// four lanes of an aligned group of four hand their pairs round through DPP operands.  Accumulators
// (OUT) and the second dense operand (DW) stay in registers for the whole contraction.
//
// What bounds it, and why this shape.  Every multiply-add needs its own operand from LDS and its own
// VALU lane: per step and wavefront 8 v_fmac (16 with DW), 3 for addresses and the weight, 2.5 for the
// sums over eight lanes; the walk itself runs at 90 % of the VALU issue rate (counters at 3072 x 768,
// density 0.10, 8192 tokens).  The whole kernel takes 89 % of the issue slots at density 0.10, 83 % at 0.05 and 73 % at 0.02
// (Y of 1280 -> 5120): the first stage, the barriers and the output, which nothing else of the CU covers, weigh more the
// shorter the walk.  The rest is what the format and the phases add, so:
//   - chunks of 640 instead of 128 indices: an ELL slice pads to the longest of its rows per chunk, and
//     25.6 instead of 2.6 entries a row and chunk at density 0.02 waste 0.25-0.30 instead of 0.44 of
//     the steps, and there are five times fewer barriers, over slabs of up to 768 rows;
//   - rows that are long in the same chunks share an octet (k_block_rank): 0.15 of the steps wasted with two
//     chunks, 0.24 with five, 0.27 with eight (8192 tokens, density 0.02: Y of 1280 -> 5120 100.5 -> 95, of 5120 -> 1280
//     88 -> 86, both gradients of the two 188 -> 184 and 204 -> 193);
//   - eight tokens a lane: the address, weight and row-sum instructions are shared by eight tokens;
//   - odd lane groups read the upper token half of a row first, even ones the lower: with the swizzle
//     of lds_off the reads are then free of bank conflicts (1.5 M conflict cycles instead of 26 M in
//     the case above, 150 -> 135 us);
//   - the weight goes through one v_mov_b32_dpp: a plain v_fmac_f32 issues in 3.4 clocks, one with a
//     DPP operand in 5.2;
//   - the wavefronts' octets are dealt in a snake over the blocks of the slab (octet w, then 15 - w), so that the longest
//     octets of blocks whose rows are ranked by length meet in no wavefront.  In blocks whose rows are halved by the lengths in parts of
//     the chunks no octet is the longest: 15 - w is of the other half in the first and the third split and of the same in the others;
//   - a wavefront's priority falls with the octets it has left.  With equal ones the oldest wavefront of a SIMD unit is
//     served first: of a chunk's 7 us at 1280 -> 5120, density 0.02, the last wavefront walked 2.6 us longer than the mean
//     one, alone on its unit and waiting for its own reads, with the priorities 0.9 us.  Y there 118 -> 113, at density 0.05
//     183 -> 172, dX 168 -> 158.  Where an octet is twice as long (both gradients) the last two octets count in halves:
//     199 -> 190 and 374 -> 361 (in whole octets 192 and 363);
// Measured (us; before = 128-token tiles over 128-index chunks, 8192 tokens, density 0.02):
//   Y of 1280 -> 5120: 168 -> 118;  dX of it: 210 -> 104;  both gradients of it: 300 -> 190.
#pragma once
#include <type_traits>
#include <utility>

#include "common.h"

namespace mst {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;     // the tile starts at LDS address 0 (allow_lds refuses a kernel with static LDS)
typedef __attribute__((address_space(4))) const int const_int;        // read through the scalar cache

constexpr int WALK_NW = OPB;                 // wavefronts per workgroup: one octet of a block each
constexpr int WALK_NT = WALK_NW * 64;
constexpr int STAGE_BYTES = WT * RB * 4;     // one row block's [64 tokens x 128 rows] on its way in or out

// One view with its operands
struct WalkSide {
    const void* A;               // staged in LDS [T x K]
    const void* B;               // kept in registers [T x R] (DW)
    const int* ptr;
    const uint4* ent;
    const int* rowmap;
    const int *perm, *rowpos;    // read for outputs that come out as NaN (OUT)
    int K, KC, R, NBpad, nchunk, nslab;
};
struct WalkArgs {
    float* out;                  // [T x R], or [splits][T x R] partial outputs (OUT)
    float* partial;              // [token tile][slots] (DW)
    int64_t slots_stride;
    int T, ntile;
    int chunks_per_split;        // blockIdx.y takes a range of chunks
};

// Which view drives the weight gradient: each one's cost as counted when it was built (the host never
// reads it back) times the time of a unit of it at this batch size and launch shape.
struct WalkDrive {
    const unsigned long long* cost;    // [2]: row view, col view
    float row_unit, col_unit;
};
__device__ inline bool drive_by_col(const WalkDrive& d) {
    typedef const __attribute__((address_space(4))) unsigned long long const_u64;
    const const_u64* c = (const const_u64*)d.cost;
    return (float)c[1] * d.col_unit < (float)c[0] * d.row_unit;
}

// one translation unit per activation type (walk_f32.hip, walk_bf16.hip); q = row blocks per workgroup
int walk_out_f32(int q, const WalkSide& sd, const WalkArgs& wa, hipStream_t s);                       // q = 1 .. 6
int walk_out_bf16(int q, const WalkSide& sd, const WalkArgs& wa, hipStream_t s);
int walk_both_f32(int q, const WalkSide& sd, const WalkArgs& wa, int nsplit, hipStream_t s);          // q = 1 .. 4
int walk_both_bf16(int q, const WalkSide& sd, const WalkArgs& wa, int nsplit, hipStream_t s);
int walk_dw_f32(int q, const WalkSide& row, const WalkSide& col, const WalkArgs& wa, const WalkDrive& drive, hipStream_t s);   // q = 1 .. 6
int walk_dw_bf16(int q, const WalkSide& row, const WalkSide& col, const WalkArgs& wa, const WalkDrive& drive, hipStream_t s);

// raw buffer of `bytes` bytes from p, rounded up to a dword: reads past the end give zeros (per dword)
// without an access
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)((bytes + 3) & ~3u), 0x00020000);
}
// Four consecutive elements as fp32, zeros from `end` (bytes) on if the first is there.  The hardware wants
// dword-aligned addresses: where rows of bfloat16 have an odd length (`even` false), every other row starts in
// the middle of a dword and is shifted into place, and the last dword may hold one element past the end.
// (Element by element such a layer's products took two to four times as long.)
template <typename TIn>
__device__ inline float4 buffer_quad(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off, uint32_t end, bool even);
template <>
__device__ inline float4 buffer_quad<float>(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off, uint32_t, bool) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)byte_off, 0, 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
template <>
__device__ inline float4 buffer_quad<uint16_t>(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off, uint32_t end, bool even) {
    u32x2 u;
    if (even) {
        u = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)byte_off, 0, 0);
    } else {
        const uint32_t sh = (byte_off & 2u) << 3;
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(byte_off & ~3u), 0, 0);
        const uint32_t e = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(byte_off & ~3u) + 8, 0, 0);
        u.x = byte_off < end ? __builtin_amdgcn_alignbit(w.y, w.x, sh) : 0u;
        u.y = __builtin_amdgcn_alignbit(e, w.y, sh);
    }
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                       __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u));
}

// a lane's 16 bytes of the batch of four pairs that starts at pair p (p the same in all lanes)
__device__ inline uint4 load_batch(const uint4* __restrict__ ent, int p, uint32_t lane_byte) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(buffer_of(ent + (int64_t)p * OCT, 4 * OCT * 16), (int)lane_byte, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// value of v in lane JJ of this lane's aligned group of four lanes
template <int JJ>
__device__ inline uint32_t quad_bcast(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, JJ * 0x55, 0xf, 0xf, true);
}

// Eight FMAs whose common factor W comes from lane JJ of the group of four lanes.  The leading s_nop
// covers the two wait states a DPP read needs after a VALU write of its source, whatever was
// scheduled in front of the block.
#define MST_FMA8_BC(JJ, ACC, W, X, Y)                                                                          \
    do {                                                                                                       \
        float wb_;                                                                                             \
        asm("s_nop 1\n\t"                                                                                      \
            "v_mov_b32_dpp %8, %9 quad_perm:[" #JJ "," #JJ "," #JJ "," #JJ "] row_mask:0xf bank_mask:0xf\n\t"   \
            "v_fmac_f32 %0, %8, %10\n\tv_fmac_f32 %1, %8, %11\n\tv_fmac_f32 %2, %8, %12\n\tv_fmac_f32 %3, %8, %13\n\t" \
            "v_fmac_f32 %4, %8, %14\n\tv_fmac_f32 %5, %8, %15\n\tv_fmac_f32 %6, %8, %16\n\tv_fmac_f32 %7, %8, %17"     \
            : "+v"(ACC[0]), "+v"(ACC[1]), "+v"(ACC[2]), "+v"(ACC[3]), "+v"(ACC[4]), "+v"(ACC[5]), "+v"(ACC[6]),    \
              "+v"(ACC[7]), "=&v"(wb_)                                                                         \
            : "v"(W), "v"(X.x), "v"(X.y), "v"(X.z), "v"(X.w), "v"(Y.x), "v"(Y.y), "v"(Y.z), "v"(Y.w));           \
    } while (0)

// Sums of a and b over each group of eight lanes with four adds: a's ends up in lanes 0..3 of the group,
// b's in lanes 4..7 (the first add of each writes its half of the group only).
__device__ inline float sum8_pair(float a, float b) {
    float r;
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
        : "=&v"(r) : "v"(a), "v"(b));
    return r;
}

template <typename TIn>
__device__ inline float element(const TIn* p);
template <>
__device__ inline float element<float>(const float* p) { return *p; }
template <>
__device__ inline float element<uint16_t>(const uint16_t* p) { return __uint_as_float((uint32_t)*p << 16); }

// The arguments of k_walk, read again where they are needed: what a rare branch after the walk uses would
// otherwise sit in scalar registers throughout it (1 % of the time of a step).
struct WalkParams {
    WalkSide sd;
    WalkArgs wa;
};
__device__ __forceinline__ const WalkParams& walk_params() {
    auto* p = (__attribute__((address_space(4))) const WalkParams*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const WalkParams*)p;
}

// out[t, row] over this workgroup's chunks from the row's own entries, in the order of the walk.  A padding entry
// has weight 0 and multiplies the first index of the chunk, so an infinity (or NaN) there makes NaN of every row with
// padding; an output that is NaN is formed again, up to the first term that makes it NaN by itself.  No other
// output pays more than a compare.
template <typename TIn>
__device__ __forceinline__ float own_entries_sum(int t, int row) {
    const WalkParams& wp = walk_params();
    const WalkSide& sd = wp.sd;
    const TIn* const a = static_cast<const TIn*>(sd.A) + (int64_t)t * sd.K;
    const int c0 = (int)blockIdx.y * wp.wa.chunks_per_split, c1 = min(sd.nchunk, c0 + wp.wa.chunks_per_split);
    const int rp = sd.rowpos[row], slot = rp & ~SPREAD_FLAG;
    const bool spread = (rp & SPREAD_FLAG) != 0;
    const uint2* __restrict__ ent = reinterpret_cast<const uint2*>(sd.ent);
    float one = 0.f, two = 0.f, four = 0.f, sum = 0.f;       // a spread row: its eight lane groups' sums, added pairwise
#pragma unroll 1
    for (int g = spread ? 0 : slot % OCT, last = spread ? OCT - 1 : g; g <= last; ++g) {
        sum = 0.f;
#pragma unroll 1
        for (int c = c0; c < c1 && sum == sum; ++c) {
            const int* pp = sd.ptr + ((int64_t)c * sd.NBpad + row / RB) * OPB + slot / OCT;
            const int steps = 2 * (pp[1] - pp[0]);
#pragma unroll 1
            for (int j = 0; j < steps && sum == sum; ++j) {
                const int64_t e = (((int64_t)pp[0] + (j >> 1)) * OCT + g) * 2 + (j & 1);
                if (sd.perm[e] >= 0) sum = fmaf(__uint_as_float(ent[e].y), element<TIn>(a + c * sd.KC + (ent[e].x >> 8)), sum);
            }
        }
        if (!spread) break;
        if ((g & 1) == 0) { one = sum; continue; }
        sum = one + sum;
        if ((g & 2) == 0) { two = sum; continue; }
        sum = two + sum;
        if ((g & 4) == 0) { four = sum; continue; }
        sum = four + sum;
    }
    return sum;
}

// octet of block q of the slab that wavefront `wave` walks (see the head of this file)
__device__ inline int octet_of(int wave, int q) { return (((q & 1) ? OPB - 1 - wave : wave) + 4 * (q >> 1)) & (OPB - 1); }

// token (inside the tile) of a lane's e-th value, e = 0..7; s = lane & 7, g = lane group
__device__ inline int lane_token(int s, int g, int e) { return 32 * ((e >> 2) ^ (g & 1)) + 4 * s + (e & 3); }

// byte of (token tl, row rl of the block) in the staging area of one block: token tl owns 512 bytes, the
// 16-byte unit j of rows 4j .. 4j+3 sits at unit j ^ ((tl >> 2) & 15)
__device__ inline uint32_t stage_unit(int tl, int j) { return (uint32_t)(tl * (RB * 4) + ((j ^ ((tl >> 2) & 15)) << 4)); }
__device__ inline uint32_t stage_byte(int tl, int rl) { return stage_unit(tl, rl >> 2) | (uint32_t)((rl & 3) << 2); }

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl(std::make_integer_sequence<int, N>{}, f); }

// row blocks of B that pass through LDS between two barriers of the prologue
constexpr int walk_areas(int q) { return q <= 5 ? q : 3; }

// lds: at least max(KC * 256, 2 * STAGE_BYTES) bytes, with DW max(KC * 256, walk_areas(Q) * STAGE_BYTES)
template <typename TIn, int Q, bool OUT, bool DW>
__device__ __forceinline__ void walk_body(const WalkSide& sd, const WalkArgs& wa, char* lds) {
    constexpr int NI = (KCMAX / 4 + 63) / 64;        // items of 4 tokens x 4 indices a thread stages per chunk
    // of them fetched before the barrier that ends the previous chunk's walk, while slower wavefronts
    // still walk (as many as the registers beside accumulators and register operand hold)
    constexpr int NPRE = DW && OUT ? (Q >= 4 ? 1 : 2) : Q >= 6 ? 1 : 2;
    // XCD x takes a contiguous share of the (tile, slab) pairs: the slabs of a token tile read the same
    // activations, and a share is never off by more than one workgroup however few tiles there are
    const int total = wa.ntile * sd.nslab, per = (total + 7) >> 3;
    const int id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || id >= total) return;
    const int tile_id = id / sd.nslab, slab = id - tile_id * sd.nslab;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = tile_id * WT;
    const int g = lane >> 3, s = lane & 7;
    const int b0 = slab * Q;
    const int T = wa.T, K = sd.K, KC = sd.KC, R = sd.R;
    const uint32_t lbase = ((uint32_t)s << 4) | ((uint32_t)(g & 1) << 7);
    const uint32_t ebyte = (uint32_t)((lane & 3) * OCT + g) * 16u;      // this lane's 16 bytes of a batch
    const uint32_t pbyte = (uint32_t)(g * 2 + (s >> 2)) * 4u;           // slot of this lane's sum inside a pair's sixteen
    float* const pt = DW ? wa.partial + (int64_t)tile_id * wa.slots_stride : nullptr;
    const TIn* __restrict__ A = static_cast<const TIn*>(sd.A);
    const int c_begin = (int)blockIdx.y * wa.chunks_per_split, c_end = min(sd.nchunk, c_begin + wa.chunks_per_split);
    const int nkq = KC >> 2;
    const uint32_t rows = (uint32_t)min(T - t0, WT);                    // token rows of the tile inside the batch

    // ---- the chunk's tile, two steps: global -> registers, registers -> LDS (transposed).  Item: 4 tokens
    // (quad tq) x 4 indices (quad kq).  The four lanes of a quad take consecutive kq (64 bytes of a row), the
    // four quads of a 16-lane group the four 64-byte quarters of an LDS row.  (Lane offsets are worked out
    // again every time instead of being kept in registers across the walk.)
    float4 st[NI][4];
    auto item_of = [&](int& tq, int& kq0) __attribute__((always_inline)) {
        int ln = (int)threadIdx.x & 63;
        asm volatile("" : "+v"(ln));
        tq = (wave & 3) + 4 * ((ln >> 2) & 3);
        kq0 = (wave >> 2) * 16 + ((ln & 3) | ((ln >> 4) << 2));
    };
    auto fetch = [&](int c, auto lo, auto hi) __attribute__((always_inline)) {
        int tq, kq0;
        item_of(tq, kq0);
        const uint32_t ld = (uint32_t)K * (uint32_t)sizeof(TIn);
        const uint32_t end = rows * ld - (uint32_t)(c * KC) * (uint32_t)sizeof(TIn);
        const __amdgpu_buffer_rsrc_t rs = buffer_of(A + (int64_t)t0 * K + c * KC, end);
        const uint32_t o0 = (uint32_t)(4 * tq) * ld + (uint32_t)(4 * kq0) * (uint32_t)sizeof(TIn);
#pragma unroll
        for (int i = lo; i < hi; ++i) {
            // (items past the chunk: an offset past the end, zeros without an access)
            const uint32_t oi = kq0 + 64 * i < nkq ? o0 + (uint32_t)(256 * i) * (uint32_t)sizeof(TIn) : 0xC0000000u;
#pragma unroll
            for (int r = 0; r < 4; ++r) st[i][r] = buffer_quad<TIn>(rs, oi + (uint32_t)r * ld, end, (K & 1) == 0);
        }
    };
    auto put = [&](auto lo, auto hi) __attribute__((always_inline)) {
        int tq, kq0;
        item_of(tq, kq0);
#pragma unroll
        for (int i = lo; i < hi; ++i) {
            const int kq = kq0 + 64 * i;
            if (kq < nkq) {
                char* p = lds + (((uint32_t)kq << 10) | (uint32_t)((tq ^ (kq & 3)) << 4));
                *reinterpret_cast<float4*>(p) = make_float4(st[i][0].x, st[i][1].x, st[i][2].x, st[i][3].x);
                *reinterpret_cast<float4*>(p + 256) = make_float4(st[i][0].y, st[i][1].y, st[i][2].y, st[i][3].y);
                *reinterpret_cast<float4*>(p + 512) = make_float4(st[i][0].z, st[i][1].z, st[i][2].z, st[i][3].z);
                *reinterpret_cast<float4*>(p + 768) = make_float4(st[i][0].w, st[i][1].w, st[i][2].w, st[i][3].w);
            }
        }
    };
    const std::integral_constant<int, 0> i_first;
    const std::integral_constant<int, NPRE> i_pre;
    const std::integral_constant<int, NI> i_all;

    // ---- DW: B of this lane's tokens for the row of each of its octets, through LDS so that the global
    // reads are contiguous runs; all lane groups of a spread octet work on the row of lane group 0.  The loads
    // of all blocks go out together and as many blocks as the LDS holds pass between two barriers: block by block
    // the prologue waited for memory Q times (dW of 1024 -> 4096, 4099 tokens, density 0.04, bf16: 94 -> 84 us).
    float xr[DW ? Q : 1][8];
    if constexpr (DW) {
        constexpr int AREAS = walk_areas(Q), NB4 = WT * RB / 4 / WALK_NT;
        const TIn* __restrict__ B = static_cast<const TIn*>(sd.B);
        const uint32_t ldb = (uint32_t)R * (uint32_t)sizeof(TIn);
        int rm[Q];
        float4 bq[Q][NB4];
#pragma unroll
        for (int q = 0; q < Q; ++q) rm[q] = sd.rowmap[((b0 + q) * OPB + octet_of(wave, q)) * OCT + g];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int row0 = (b0 + q) * RB;
            // (a block past the last row: no accesses, zeros)
            const uint32_t end = row0 < R ? rows * ldb - (uint32_t)row0 * (uint32_t)sizeof(TIn) : 0u;
            const __amdgpu_buffer_rsrc_t rs = buffer_of(B + (int64_t)t0 * R + (row0 < R ? row0 : 0), end);
#pragma unroll
            for (int it = 0; it < NB4; ++it) {
                const int item = it * WALK_NT + tid, tl = item / (RB / 4), j = item % (RB / 4);
                bq[q][it] = buffer_quad<TIn>(rs, (uint32_t)tl * ldb + (uint32_t)(4 * j) * (uint32_t)sizeof(TIn), end, (R & 1) == 0);
            }
        }
#pragma unroll
        for (int q0 = 0; q0 < Q; q0 += AREAS) {
            if (q0 > 0) __syncthreads();
#pragma unroll
            for (int q = q0; q < min(Q, q0 + AREAS); ++q)
#pragma unroll
                for (int it = 0; it < NB4; ++it) {
                    const int item = it * WALK_NT + tid, tl = item / (RB / 4), j = item % (RB / 4);
                    *reinterpret_cast<float4*>(lds + (q - q0) * STAGE_BYTES + stage_unit(tl, j)) = bq[q][it];
                }
            __syncthreads();
#pragma unroll
            for (int q = q0; q < min(Q, q0 + AREAS); ++q) {
                const int row = (rm[q] & SPREAD_FLAG) ? __builtin_amdgcn_readfirstlane(rm[q]) : rm[q];
                const int rl = (row & ~SPREAD_FLAG) - (b0 + q) * RB;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    xr[q][e] = *reinterpret_cast<const float*>(lds + (q - q0) * STAGE_BYTES + stage_byte(lane_token(s, g, e), rl & (RB - 1)));
            }
        }
    }
    float acc[OUT ? Q : 1][8];
    if constexpr (OUT) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[q][e] = 0.f;
    }

    // first and last pairs of this wavefront's octets in a chunk: the same in all lanes, read through
    // scalar loads one chunk ahead
    int pb[Q], pe[Q];
    auto pointers = [&](int c, int (&x)[Q], int (&y)[Q]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const_int* pp = (const_int*)sd.ptr + ((int64_t)c * sd.NBpad + b0 + q) * OPB + octet_of(wave, q);
            x[q] = pp[0];
            y[q] = pp[1];
        }
    };
    pointers(c_begin, pb, pe);
    fetch(c_begin, i_first, i_pre);
    for (int c = c_begin; c < c_end; ++c) {
        if (DW || c > c_begin) __syncthreads();
        put(i_first, i_pre);
        if (nkq > 64 * NPRE) { fetch(c, i_pre, i_all); put(i_pre, i_all); }
        int nb[Q], ne[Q];
        pointers(c + 1 < c_end ? c + 1 : c, nb, ne);
        // first pair of what is walked from octet q on (an empty segment is passed over); the last one is not
        // used, a batch there stays in the tail
        int from[Q + 1];
        from[Q] = pe[Q - 1];
#pragma unroll
        for (int q = Q - 1; q >= 0; --q) from[q] = pe[q] > pb[q] ? pb[q] : from[q + 1];
        uint4 nxt = load_batch(sd.ent, from[0], ebyte);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            // (see the head: the fewer octets are left, the less priority a wavefront has)
            constexpr bool HALVES = OUT && DW;
            if (HALVES ? q < Q - 1 : q < Q - 3) __builtin_amdgcn_s_setprio(3);
            else if (!HALVES && q == Q - 3) __builtin_amdgcn_s_setprio(2);
            else if (HALVES || q == Q - 2) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
            int p = pb[q];
            const int pend = pe[q];
            const int after = from[q + 1];                    // first batch of what is walked next
            float (&ac)[8] = acc[OUT ? q : 0];
            float (&xq)[8] = xr[DW ? q : 0];
            f32x4 xa[2], xb[2];
            uint4 cur;
            float r0 = 0.f;
            auto rd = [&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                const uint32_t a = lbase ^ quad_bcast<(i >> 1)>((i & 1) ? cur.z : cur.x);
                xa[i & 1] = *(lds_f32x4*)(a);
                xb[i & 1] = *(lds_f32x4*)(a ^ 128u);
            };
            auto use = [&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value, JJ = i >> 1, b = i & 1;
                float d = 0.f;
                if constexpr (DW) {
                    d = xq[0] * xa[b].x;
                    d = fmaf(xq[1], xa[b].y, d); d = fmaf(xq[2], xa[b].z, d); d = fmaf(xq[3], xa[b].w, d);
                    d = fmaf(xq[4], xb[b].x, d); d = fmaf(xq[5], xb[b].y, d);
                    d = fmaf(xq[6], xb[b].z, d); d = fmaf(xq[7], xb[b].w, d);
                }
                if constexpr (OUT) {
                    const uint32_t w = (i & 1) ? cur.w : cur.y;
                    if constexpr (JJ == 0) MST_FMA8_BC(0, ac, w, xa[b], xb[b]);
                    else if constexpr (JJ == 1) MST_FMA8_BC(1, ac, w, xa[b], xb[b]);
                    else if constexpr (JJ == 2) MST_FMA8_BC(2, ac, w, xa[b], xb[b]);
                    else MST_FMA8_BC(3, ac, w, xa[b], xb[b]);
                }
                if constexpr (DW && b == 0) r0 = d;
                if constexpr (DW && b == 1)                   // a pair is complete: four lanes store the same sum
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sum8_pair(r0, d)),
                                                          buffer_of(pt + (int64_t)(p + JJ) * (2 * OCT), 2 * OCT * 4), (int)pbyte, 0, 0);
            };
            // The NP pairs of the batch held in `nxt`, with the batch at pair pn fetched meanwhile.  The reads of
            // step i + 1 are issued before the arithmetic of step i; the compiler on its own reads, waits and
            // multiplies step by step.  (The copy out of nxt is spelt out: left to the compiler a part of it
            // lands at the end of the loop, behind a wait for the batch that was just requested.)
            auto batch = [&](auto npc, int pn) __attribute__((always_inline)) {
                constexpr int NS = 2 * decltype(npc)::value;
                asm volatile("v_mov_b32 %0, %4\n\tv_mov_b32 %1, %5\n\tv_mov_b32 %2, %6\n\tv_mov_b32 %3, %7"
                             : "=&v"(cur.x), "=&v"(cur.y), "=&v"(cur.z), "=&v"(cur.w)
                             : "v"(nxt.x), "v"(nxt.y), "v"(nxt.z), "v"(nxt.w));
                nxt = load_batch(sd.ent, pn, ebyte);
                __builtin_amdgcn_sched_barrier(0);
                static_for<NS + 1>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (i < NS) rd(ic);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (i > 0) {
                        use(std::integral_constant<int, i - 1>{});
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
            };
            const int mid = (p + pend) >> 1;
            while (p + 4 <= pend) {
                if (HALVES && q == Q - 2 && p >= mid) __builtin_amdgcn_s_setprio(2);
                if (HALVES && q == Q - 1 && p >= mid) __builtin_amdgcn_s_setprio(0);
                batch(std::integral_constant<int, 4>{}, p + 4 < pend ? p + 4 : after);
                p += 4;
            }
            const int rem = pend - p;
            if (rem == 1) batch(std::integral_constant<int, 1>{}, after);
            else if (rem == 2) batch(std::integral_constant<int, 2>{}, after);
            else if (rem == 3) batch(std::integral_constant<int, 3>{}, after);
        }
        if (c + 1 < c_end) fetch(c + 1, i_first, i_pre);
#pragma unroll
        for (int q = 0; q < Q; ++q) { pb[q] = nb[q]; pe[q] = ne[q]; }
    }

    // ---- OUT: a block at a time through LDS (two staging areas in turn), so that every token's 128 rows
    // leave as one contiguous run
    if constexpr (OUT) {
        float* const out = wa.out + (int64_t)blockIdx.y * T * R;
        int tid_e = threadIdx.x;                              // (lane constants worked out again)
        asm volatile("" : "+v"(tid_e));
        const int g_e = (tid_e >> 3) & 7, s_e = tid_e & 7;
        bool nan = false;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int row0 = (b0 + q) * RB;
            if (row0 >= R) break;
            char* half = lds + (q & 1) * STAGE_BYTES;
            const int rm = sd.rowmap[((b0 + q) * OPB + octet_of(wave, q)) * OCT + g_e];
            if (__builtin_amdgcn_readfirstlane(rm & SPREAD_FLAG)) {
                // one long row dealt over the lane groups: group 0 takes the sum of all eight, the others -- whose
                // output positions belong to empty rows -- zero (odd groups hold the token halves exchanged)
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (g_e & 1) ? acc[q][e ^ 4] : acc[q][e];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[e] += __shfl_xor(v[e], 8, 64);
                    v[e] += __shfl_xor(v[e], 16, 64);
                    v[e] += __shfl_xor(v[e], 32, 64);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[q][e] = g_e == 0 ? v[e] : 0.f;
            }
            const int rl = (rm & ~SPREAD_FLAG) - row0;
#pragma unroll
            for (int e = 0; e < 8; ++e) *reinterpret_cast<float*>(half + stage_byte(lane_token(s_e, g_e, e), rl)) = acc[q][e];
            __syncthreads();
#pragma unroll
            for (int it = 0; it < WT * RB / 4 / WALK_NT; ++it) {
                const int item = it * WALK_NT + tid_e, tl = item / (RB / 4), j = item % (RB / 4);
                const int t = t0 + tl, row = row0 + 4 * j;
                if (t < T && row < R) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(half + stage_unit(tl, j));
                    float* o = out + (int64_t)t * R + row;
                    // streaming stores: the output is not read again by this kernel and should not push the
                    // activation tiles out of the L2
                    typedef f32x4 f32x4_dword __attribute__((aligned(4)));
                    if (row + 3 < R) {
                        __builtin_nontemporal_store(v, reinterpret_cast<f32x4_dword*>(o));
                    } else {
                        __builtin_nontemporal_store(v.x, o);
                        if (row + 1 < R) __builtin_nontemporal_store(v.y, o + 1);
                        if (row + 2 < R) __builtin_nontemporal_store(v.z, o + 2);
                    }
                    nan |= __builtin_isunordered(v.x, v.y) | __builtin_isunordered(v.z, v.w);
                }
            }
        }
        if (nan) {                                            // (see own_entries_sum)
#pragma unroll 1
            for (int i = 0; i < Q * (WT * RB / WALK_NT); ++i) {
                const int item = (i / 4) % (WT * RB / 4 / WALK_NT) * WALK_NT + tid_e, tl = item / (RB / 4);
                const int t = t0 + tl, row = (b0 + i / (WT * RB / WALK_NT)) * RB + 4 * (item % (RB / 4)) + (i & 3);
                if (t >= T || row >= R) continue;
                float* o = out + (int64_t)t * R + row;
                if (*o != *o) *o = own_entries_sum<TIn>(t, row);
            }
        }
    }
}

}  // namespace mst
