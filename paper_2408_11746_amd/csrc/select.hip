// Exact k-selection with index tie-break, and the device side of one Mixed-Growing
// update (Algorithm 1: ArgTopK of -|theta . M|, ArgTopK of |grad| over the inactive
// positions, RandK over the rest, then the mask / weight update).
//
// Each of the three selections is "the k candidates with the smallest (key, index)":
//   prune   candidates = active weights,            key = |w| bits            (32 bit)
//   grad    candidates = inactive positions,        key = 0x7FFFFFFF - |g| bits (32 bit)
//   random  candidates = inactive, not grad-grown,  key = SplitMix64(seed)[f]  (64 bit)
// A most-significant-digit radix select (the keys have 31 bits: digits of 10, 11 and 10, one kernel per digit; every
// block of the next kernel picks the bin for itself; the search stops early when a bin holds
// exactly the keys still wanted) finds the k-th smallest key tau on the device; a last ordered pass takes every key
// below tau and, among the keys equal to tau, the lowest indices until k are taken.
// Nothing is read back to the host.
//
// The chain is bound by its launches and by what a block costs whatever it reads (waiting for memory, clearing and
// summing histograms): a layer of 3072 x 768 has 12 MB to read in a pass, 2 us for the chip.  So it has seven links: start,
// three digits, flags with the random selection's histogram, that selection's list, its end beside the pruning.
#include "common.h"

namespace mst {

__device__ inline uint32_t abs_bits(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

__device__ inline uint64_t splitmix64_at(uint64_t seed, uint64_t f) {
    uint64_t z = seed + (f + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// A key source answers get(i, key): is index i a candidate, and with which key.  get4 does the
// same for the four indices i .. i+3 of an aligned group (i a multiple of 4, all below n) with
// vector loads where the arrays allow it.
// |w|, or with lambda (flat and G then given) |w| + lambda |grad|, both roundings explicit (no contraction into one fused
// operation); a non-negative float orders like its bit pattern
struct PruneKeys {
    typedef uint32_t key_t;
    const float* vals;
    const int* flat;
    const float* G;
    float lambda;
    __device__ bool get(int64_t k, key_t& key) const {
        key = lambda == 0.f ? abs_bits(vals[k]) : __float_as_uint(__fadd_rn(fabsf(vals[k]), __fmul_rn(lambda, fabsf(G[flat[k]]))));
        return true;
    }
    __device__ void get4(int64_t k, key_t (&key)[4], bool (&ok)[4]) const {
        if (lambda == 0.f) {
            const float4 v = *reinterpret_cast<const float4*>(vals + k);
            key[0] = abs_bits(v.x); key[1] = abs_bits(v.y); key[2] = abs_bits(v.z); key[3] = abs_bits(v.w);
            ok[0] = ok[1] = ok[2] = ok[3] = true;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) ok[u] = get(k + u, key[u]);
        }
    }
};
struct GradKeys {
    typedef uint32_t key_t;
    const float* G;
    const uint8_t* mask;
    __device__ bool get(int64_t f, key_t& key) const {
        if (mask[f]) return false;
        key = 0x7FFFFFFFu - abs_bits(G[f]);
        return true;
    }
    __device__ void get4(int64_t f, key_t (&key)[4], bool (&ok)[4]) const {
        const uint32_t m = *reinterpret_cast<const uint32_t*>(mask + f);
        const float4 g = *reinterpret_cast<const float4*>(G + f);
        key[0] = 0x7FFFFFFFu - abs_bits(g.x); key[1] = 0x7FFFFFFFu - abs_bits(g.y);
        key[2] = 0x7FFFFFFFu - abs_bits(g.z); key[3] = 0x7FFFFFFFu - abs_bits(g.w);
        ok[0] = (m & 0xFFu) == 0; ok[1] = (m & 0xFF00u) == 0; ok[2] = (m & 0xFF0000u) == 0; ok[3] = (m & 0xFF000000u) == 0;
    }
};
struct RandKeys {
    typedef uint64_t key_t;
    const uint8_t* mask;
    const uint8_t* sel;
    uint64_t seed;
    __device__ bool get(int64_t f, key_t& key) const {
        if (mask[f] || sel[f]) return false;
        key = splitmix64_at(seed, (uint64_t)f);
        return true;
    }
    __device__ void get4(int64_t f, key_t (&key)[4], bool (&ok)[4]) const {
        const uint32_t m = *reinterpret_cast<const uint32_t*>(mask + f) | *reinterpret_cast<const uint32_t*>(sel + f);
        ok[0] = (m & 0xFFu) == 0; ok[1] = (m & 0xFF00u) == 0; ok[2] = (m & 0xFF0000u) == 0; ok[3] = (m & 0xFF000000u) == 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) key[u] = splitmix64_at(seed, (uint64_t)(f + u));
    }
};

// Keys of G aligned groups of four indices, `stride` apart, of which those below n4 (a multiple of 4, at least 4) exist.  The
// others read the last group there is and are no candidates: with a branch for each the loads of one group are waited for
// before those of the next go out (a digit pass of 3072 x 768 took 16 us instead of 7).  The up to three indices behind the last
// group are the caller's.
template <int G, typename KS>
__device__ __forceinline__ void keys_of_groups(const KS& ks, int64_t i0, int64_t stride, int64_t n4, typename KS::key_t (&key)[G][4], bool (&ok)[G][4]) {
#pragma unroll
    for (int v = 0; v < G; ++v) ks.get4(min(i0 + v * stride, n4 - 4), key[v], ok[v]);
#pragma unroll
    for (int v = 0; v < G; ++v)
#pragma unroll
        for (int u = 0; u < 4; ++u) ok[v][u] = ok[v][u] && i0 + v * stride < n4;
}

// State of one selection (uint64 words).  Random growth: [0] key prefix fixed so far, [1] how many still to take inside the
// prefix, [2] mode (0: keys below [0] are taken and the first [1] keys equal to it in index order; 1: every key <= [0]
// is taken, the search ended early; 2: keys below [0] and keys equal to it with index <= [6]), [4] length of its
// candidate list, [6] index cut of mode 2.  The others: [3] tickets of the flag pass, [8..10] prefix, count and mode after the
// first digit, [11..13] after the second.  All: [5] how many to take; from word SEL_CTRL on the uint32 histograms.
// All states of an update are set by k_update_init.

constexpr int SEL_NT = 1024;     // threads of a histogram block (16 wavefronts share one LDS histogram)

// A digit's histogram in the state: `copies` of it (block b adds to copy b mod copies: the first digit, the exponent and
// two more bits, has a handful of hot bins, and hundreds of blocks adding to the same addresses queue up at the memory side).
template <int P> struct Digit;
template <> struct Digit<1> { static constexpr int bits = 10, shift = 21, copies = 4, at = 0; };
template <> struct Digit<2> { static constexpr int bits = 11, shift = 10, copies = 1, at = 4096; };
template <> struct Digit<3> { static constexpr int bits = 10, shift = 0, copies = 1, at = 6144; };
static_assert(SEL_CTRL + (6144 + 1024) / 2 <= SEL_STATE_WORDS, "the three histograms");
__device__ inline uint32_t* histogram(uint64_t* state) { return reinterpret_cast<uint32_t*>(state + SEL_CTRL); }
__device__ inline const uint32_t* histogram(const uint64_t* state) { return reinterpret_cast<const uint32_t*>(state + SEL_CTRL); }

// The bin with (total before it) < need <= (total including it), by a block of SEL_NT threads from a histogram that an
// earlier kernel finished.  (Done by every block of the kernel that wants it: the histogram is a few KB in the L2, while a
// last block that picks for all of them is a ticket, a round trip and a scan at the end of every pass.)
struct PickShared {
    uint32_t wsum[SEL_NT / 64], bin, before, count;
};
template <int BINS, int COPIES>
__device__ void pick_bin(const uint32_t* __restrict__ hist, uint32_t need, PickShared& sh) {
    constexpr int PER = BINS / SEL_NT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t c[PER], tot = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        c[u] = 0;
#pragma unroll
        for (int g = 0; g < COPIES; ++g) c[u] += hist[g * BINS + tid * PER + u];
        tot += c[u];
    }
    uint32_t x = tot;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) sh.wsum[wave] = x;
    if (tid == 0) { sh.bin = BINS - 1; sh.before = 0; sh.count = 0; }
    __syncthreads();
    uint32_t before = x - tot;
    for (int w = 0; w < wave; ++w) before += sh.wsum[w];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (before < need && before + c[u] >= need) { sh.bin = (uint32_t)(tid * PER + u); sh.before = before; sh.count = c[u]; }
        before += c[u];
    }
    __syncthreads();
}

// What the search knows after a digit
struct Search {
    uint32_t prefix, need;
    int mode;
};
template <int P>
__device__ void pick_digit(const uint64_t* __restrict__ state, Search& f, PickShared& sh) {
    pick_bin<1 << Digit<P>::bits, Digit<P>::copies>(histogram(state) + Digit<P>::at, f.need, sh);
    f.prefix |= sh.bin << Digit<P>::shift;
    f.need -= sh.before;
    if (f.need == sh.count) {                        // the whole bin is wanted: no ties to break, no digits left to look at
        f.prefix |= (1u << Digit<P>::shift) - 1u;
        f.mode = 1;
    }
}
// after digit P - 1; block 0 leaves it for the kernels behind the next one
template <int P>
__device__ Search search_before(uint64_t* __restrict__ state, bool keep, PickShared& sh) {
    Search f{0u, (uint32_t)state[5], 0};
    if constexpr (P >= 3) f = Search{(uint32_t)state[3 * P - 1], (uint32_t)state[3 * P], (int)state[3 * P + 1]};
    if constexpr (P >= 2) {
        if (f.mode == 0) pick_digit<P - 1>(state, f, sh);
        if (keep && threadIdx.x == 0) {
            state[3 * P + 2] = f.prefix;
            state[3 * P + 3] = f.need;
            state[3 * P + 4] = (uint64_t)f.mode;
        }
    }
    return f;
}

// One digit of the search by block `blk` of `nblk`: every block adds its LDS histogram of the
// digit (of the keys that match the prefix) to the global one.
// The LDS histogram keeps 16 (8) copies of every bin, one per lane mod 16 (8), 64 KB in all: with a single copy the
// hot bins of the leading digit (exponent bits of |w| and |grad|) serialise the whole pass.
struct DigitShared {
    alignas(16) uint32_t h[16384];
    PickShared pick;
};

template <int P, typename KS>
__device__ void select_digit_block(KS ks, int64_t n, uint64_t* __restrict__ state, int blk, int nblk, DigitShared& sh) {
    constexpr int BINS = 1 << Digit<P>::bits, COPIES = 16384 / BINS, shift = Digit<P>::shift, bits = Digit<P>::bits, GROUPS = 4;
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < 16384 / 4; i += SEL_NT) reinterpret_cast<uint4*>(sh.h)[i] = make_uint4(0u, 0u, 0u, 0u);
    // a thread takes aligned groups of four consecutive indices (vector loads), four groups per round; the first round's loads
    // go out before the bin of the digit before is picked
    const int64_t stride = (int64_t)nblk * SEL_NT * 4, n4 = n & ~(int64_t)3;
    int64_t i0 = ((int64_t)blk * SEL_NT + tid) * 4;
    uint32_t key[GROUPS][4];
    bool ok[GROUPS][4];
    if (n4 > 0) keys_of_groups(ks, i0, stride, n4, key, ok);
    const Search f = search_before<P>(state, blk == 0, sh.pick);
    if (f.mode != 0) return;                         // search already over (same value for every thread)
    __syncthreads();
    auto add = [&](uint32_t k, bool is) __attribute__((always_inline)) {
        if (!is || (P > 1 && (k >> (shift + bits)) != (f.prefix >> (shift + bits)))) return;
        atomicAdd(&sh.h[((k >> shift) & (BINS - 1)) * COPIES + (lane & (COPIES - 1))], 1u);
    };
    while (i0 < n4) {
#pragma unroll
        for (int v = 0; v < GROUPS; ++v)
#pragma unroll
            for (int u = 0; u < 4; ++u) add(key[v][u], ok[v][u]);
        i0 += GROUPS * stride;
        if (i0 < n4) keys_of_groups(ks, i0, stride, n4, key, ok);
    }
    if (blk == 0 && tid < (int)(n - n4)) {
        uint32_t k = 0;
        const bool is = ks.get(n4 + tid, k);
        add(k, is);
    }
    __syncthreads();
    // (the kernels that read the global histogram come later on the stream: plain adds, nothing to wait for)
    uint32_t* const gmine = histogram(state) + Digit<P>::at + (blk % Digit<P>::copies) * BINS;
#pragma unroll
    for (int b = 0; b < BINS / SEL_NT; ++b) {
        const int bin = b * SEL_NT + tid;
        uint32_t c = 0;
#pragma unroll
        for (int r = 0; r < COPIES; r += 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(&sh.h[bin * COPIES + r]);
            c += v.x + v.y + v.z + v.w;
        }
        if (c) atomicAdd(&gmine[bin], c);
    }
}

// What the flag pass of a selection does with index i beyond flags[i] = code for a selected one.
struct FlagSink {
    uint8_t* flags;
    uint8_t code;
    int full;            // 1: every index below n gets its flag (0 if not selected); 0: only the selected ones are written
    uint8_t* grow_mask;  // not null: a selected position becomes active ...
    float* grow_w;       // ... and its weight in the dense scratch starts at zero
    __device__ void put(int64_t i, bool take) const {
        if (take) {
            flags[i] = code;
            if (grow_mask) { grow_mask[i] = 1; grow_w[i] = 0.f; }
        } else if (full) {
            flags[i] = 0;
        }
    }
    // an aligned group of four (full): one store for their flags
    __device__ void put4(int64_t i, const bool (&take)[4]) const {
        const uint32_t c = code;
        *reinterpret_cast<uint32_t*>(flags + i) = (take[0] ? c : 0u) | (take[1] ? c << 8 : 0u) | (take[2] ? c << 16 : 0u) | (take[3] ? c << 24 : 0u);
        if (grow_mask)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (take[u]) { grow_mask[i + u] = 1; grow_w[i + u] = 0.f; }
    }
};

// Two independent selections of every layer (the prune set over its nnz active weights, the gradient-growth set over all N
// positions) share their passes: the first nb0 blocks of a layer work on the first, the others on the second (no blocks:
// no such selection).
struct SelectArgs {
    PruneKeys pk;
    GradKeys gk;
    int64_t nnz, N;
    uint64_t *st_p, *st_g;
    int dig0, dig1;      // blocks for the first and for the second
};
template <int P, int CAP>
__global__ __launch_bounds__(SEL_NT) void k_select_digit(const Batch<SelectArgs, CAP> batch) {
    __shared__ DigitShared sh;
    if (batch.surplus()) return;
    const unsigned b = blockIdx.x;
    const SelectArgs a = batch.entry();
    if ((int)b < a.dig0) select_digit_block<P>(a.pk, a.nnz, a.st_p, (int)b, a.dig0, sh);
    else select_digit_block<P>(a.gk, a.N, a.st_g, (int)b - a.dig0, a.dig1, sh);
}

// The inactive positions, without keys (a random selection with no gradient growth before it)
struct InactiveKeys {
    typedef uint32_t key_t;
    const uint8_t* mask;
    __device__ bool get(int64_t f, key_t& key) const { key = 0xFFFFFFFFu; return mask[f] == 0; }
    __device__ void get4(int64_t f, key_t (&key)[4], bool (&ok)[4]) const {
        const uint32_t m = *reinterpret_cast<const uint32_t*>(mask + f);
        key[0] = key[1] = key[2] = key[3] = 0xFFFFFFFFu;
        ok[0] = (m & 0xFFu) == 0; ok[1] = (m & 0xFF00u) == 0; ok[2] = (m & 0xFF0000u) == 0; ok[3] = (m & 0xFF000000u) == 0;
    }
};

constexpr int RAND_TOP_BITS = 10, RAND_BINS = 1 << RAND_TOP_BITS, RAND_SHIFT = 64 - RAND_TOP_BITS;
static_assert(RAND_BINS == SEL_NT, "one bin per thread");

struct FlagShared {
    PickShared pick;
    uint32_t h[RAND_BINS];
    uint32_t wsum[SEL_NT / 64];
    uint32_t range;
};

// sum over the block (every thread gets it) and sum over the threads before this one
__device__ inline uint32_t block_scan(uint32_t v, uint32_t& before, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    __syncthreads();                                 // (wsum free again)
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint32_t total = 0;
    before = x - v;
    for (int w = 0; w < SEL_NT / 64; ++w) {
        if (w < wave) before += wsum[w];
        total += wsum[w];
    }
    return total;
}

// Flags of a contiguous range of `per` indices (a multiple of 4 SEL_NT).  state null: nothing is selected.  Keys equal to the
// threshold are taken in index order: a key's rank is the count of such keys in the ranges before this one plus
// those before it in the range.  The blocks count them first and tell each other (a range is handed out by ticket, so that the
// ranges a block waits for belong to blocks that are running or done, and they count before they wait).
// RAND: the candidates that are left go into the histogram of the random selection, in the same pass: its keys are hashes of
// the index, so there are no hot bins and one LDS copy does.
template <bool RAND, typename KS>
__device__ void select_flag_block(KS ks, int64_t n, uint64_t* __restrict__ state, int* __restrict__ blk, const FlagSink& sink,
                                  int64_t per, int b, uint64_t seed, uint64_t* __restrict__ rand_state, FlagShared& sh) {
    const int tid = threadIdx.x;
    constexpr int ROUND = 4 * SEL_NT, GROUPS = 4;
    if constexpr (RAND) sh.h[tid] = 0;
    Search f{0u, 0u, 1};
    if (state) {
        f = Search{(uint32_t)state[11], (uint32_t)state[12], (int)state[13]};
        if (f.mode == 0) pick_digit<3>(state, f, sh.pick);
    }
    __syncthreads();
    auto rest = [&](int64_t i, bool left) __attribute__((always_inline)) {
        if constexpr (RAND)
            if (left) atomicAdd(&sh.h[(uint32_t)(splitmix64_at(seed, (uint64_t)i) >> RAND_SHIFT)], 1u);
    };
    const int64_t n4 = n & ~(int64_t)3;
    if (f.mode != 0) {
        const int64_t lo = (int64_t)b * per, hi = min(n4, lo + per);
        for (int64_t i0 = lo + 4 * tid; i0 < hi; i0 += GROUPS * ROUND) {
            uint32_t key[GROUPS][4];
            bool ok[GROUPS][4], take[4];
            keys_of_groups(ks, i0, ROUND, hi, key, ok);
#pragma unroll
            for (int v = 0; v < GROUPS; ++v) {
#pragma unroll
                for (int u = 0; u < 4; ++u) take[u] = state && ok[v][u] && key[v][u] <= f.prefix;
                if (i0 + v * ROUND < hi) sink.put4(i0 + v * ROUND, take);
#pragma unroll
                for (int u = 0; u < 4; ++u) rest(i0 + v * ROUND + u, ok[v][u] && !take[u]);
            }
        }
        if (n4 >= lo && n4 < lo + per && tid < (int)(n - n4)) {
            uint32_t key = 0;
            const bool ok = ks.get(n4 + tid, key), take = state && ok && key <= f.prefix;
            sink.put(n4 + tid, take);
            rest(n4 + tid, ok && !take);
        }
    } else {
        if (tid == 0) sh.range = (uint32_t)atomicAdd(reinterpret_cast<unsigned long long*>(state + 3), 1ull);
        __syncthreads();
        const int range = (int)sh.range;
        const int64_t lo = (int64_t)range * per, hi = min(n, lo + per);
        // (a thread's four indices: one group)
        auto group = [&](int64_t i4, uint32_t (&key)[4], bool (&ok)[4]) __attribute__((always_inline)) {
            if (i4 + 3 < n) {
                ks.get4(i4, key, ok);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) ok[u] = i4 + u < n && ks.get(i4 + u, key[u]);
            }
            uint32_t eq = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) eq += ok[u] && key[u] == f.prefix;
            return eq;
        };
        uint32_t key[4], eq = 0, before = 0;
        bool ok[4], take[4];
        for (int64_t i4 = lo + 4 * tid; i4 < hi; i4 += ROUND) eq += group(i4, key, ok);
        eq = block_scan(eq, before, sh.wsum);
        if (tid == 0) __hip_atomic_store(&blk[range], (int)(eq + 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        eq = 0;
        for (int r = tid; r < range; r += SEL_NT) {
            int c;
            while ((c = __hip_atomic_load(&blk[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) __builtin_amdgcn_s_sleep(2);
            eq += (uint32_t)c - 1u;
        }
        uint32_t rank = block_scan(eq, before, sh.wsum);
        for (int64_t j = lo; j < hi; j += ROUND) {
            const int64_t i4 = j + 4 * tid;
            eq = group(i4, key, ok);
            const uint32_t total = block_scan(eq, before, sh.wsum);
            before += rank;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                take[u] = ok[u] && key[u] < f.prefix;
                if (ok[u] && key[u] == f.prefix) { take[u] = before < f.need; ++before; }
            }
            rank += total;
            if (i4 + 3 < n) sink.put4(i4, take);
            else for (int u = 0; u < 4; ++u)
                if (i4 + u < n) sink.put(i4 + u, take[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) rest(i4 + u, ok[u] && !take[u]);
        }
    }
    if constexpr (RAND) {
        __syncthreads();
        const uint32_t c = sh.h[tid];
        if (c) atomicAdd(&histogram(rand_state)[tid], c);
    }
}

struct FlagArgs {
    PruneKeys pk;
    GradKeys gk;
    int64_t nnz, N, per_p, per_g;                    // indices of a block
    uint64_t *st_p, *st_g, *st_r;                    // st_g null: no gradient growth; st_r null: no random growth
    int *blk_p, *blk_g;
    FlagSink sink_p, sink_g;
    uint64_t seed;
    int nb0;                                         // blocks for the prune selection
};
template <int CAP>
__global__ __launch_bounds__(SEL_NT) void k_select_flag(const Batch<FlagArgs, CAP> batch) {
    __shared__ FlagShared sh;
    if (batch.surplus()) return;
    const unsigned b = blockIdx.x;
    const FlagArgs a = batch.entry();
    const int bg = (int)b - a.nb0;
    if (bg < 0) select_flag_block<false>(a.pk, a.nnz, a.st_p, a.blk_p, a.sink_p, a.per_p, (int)b, 0ull, nullptr, sh);
    else if (!a.st_g) select_flag_block<true>(InactiveKeys{a.gk.mask}, a.N, nullptr, nullptr, a.sink_g, a.per_g, bg, a.seed, a.st_r, sh);
    else if (!a.st_r) select_flag_block<false>(a.gk, a.N, a.st_g, a.blk_g, a.sink_g, a.per_g, bg, 0ull, nullptr, sh);
    else select_flag_block<true>(a.gk, a.N, a.st_g, a.blk_g, a.sink_g, a.per_g, bg, a.seed, a.st_r, sh);
}

// ---- the random selection.  Its keys are 64-bit hashes of the index: uniform, and distinct for
// distinct indices.  The flag pass before it builds the histogram of the top 10 bits; one pass picks the bin of the k-th key
// and appends the candidates of that bin -- about n / 1024 of them -- to a list; one block finishes the search on the list
// (seven more 8-bit digits, then the index cut among equal keys).  Selected positions are marked
// where they are decided: candidates below the picked bin by the list pass, those inside it by
// the finishing block.
struct RandItem {
    uint64_t key;
    int64_t f;
};

struct RandArgs {
    RandKeys ks;
    int64_t n;
    uint64_t* state;
    RandItem* list;
    FlagSink sink;
};

// block of 1024 threads, 16 indices each.  Candidates in a bin below the picked one are selected on
// the spot; those of the picked bin (about 16 per block) are gathered in LDS and appended to the
// list with ONE add to its length (an add per hit would queue up at the counter)
constexpr int COMPACT_PER_BLOCK = SEL_NT * 16, COMPACT_STAGE = 512;
template <int CAP>
__global__ __launch_bounds__(SEL_NT) void k_rand_compact(const Batch<RandArgs, CAP> batch) {       // COMPACT_PER_BLOCK indices per block
    if (batch.surplus()) return;
    const unsigned blk = blockIdx.x;
    const RandArgs a = batch.entry();
    const RandKeys ks = a.ks;
    const int64_t n = a.n;
    uint64_t* __restrict__ state = a.state;
    RandItem* __restrict__ list = a.list;
    const FlagSink sink = a.sink;
    __shared__ RandItem stage[COMPACT_STAGE];
    __shared__ unsigned int nstage;
    __shared__ unsigned long long base_s;
    __shared__ PickShared pick;
    const int tid = threadIdx.x;
    if (tid == 0) nstage = 0;
    const uint32_t k = (uint32_t)state[5];
    pick_bin<RAND_BINS, 1>(histogram(state), k, pick);
    const uint64_t top = pick.bin;
    const uint32_t need = k - pick.before;
    const bool whole_bin = need == pick.count;       // every candidate of the picked bin is wanted: no list
    if (blk == 0 && tid == 0) {
        state[0] = (top << RAND_SHIFT) | (whole_bin ? (1ull << RAND_SHIFT) - 1ull : 0ull);
        state[1] = need;
        state[2] = whole_bin ? 1 : 0;
    }
    unsigned long long* len = reinterpret_cast<unsigned long long*>(state + 4);
    const int64_t b0 = (int64_t)blk * COMPACT_PER_BLOCK, n4 = n & ~(int64_t)3;
    auto item = [&](int64_t i, uint64_t key, bool is) __attribute__((always_inline)) {
        if (!is) return;
        const uint64_t bin = key >> RAND_SHIFT;
        if (bin < top || (whole_bin && bin == top)) {     // decided here: selected (each thread owns its indices)
            sink.put(i, true);
            return;
        }
        if (bin != top) return;
        const unsigned int at = atomicAdd(&nstage, 1u);
        if (at < COMPACT_STAGE) stage[at] = RandItem{key, i};
        else list[atomicAdd(len, 1ull)] = RandItem{key, i};      // (a block with more hits than the stage holds)
    };
    constexpr int GROUPS = COMPACT_PER_BLOCK / (4 * SEL_NT);
    const int64_t i0 = b0 + 4 * tid;
    if (i0 < n4) {
        uint64_t key[GROUPS][4];
        bool ok[GROUPS][4];
        keys_of_groups(ks, i0, 4 * SEL_NT, n4, key, ok);
#pragma unroll
        for (int v = 0; v < GROUPS; ++v)
#pragma unroll
            for (int u = 0; u < 4; ++u) item(i0 + v * 4 * SEL_NT + u, key[v][u], ok[v][u]);
    }
    if (n4 >= b0 && n4 < b0 + COMPACT_PER_BLOCK && tid < (int)(n - n4)) {
        uint64_t key = 0;
        const bool is = ks.get(n4 + tid, key);
        item(n4 + tid, key, is);
    }
    __syncthreads();
    const unsigned int m = min(nstage, (unsigned int)COMPACT_STAGE);
    if (tid == 0 && m) base_s = atomicAdd(len, (unsigned long long)m);
    __syncthreads();
    for (unsigned int i = tid; i < m; i += SEL_NT) list[base_s + i] = stage[i];
}

// one block: the state[1]-th smallest (key, index) of the list decides the threshold.  Lists of up to
// RAND_LDS_KEYS items (the usual case by far) are searched in LDS.
constexpr int RAND_LDS_KEYS = 7168;
struct FinishShared {
    uint64_t keys[RAND_LDS_KEYS];
    uint32_t h[SEL_BINS];
    uint32_t wtot[4];
    uint64_t prefix, need;
    int done;
    long long cut;
};
__device__ void rand_finish(const RandArgs& a, FinishShared& sh) {
    uint64_t* __restrict__ state = a.state;
    const RandItem* __restrict__ list = a.list;
    const FlagSink sink = a.sink;
    uint64_t* const keys = sh.keys;
    uint32_t *const h = sh.h, *const wtot = sh.wtot;
    uint64_t &prefix_s = sh.prefix, &need_s = sh.need;
    int& done_s = sh.done;
    long long& cut_s = sh.cut;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (state[2] != 0) return;
    const int64_t c = (int64_t)state[4];
    const bool in_lds = c <= RAND_LDS_KEYS;
    if (in_lds)
        for (int64_t i = tid; i < c; i += SEL_NT) keys[i] = list[i].key;
    if (tid == 0) { prefix_s = state[0]; need_s = state[1]; done_s = 0; }
    __syncthreads();
    // the 54 bits below the top digit: six digits of 8 bits, then one of 6
    for (int top = RAND_SHIFT; top > 0 && !done_s; top -= SEL_DIGIT_BITS) {
        const int shift = max(0, top - SEL_DIGIT_BITS), width = top - shift;
        for (int i = tid; i < SEL_BINS; i += SEL_NT) h[i] = 0;
        __syncthreads();
        const uint64_t prefix = prefix_s;
        for (int64_t i = tid; i < c; i += SEL_NT) {
            const uint64_t key = in_lds ? keys[i] : list[i].key;
            if ((key >> top) == (prefix >> top)) atomicAdd(&h[(uint32_t)(key >> shift) & ((1u << width) - 1u)], 1u);
        }
        __syncthreads();
        // pick by the first 256 threads, one bin each: inclusive scan over the four wavefronts
        uint32_t cb = 0, x = 0;
        if (tid < SEL_BINS) {
            cb = h[tid];
            x = cb;
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t y = __shfl_up(x, d, 64);
                if (lane >= d) x += y;
            }
            if (lane == 63) wtot[wave] = x;
        }
        __syncthreads();
        if (tid < SEL_BINS) {
            uint64_t incl = x;
            for (int w = 0; w < wave; ++w) incl += wtot[w];
            const uint64_t k = need_s, before = incl - cb;
            if (before < k && incl >= k) {                // exactly one bin
                uint64_t pre = prefix | ((uint64_t)tid << shift);
                if (k - before == cb) {                   // the whole bin: every key <= prefix | ones is taken
                    pre |= shift ? ((1ull << shift) - 1ull) : 0ull;
                    done_s = 1;
                }
                prefix_s = pre;
                need_s = k - before;
            }
        }
        __syncthreads();
    }
    if (done_s) {                                     // every listed key <= prefix_s is taken
        const uint64_t top_key = prefix_s;
        for (int64_t i = tid; i < c; i += SEL_NT)
            if (list[i].key <= top_key) sink.put(list[i].f, true);
        if (tid == 0) { state[0] = prefix_s; state[1] = need_s; state[2] = 1; }
        return;
    }
    // equal keys (cannot happen with distinct indices, kept for exactness): the need_s lowest indices.
    // The cut is the need_s-th smallest index among the items whose key is the threshold.
    if (tid == 0) {
        const uint64_t tau = prefix_s, need = need_s;
        long long lo = -1;
        for (uint64_t r = 0; r < need; ++r) {          // repeated minimum above lo: need is 1 unless keys collide
            long long best = -1;
            for (int64_t i = 0; i < c; ++i)
                if (list[i].key == tau && list[i].f > lo && (best < 0 || list[i].f < best)) best = list[i].f;
            lo = best;
        }
        state[0] = tau;
        state[1] = need;
        state[2] = 2;
        state[6] = (uint64_t)lo;
        cut_s = lo;
    }
    __syncthreads();
    const uint64_t tau = prefix_s;
    const long long cut = cut_s;
    for (int64_t i = tid; i < c; i += SEL_NT) {
        const RandItem it = list[i];
        if (it.key < tau || (it.key == tau && (long long)it.f <= cut)) sink.put(it.f, true);
    }
}

// start of an update: the three selection states of every layer, and the counts that blocks of the flag pass wait for
struct InitArgs {
    uint64_t *state, k[SEL_STATES];
    int *blk_p, *blk_g, nb_p, nb_g;
};
template <int CAP>
__global__ __launch_bounds__(256) void k_update_init(const Batch<InitArgs, CAP> batch) {
    if (batch.surplus()) return;
    const unsigned b = blockIdx.x;
    const InitArgs a = batch.entry();
    const int64_t i = (int64_t)b * blockDim.x + threadIdx.x;
    if (i < (int64_t)SEL_STATES * SEL_STATE_WORDS) {
        const int w = (int)(i % SEL_STATE_WORDS), which = (int)(i / SEL_STATE_WORDS);
        a.state[i] = (w == 5) ? (which == 0 ? a.k[0] : which == 1 ? a.k[1] : a.k[2]) : 0ull;
    }
    if (i < a.nb_p) a.blk_p[i] = 0;
    if (i < a.nb_g) a.blk_g[i] = 0;
}

// kept weights go to the dense scratch, pruned positions leave the mask (psel null: nothing is pruned)
// (zero_pruned: Wd is the layer's dense copy, whose inactive positions must read 0)
struct PruneArgs {
    const float* vals;
    const int* flat;
    const uint8_t* psel;
    int64_t nnz;
    float* Wd;
    uint8_t* mask;
    int zero_pruned;
};
__device__ inline void apply_prune(const PruneArgs& a, int64_t k) {
    if (k >= a.nnz) return;
    const int f = a.flat[k];
    if (a.psel && a.psel[k]) {
        a.mask[f] = 0;
        if (a.zero_pruned) a.Wd[f] = 0.f;
    } else {
        a.Wd[f] = a.vals[k];
    }
}

// The end of the random selection (block 0, if there is one) and the pruning beside it: the one writes positions that were
// inactive before the update, the other those that were active.
struct EndArgs {
    RandArgs rand;
    PruneArgs prune;
    int has_rand;
};
template <int CAP>
__global__ __launch_bounds__(SEL_NT) void k_update_end(const Batch<EndArgs, CAP> batch) {
    __shared__ FinishShared sh;
    if (batch.surplus()) return;
    const EndArgs a = batch.entry();
    const int b = (int)blockIdx.x - a.has_rand;
    if (b < 0) rand_finish(a.rand, sh);
    else apply_prune(a.prune, (int64_t)b * SEL_NT + threadIdx.x);
}

// Blocks of a digit pass over n keys: 16 keys per thread, one round up to 4 million of them, and together no more than what the
// chip holds at a time (two of 64 KB on a CU): a block costs the clearing and the sum of its histogram whatever it reads, and the
// chains of other layers run beside this one (four layers of a GPT-2-small block, a stream each, with 4 keys per thread
// and twice the blocks: 216 us, like this 196; 16 instead of 8 keys per thread in the flag and list passes 192).
// `total`: keys of all selections of the launch.
static unsigned digit_blocks(int64_t n, int64_t total) {
    const int64_t share = std::max<int64_t>(1, 512 * n / std::max<int64_t>(total, 1));
    return (unsigned)std::min<int64_t>(std::min<int64_t>(cdiv(n, SEL_NT * 16), 256), share);
}
// Indices of a block of the flag pass: whole rounds of 16 per thread, and no more than 256 blocks (each adds 1024 bins to the
// random selection's histogram)
static int64_t flag_range(int64_t n) { return 16 * SEL_NT * cdiv(cdiv(n, 16 * SEL_NT), 256); }

// The updates of several layers, one launch per link of the chain for all of them (up to 7 links and those of the
// rebuild).
int mask_update_device(const UpdateItem* items, int n, hipStream_t s) {
    Batch<InitArgs> init;
    Batch<SelectArgs> digit;
    Batch<FlagArgs> flag;
    Batch<RandArgs> compact;
    Batch<EndArgs> end;
    BuildItem views[BATCH_MAX], canonical[BATCH_MAX];
    mst_layer* runs[BATCH_MAX];
    int n_views = 0, n_canonical = 0, n_runs = 0, rc;
    bool recording;
    if ((rc = stream_recording(s, &recording)) != MST_OK) return rc;
    int64_t keys = 0;                                 // of all selections
    for (int x = 0; x < n; ++x)
        keys += (items[x].st.n_prune > 0 ? items[x].L->nnz : 0) + (items[x].st.n_grad > 0 ? items[x].L->N : 0);
    for (int x = 0; x < n; ++x) {
        mst_layer* L = items[x].L;
        const mst_update_stats& st = items[x].st;
        const Workspace& ws = items[x].ws;
        const int64_t N = L->N, nnz = L->nnz;
        // Where the new dense weights are formed.  A layer that stays on the dense contractions after
        // this update gets them straight into its dense copy (zero at every inactive position: kept
        // weights are rewritten, pruned and grown positions written 0) and only vals / flat / rowptr
        // are rebuilt; otherwise they go to the workspace and both index views are rebuilt from them.
        L->nnz = st.nnz_after;
        L->choice.store(0, std::memory_order_relaxed);
        const bool with_views = views_wanted(L);
        L->nnz = nnz;
        L->choice.store(0, std::memory_order_relaxed);
        float* const Wnew = with_views ? ws.Wd : L->Wd;
        if (with_views) views[n_views++] = BuildItem{L, ws.Wd, ws, false};
        else canonical[n_canonical++] = BuildItem{L, L->Wd, ws, false};
        if (!with_views && (!L->Wd_zeros || L->Wd_pending) && (rc = fill_u32(L->Wd, 0u, N, s)) != MST_OK) return rc;
        uint64_t* const st0 = ws.sel_state;
        // During the selections the mask still means "active before this update" for every position
        // a later selection looks at: positions grown by gradient become active at once (random
        // growth must skip them anyway), pruned positions leave the mask only at the very end.
        const bool do_p = st.n_prune > 0 && nnz > 0, do_g = st.n_grad > 0, do_r = st.n_rand > 0;
        int* const blk_g = reinterpret_cast<int*>(ws.blk);
        int* const blk_p = blk_g + cdiv(N, SELECT_BLOCK) + 1;
        const int64_t per_p = flag_range(std::max<int64_t>(nnz, 1)), per_g = flag_range(N);
        const int nb_p = do_p ? (int)cdiv(nnz, per_p) : 0, nb_g = do_g || do_r ? (int)cdiv(N, per_g) : 0;
        init.add(InitArgs{st0, {(uint64_t)st.n_prune, (uint64_t)st.n_grad, (uint64_t)st.n_rand}, blk_p, blk_g, nb_p, nb_g},
                 cdiv((int64_t)SEL_STATES * SEL_STATE_WORDS, 256));
        const PruneKeys pk{L->vals, L->flat, items[x].G, L->prune_lambda};
        const GradKeys gk{items[x].G, L->mask};
        uint64_t *const st_p = st0, *const st_g = st0 + SEL_STATE_WORDS, *const st_r = st0 + 2 * SEL_STATE_WORDS;
        if (do_p || do_g) {
            const int dig0 = do_p ? (int)digit_blocks(nnz, keys) : 0, dig1 = do_g ? (int)digit_blocks(N, keys) : 0;
            digit.add(SelectArgs{pk, gk, nnz, N, st_p, st_g, dig0, dig1}, dig0 + dig1);
        }
        if (nb_p + nb_g > 0)
            flag.add(FlagArgs{pk, gk, nnz, N, per_p, per_g, st_p, do_g ? st_g : nullptr, do_r ? st_r : nullptr, blk_p, blk_g,
                              FlagSink{ws.psel, 1, 1, nullptr, nullptr}, FlagSink{ws.sel, 2, 1, L->mask, Wnew}, items[x].seed, nb_p},
                     nb_p + nb_g);
        // selected positions become active (weight 0) where they are decided: below the picked bin in the
        // list pass, inside it by the finishing block; no separate flag pass
        const RandArgs rand{RandKeys{L->mask, ws.sel, items[x].seed}, N, st_r,
                            reinterpret_cast<RandItem*>(ws.gemm),           // 2 N items fit: more than any candidate count
                            FlagSink{ws.sel, 3, 0, L->mask, Wnew}};
        if (do_r) compact.add(rand, cdiv(N, COMPACT_PER_BLOCK));
        if (do_r || nnz > 0)
            end.add(EndArgs{rand, PruneArgs{L->vals, L->flat, do_p ? ws.psel : nullptr, nnz, Wnew, L->mask, with_views ? 0 : 1}, do_r ? 1 : 0},
                    (do_r ? 1 : 0) + cdiv(nnz, SEL_NT));
    }
    launch_batch(init, [&](const auto& b) { k_update_init<<<b.grid(), 256, 0, s>>>(b); });
    MST_LAUNCH_CHECK();
    if (digit.n > 0) {
        launch_batch(digit, [&](const auto& b) { k_select_digit<1><<<b.grid(), SEL_NT, 0, s>>>(b); });
        MST_LAUNCH_CHECK();
        launch_batch(digit, [&](const auto& b) { k_select_digit<2><<<b.grid(), SEL_NT, 0, s>>>(b); });
        MST_LAUNCH_CHECK();
        launch_batch(digit, [&](const auto& b) { k_select_digit<3><<<b.grid(), SEL_NT, 0, s>>>(b); });
        MST_LAUNCH_CHECK();
    }
    if (flag.n > 0) {
        launch_batch(flag, [&](const auto& b) { k_select_flag<<<b.grid(), SEL_NT, 0, s>>>(b); });
        MST_LAUNCH_CHECK();
    }
    if (compact.n > 0) {
        launch_batch(compact, [&](const auto& b) { k_rand_compact<<<b.grid(), SEL_NT, 0, s>>>(b); });
        MST_LAUNCH_CHECK();
    }
    if (end.n > 0) {
        launch_batch(end, [&](const auto& b) { k_update_end<<<b.grid(), SEL_NT, 0, s>>>(b); });
        MST_LAUNCH_CHECK();
    }
    for (int x = 0; x < n; ++x) {
        items[x].L->nnz = items[x].st.nnz_after;
        items[x].L->choice.store(0, std::memory_order_relaxed);
        if (items[x].L->pairs_calls >= PAIRS_CALLS) items[x].L->pairs_unknown();
        items[x].L->runs_valid = false;
        if (items[x].L->runs_kept(recording)) runs[n_runs++] = items[x].L;
        else items[x].L->runs_missed |= recording;
    }
    if (n_views > 0 && (rc = build_views(views, n_views, s)) != MST_OK) return rc;
    for (int x = 0; x < n_canonical; ++x) {
        mst_layer* L = canonical[x].L;
        L->Wd_valid = L->Wd_zeros = true;
        L->Wd_pending = false;
        L->planes_valid = L->planes_kept();
        if (L->planes_valid && (rc = make_planes(L, s)) != MST_OK) return rc;
        L->pairs_valid = pairs_kept(L) && (L->pairs_recorded || pairs_wanted(L, false));
        L->pairs_matched = false;
        if (L->pairs_valid && (rc = make_pairs(L, s)) != MST_OK) return rc;
        L->pairs_matched = L->pairs_valid;
    }
    if (n_canonical > 0 && (rc = build_canonical(canonical, n_canonical, recording, s)) != MST_OK) return rc;
    if (n_runs == 0) return MST_OK;
    rc = make_runs(runs, n_runs, s);
    for (int x = 0; x < n_runs; ++x) {
        runs[x]->runs_valid = rc == MST_OK;
        runs[x]->runs_unread += runs[x]->runs_unread >= 0 && runs[x]->runs_unread < mst_layer::RUNS_UNREAD;
    }
    return rc;
}

}  // namespace mst
