// fp32 operands on the bf16 matrix cores: the hi / lo split and the LDS layout of bf16 operand
// tiles that the dense GEMM kernels and the heavy-row product share.
#pragma once

#include <stdint.h>
#include <hip/hip_runtime.h>

namespace mst {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// An LDS row is 64 k of bf16 = 128 bytes = eight 16-byte units; unit u of row m is kept at
// position u ^ ((m >> 1 ^ m >> 4) & 7): the MFMA operand reads of 16 consecutive rows then cover all
// banks once, and so do the stores of eight lanes to rows two, four or eight apart (a store takes 128 bytes a clock, a
// read 256).
__device__ inline uint32_t bf_unit(int m, int u) { return (uint32_t)(m * 128 + ((u ^ ((m >> 1 ^ m >> 4) & 7)) << 4)); }

__device__ inline uint32_t cvt_pk_bf16(float a, float b) {       // {bf16(a), bf16(b)}, round to nearest even
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// x = hi + lo + (at most 2^-16 |x|): hi = bf16(x), lo = bf16(x - hi); x - hi is exact in fp32
__device__ inline void split_pair(float x0, float x1, uint32_t& hi, uint32_t& lo) {
    hi = cvt_pk_bf16(x0, x1);
    lo = cvt_pk_bf16(x0 - __uint_as_float(hi << 16), x1 - __uint_as_float(hi & 0xFFFF0000u));
}

// ---- loads that go straight to LDS
// 16 bytes per lane from base + voff to LDS, lane l to lds + 16 l; base and lds uniform.  The load has no register to
// return to; whoever reads the LDS waits for it (vmcnt) and for the other wavefronts (barrier) first.
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory");
}
template <int LATER>
__device__ __forceinline__ void wait_loads() {        // until all but the LATER youngest loads of this wavefront have arrived
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LATER) : "memory");
}
// this wavefront's LDS accesses are done, and everyone's
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Tile number -> tile coordinates for the 256-row kernels.  Tiles are numbered in bands of four tile
// rows, column by column inside a band: the 32 tiles an XCD works on at a time then span about
// 4 rows x 8 columns instead of 2 x 20, so its L2 is filled with 12 operand panels instead of 22.
constexpr int TILE_BAND = 4;
__device__ inline void tile_coords(int tile_id, int gm, int gn, int& mi, int& ni) {
    const int band = tile_id / (TILE_BAND * gn), rem = tile_id - band * TILE_BAND * gn;
    const int hgt = min(TILE_BAND, gm - band * TILE_BAND);
    ni = rem / hgt;
    mi = band * TILE_BAND + rem - ni * hgt;
}

}  // namespace mst
