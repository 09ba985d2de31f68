// From a position of a layer to its place among the active ones: outputs of the weight gradient on the dense matrix cores, weights that
// are packed.
#pragma once

#include <stdint.h>
#include <hip/hip_runtime.h>

namespace mst {

// words[row * per_row + col / 32] = the inactive columns among 32 of a row and the canonical index of the first of them
struct ActiveRuns {
    const uint2* words;
    int per_row;
    uint32_t bytes;            // of an output of the active positions alone
};

__device__ inline __amdgpu_buffer_rsrc_t active_buffer(float* out, const ActiveRuns& runs) {
    return __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)runs.bytes, 0x00020000);
}
// offset in bytes of column c of word w (below: the bits under it), far past the end where that is inactive
__device__ __forceinline__ uint32_t active_offset(uint2 w, uint32_t c, uint32_t below) {
    const uint32_t at = w.y + (uint32_t)__popc(below & ~w.x);                     // (w.x: the inactive ones)
    return at << 2 | (uint32_t)((int)(w.x << (31u - c)) >> 31);
}
// column lane % 32 of word w (below: the bits under it); an inactive one is stored past the end, that is nowhere
__device__ __forceinline__ void store_active(__amdgpu_buffer_rsrc_t out, uint2 w, int lane, uint32_t below, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), out, (int)active_offset(w, (uint32_t)lane & 31u, below), 0, 0);
}

}  // namespace mst
