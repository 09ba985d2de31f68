// Products of which only the active outputs are wanted: the weight gradient on the dense matrix cores.
#pragma once

#include <stdint.h>
#include <hip/hip_runtime.h>

namespace mst {

// Where they go: words[row * per_row + col / 32] = the inactive columns among 32 of a row and the canonical index of the first of them
struct ActiveRuns {
    const uint2* words;
    int per_row;
    uint32_t bytes;            // of an output of the active positions alone
};

__device__ inline __amdgpu_buffer_rsrc_t active_buffer(float* out, const ActiveRuns& runs) {
    return __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)runs.bytes, 0x00020000);
}
// column lane % 32 of word w (below: the bits under it); an inactive one is stored past the end, that is nowhere
__device__ __forceinline__ void store_active(__amdgpu_buffer_rsrc_t out, uint2 w, int lane, uint32_t below, float v) {
    const uint32_t at = w.y + (uint32_t)__popc(below & ~w.x);                     // (w.x: the inactive ones)
    const uint32_t off = at << 2 | (uint32_t)((int)(w.x << (31 - (lane & 31))) >> 31);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), out, (int)off, 0, 0);
}

}  // namespace mst
