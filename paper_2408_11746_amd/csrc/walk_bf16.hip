// Walk kernels with bfloat16 activations.
#include "walk_launch.h"

namespace mst {

int walk_out_bf16(int q, const WalkSide& sd, const WalkArgs& wa, hipStream_t s) { return launch_out_any<uint16_t>(q, sd, wa, s); }
int walk_both_bf16(int q, const WalkSide& sd, const WalkArgs& wa, int nsplit, hipStream_t s) {
    return launch_both_any<uint16_t>(q, sd, wa, nsplit, s);
}
int walk_dw_bf16(int q, const WalkSide& row, const WalkSide& col, const WalkArgs& wa, const WalkDrive& drive, hipStream_t s) {
    return launch_dw_any<uint16_t>(q, row, col, wa, drive, s);
}

}  // namespace mst
