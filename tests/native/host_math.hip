// Host build of the arithmetic that the kernels share with the host (csrc/internal.h), for
// tests/test_host_math.py.
#include "internal.h"

extern "C" {

// xs, d and mine of the lane at x in a row of X voxels
void row_lane(int wide, int32_t x, int32_t X, int32_t out[3]) {
    const fc::RowLane r = wide ? fc::row_lane<true>(x, X) : fc::row_lane<false>(x, X);
    out[0] = r.xs;
    out[1] = r.d;
    out[2] = (int32_t)r.mine;
}

}
