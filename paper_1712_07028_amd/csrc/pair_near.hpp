// The FP32 test that goes before the FP64 one when every pair of a small table is tested: pure
// functions, compiled for the device (candidate pairs) and for the host (the check that no
// pair within reach is lost).
#pragma once

#include <math.h>

namespace fsl {

// Boxes whose axes the FP32 test covers.  A coordinate below 2^16 rounds by at most 2^-9, a distance
// along an axis by twice that and a unit more, far below the half cell of slack; at 2^22 the
// slack is used up (a coordinate rounds by a quarter), at 2^24 pairs within reach are lost.
// Longer boxes take the grid, which compares in FP64.
constexpr int PAIRS_AXIS = 1 << 16;
__host__ __device__ inline bool pairs_direct_box(int nx, int ny, int nz) {
    return nx <= PAIRS_AXIS && ny <= PAIRS_AXIS && nz <= PAIRS_AXIS;
}

// distance along an axis, to the nearest image along a periodic one (centres in [0, n))
__host__ __device__ inline float axis_apart(float a, float b, int n, int per) {
    const float d = fabsf(a - b);
    return per ? fminf(d, (float)n - d) : d;
}
// the second sphere's share of the FP32 reach
__host__ __device__ inline float reach_of(double R, double reach) { return (float)(R + reach) + 0.5f; }
// false only for spheres whose surfaces are farther apart than the reach
__host__ __device__ inline bool pair_near(float d0, float d1, float d2, float r) {
    return d0 * d0 + d1 * d1 + d2 * d2 < r * r;
}

}  // namespace fsl
