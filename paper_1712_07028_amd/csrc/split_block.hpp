// The 3x3x3-block part of the local bubble-splitting test (bubble model, end of
// Sec. 2.2: a bubble is a connected region of gas, D3Q19 neighbours connected).
// Pure functions of bit sets, compiled for the device (the splitting test) and for
// the host (the exactness check against a global labelling).
#pragma once

#include "fsl_device.hpp"

namespace fsl {

// block cells as a 27-bit set, bit (dx + 1) + 3 (dy + 1) + 9 (dz + 1); the centre is 13
constexpr unsigned blk_layer(int axis, int v) {  // the cells with coordinate v (0..2) along an axis
    unsigned m = 0u;
    for (int b = 0; b < 27; ++b)
        if ((axis == 0 ? b % 3 : axis == 1 ? (b / 3) % 3 : b / 9) == v) m |= 1u << b;
    return m;
}
// cells of the block one step along an axis away from a cell of m
template <int A>
__host__ __device__ __forceinline__ unsigned blk_axis(unsigned m) {
    constexpr int sh = A == 0 ? 1 : A == 1 ? 3 : 9;
    constexpr unsigned lo = blk_layer(A, 0), hi = blk_layer(A, 2);
    return ((m & ~hi) << sh) | ((m & ~lo) >> sh);
}
// cells of the block one D3Q19 step away from a cell of m: one step along an axis, or one
// along each of two
__host__ __device__ __forceinline__ unsigned blk_step(unsigned m) {
    const unsigned x = blk_axis<0>(m), y = blk_axis<1>(m), z = blk_axis<2>(m);
    return x | y | z | blk_axis<1>(x) | blk_axis<2>(x) | blk_axis<2>(y);
}

// The centre cell left the gas; gas: the block's cells that are still gas of its
// root bubble, rem: those that also left it in this step.  True when the root's gas
// stays connected for certain: (1) the gas neighbours of the centre are connected
// within the block, and (2) each neighbour that also left touches that connected
// set.  A gas path through a run of removed cells can then be rerouted through the
// block gas of each cell of the run.
__host__ __device__ __forceinline__ bool split_block_ok(unsigned gas, unsigned rem) {
    const unsigned n18 = blk_step(1u << 13);
    const unsigned s = gas & n18;
    if (!s) return true;
    unsigned comp = s & (~s + 1u);
    for (int it = 0; it < 27; ++it) {
        const unsigned grown = comp | (blk_step(comp) & gas);
        if (grown == comp) break;
        comp = grown;
    }
    if (s & ~comp) return false;
    for (unsigned rm = rem & n18; rm; rm &= rm - 1u)
        if (!(blk_step(rm & (~rm + 1u)) & comp)) return false;
    return true;
}

}  // namespace fsl
