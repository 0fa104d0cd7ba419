// Force of the fluid on each no-slip face of the box over a step, the plate force of
// the sheared suspension (Sec. 3.1: mu_s = F_x / (A gamma)).  Every half-way
// bounce-back link exchanges momentum with its face as a particle link does (Eqs.
// netforce, momentum_transfer): Delta j = c_qbar (f*_qbar(x,t) + f_q(x,t+1)), in
// shifted storage -c_q (h*_qbar + h_q + 2 w_q), where h_q = h*_qbar + 6 w_q rho_t
// (c_q . u_w) (Eq. bbrule) with rho_t the cell's density at t from its own
// populations, as the stream-collide step takes it.  The kernel reads lattice A (the
// state at t) and the cell types at t, so it runs before the stream-collide launch.
#pragma once

#include "k_free_surface.hpp"
#include "k_particles.hpp"

namespace fsl {

// the face layers to walk: layer f is (axis, side); a cell that lies on the layer of
// a lower axis in the list is left to that layer, so that each cell counts once
struct FaceSet {
    int n;
    int axis[6], side[6];
    long long start[7];  // prefix sums of the layer areas
};

// Block b of nb of face layer f.  The links of a layer's cells lead almost all to the layer's own face: those sum in
// registers, then over the wave, and one lane adds to the block's sums; links of edge cells
// to other faces add by themselves.  (Every link adding to the 18 sums of the block, one
// address for most lanes, took 15 us on the plates of a 114 x 116 suspension.)
template <int ST>
__device__ __forceinline__ void wall_forces(const Geom &G, const Phys &Ph, const Dev &D, const FaceSet &FS, int f, int b,
                                            int nb) {
    using SS = Store<ST>;
    const typename SS::T *A = (const typename SS::T *)D.fA;
    __shared__ double acc[18];
    if (threadIdx.x < 18) acc[threadIdx.x] = 0.0;
    __syncthreads();
    const int nn[3] = {G.nx, G.ny, G.nz};
    {
        const int a = FS.axis[f], side = FS.side[f];
        const int p1 = a == 0 ? 1 : 0, p2 = a == 2 ? 1 : 2;  // the other two axes
        const long long area = FS.start[f + 1] - FS.start[f];
        const float *ua = D.wallu + (a * 2 + side) * 3;
        const float ua0 = ua[0], ua1 = ua[1], ua2 = ua[2];
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        for (long long r = b * 256LL + threadIdx.x; r < area; r += nb * 256LL) {
            int p[3];
            p[a] = side ? nn[a] - 1 : 0;
            p[p1] = (int)(r % nn[p1]);
            p[p2] = (int)(r / nn[p1]);
            bool dup = side && nn[a] == 1;  // one layer is both faces
            for (int k = 0; k < f; ++k) {
                const int ak = FS.axis[k];
                if (ak != a && p[ak] == (FS.side[k] ? nn[ak] - 1 : 0)) dup = true;
            }
            if (dup) continue;
            const int c = p[0] + G.nx * (p[1] + G.ny * p[2]);
            const uint8_t fl = D.flags[c];
            float h[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) h[q] = SS::ld(A + q * G.S + c, Ph.inv);
            if (fl != LIQ && fl != IFC) continue;
            const float rho_t = 1.0f + (float)cell_moments(h).drho;
#pragma unroll
            for (int q = 1; q < Q; ++q) {
                const int s[3] = {p[0] - cx(q), p[1] - cy(q), p[2] - cz(q)};
                int fa = -1;
                bool crossed = false;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (G.per[k] || (s[k] >= 0 && s[k] < nn[k])) continue;
                    crossed = true;
                    if (fa < 0 && !Ph.slip[k]) fa = k;
                }
                if (!crossed || fa < 0) continue;  // no face, or free-slip faces only
                const int sd = (fa == 0 ? s[0] : fa == 1 ? s[1] : s[2]) < 0 ? 0 : 1;
                float u0 = ua0, u1 = ua1, u2 = ua2;
                const bool own = fa == a && sd == side;
                if (!own) {
                    const float *uw = D.wallu + (fa * 2 + sd) * 3;
                    u0 = uw[0];
                    u1 = uw[1];
                    u2 = uw[2];
                }
                const float hb = h[opp(q)];
                const float hq = hb + 6.0f * wq(q) * rho_t * (cx(q) * u0 + cy(q) * u1 + cz(q) * u2);
                const double m = (double)hb + (double)hq + 2.0 * wqd(q);
                if (own) {
                    if (cx(q)) s0 -= cx(q) * m;
                    if (cy(q)) s1 -= cy(q) * m;
                    if (cz(q)) s2 -= cz(q) * m;
                } else {
                    double *dst = acc + 3 * (2 * fa + sd);
                    if (cx(q)) atomicAdd(dst + 0, -cx(q) * m);
                    if (cy(q)) atomicAdd(dst + 1, -cy(q) * m);
                    if (cz(q)) atomicAdd(dst + 2, -cz(q) * m);
                }
            }
        }
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if (lane_id() == 0) {
            double *dst = acc + 3 * (2 * a + side);
            if (s0 != 0.0) atomicAdd(dst + 0, s0);
            if (s1 != 0.0) atomicAdd(dst + 1, s1);
            if (s2 != 0.0) atomicAdd(dst + 2, s2);
        }
    }
    __syncthreads();
    if (threadIdx.x < 18 && acc[threadIdx.x] != 0.0) unsafeAtomicAdd(D.wallF + threadIdx.x, acc[threadIdx.x]);
}

// What a step can do before the lattice update, in one launch: the face forces (nb blocks
// to a layer) and, after those blocks, the candidate pairs of a small table.  Apart they
// took 12.4 and 9.5 us on a 114 x 116 x 180 suspension, 14.5 us together.
template <int ST>
__global__ __launch_bounds__(256) void k_before(Geom G, Phys Ph, Dev D, FaceSet FS, int nb, PairsDirect A) {
    const int b = blockIdx.x, nf = nb * FS.n;
    if (b < nf) wall_forces<ST>(G, Ph, D, FS, b / nb, b % nb, nb);
    else pairs_direct(D, A, b - nf);
}

}  // namespace fsl
