// k_particles.hpp -- rigid spheres (Sec. 2.3): force/torque hand-over from the
// per-particle FP64 accumulators of the stream-collide kernel, lubrication
// correction (Eq. lubrication) on a candidate-pair list from a uniform grid,
// substep time integration, and the obstacle-coverage update (nodes inside a
// sphere are obstacle nodes; covered / uncovered cells keep the mass ledger).
#pragma once

#include "cov_column.hpp"
#include "k_free_surface.hpp"
#include "pair_near.hpp"

namespace fsl {

constexpr int CLAIM_NONE = 0x7fffffff;

// per particle: F, T of the step (reported), mass paid by moving bounce-back to the
// ledger (block reduction then one atomic per block), accumulators cleared.  A particle's
// copies lie in 64 consecutive values: a wave reads and clears them in one access each (a
// thread per particle touched 64 lines an access), four particles at a time, and sums
// component (lane & 7) over the copies in order.
__global__ __launch_bounds__(256) void k_part_forces(Dev D, int integrate) {
    static_assert(ACC_COPIES * ACC_STRIDE == 64, "one value per lane");
    __shared__ double red[4];
    constexpr int U = 4;
    const int lane = (int)(threadIdx.x & 63u), wv = (int)(threadIdx.x >> 6);
    double dm = 0.0;
    for (int P0 = (blockIdx.x * 4 + wv) * U; P0 < D.np; P0 += gridDim.x * 4 * U) {
        double v[U], o[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int P = min(P0 + j, D.np - 1);
            v[j] = D.pacc[acc_at(P, 0) + lane];
            o[j] = D.pFT[(long long)P * 6 + min(lane, 5)];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int P = P0 + j;
            double s = __shfl(v[j], lane & 7);
#pragma unroll
            for (int k = 1; k < ACC_COPIES; ++k) s += __shfl(v[j], (lane & 7) + k * ACC_STRIDE);
            if (P >= D.np) continue;
            D.pacc[acc_at(P, 0) + lane] = 0.0;
            if (lane < 6) {
                D.pFTp[(long long)P * 6 + lane] = o[j];
                D.pFT[(long long)P * 6 + lane] = s;
            }
            if (lane == 6) dm += s;
            if (integrate && lane < 3) {  // the launch-per-substep update follows
                double *t = D.ptab + (long long)P * P_STRIDE;
                t[P_XOLD + lane] = t[P_X + lane];
                D.pFl[(long long)P * 3 + lane] = 0.0;
            }
        }
    }
    if (lane == 6) red[wv] = dm;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double s = (red[0] + red[1]) + (red[2] + red[3]);
        if (s != 0.0) unsafeAtomicAdd(D.ledger, -s);
    }
}

// node box [lo, hi] of a sphere: clipped to the box along walled axes, unwrapped along
// periodic ones (node_at wraps the indices; the box never holds a node twice, see
// sphere_supported); false when nothing is left (a sphere outside the box or not
// finite, which the next synchronising call reports)
__device__ __forceinline__ bool sphere_box(const Geom &G, const double *x, double R, int lo[3], int hi[3]) {
    const int n[3] = {G.nx, G.ny, G.nz};
    bool ok = true;
    for (int a = 0; a < 3; ++a) {
        const double l = floor(x[a] - R), h = ceil(x[a] + R);
        const bool in = G.per[a] ? (l >= -2.0 * n[a] && h <= 3.0 * n[a]) : (l <= n[a] - 1.0 && h >= 0.0);
        if (!in) {  // also NaN
            lo[a] = 0;
            hi[a] = -1;
            ok = false;
            continue;
        }
        if (G.per[a]) {
            lo[a] = (int)l;
            hi[a] = (int)h;
        } else {
            lo[a] = l < 0.0 ? 0 : (int)l;
            hi[a] = h > n[a] - 1.0 ? n[a] - 1 : (int)h;
        }
    }
    return ok;
}

// cell index of node coordinates that may lie beyond periodic faces (in range along
// walled axes)
__device__ __forceinline__ int node_at(const Geom &G, int i, int j, int k) {
    if (G.per[0]) i = ((i % G.nx) + G.nx) % G.nx;
    if (G.per[1]) j = ((j % G.ny) + G.ny) % G.ny;
    if (G.per[2]) k = ((k % G.nz) + G.nz) % G.nz;
    return i + G.nx * (j + G.ny * k);
}

// position of sphere t's centre as the image nearest to the point p (per axis)
__device__ __forceinline__ void image_near(const Geom &G, const double *t, const double *p, double out[3]) {
    const int n[3] = {G.nx, G.ny, G.nz};
#pragma unroll
    for (int a = 0; a < 3; ++a) out[a] = p[a] + min_img(t[a] - p[a], n[a], G.per[a]);
}

__device__ __forceinline__ bool inside(double i, double j, double k, const double *x, double R) {
    double d0 = i - x[0], d1 = j - x[1], d2 = k - x[2];
    return __dadd_rn(__dadd_rn(__dmul_rn(d0, d0), __dmul_rn(d1, d1)), __dmul_rn(d2, d2)) <= __dmul_rn(R, R);
}

// FP32 mirror used by the stream-collide kernel: integer anchor floor(x_P), the
// fraction x_P - anchor, velocity and angular velocity
__device__ __forceinline__ void mirror_store(const Dev &D, int P, const double *x, const double *u, const double *w) {
    float4 *m = D.pmir + 4LL * P;
    const double a0 = floor(x[0]), a1 = floor(x[1]), a2 = floor(x[2]);
    // PMir order: anchor, fraction, u, omega
    m[0] = make_float4((float)a0, (float)a1, (float)a2, (float)(x[0] - a0));
    m[1] = make_float4((float)(x[1] - a1), (float)(x[2] - a2), (float)u[0], (float)u[1]);
    m[2] = make_float4((float)u[2], (float)w[0], (float)w[1], (float)w[2]);
    m[3] = make_float4(0.f, 0.f, 0.f, 0.f);
}
__global__ void k_part_mirror(Dev D) {
    GRID_STRIDE(P, D.np) {
        const double *t = D.ptab + (long long)P * P_STRIDE;
        mirror_store(D, P, t + P_X, t + P_U, t + P_W);
    }
}

// ---- candidate pairs for lubrication: uniform grid ---------------------------------
struct PGrid {
    int g[3];
    double cs[3];
    double reach;  // pair candidate distance between surfaces
    int n[3], per[3];  // the box, for nearest images across periodic faces
};

__device__ __forceinline__ int pgrid_cell(const PGrid &PG, const double *x, int a) {
    int v = (int)floor(x[a] / PG.cs[a]);
    return v < 0 ? 0 : (v >= PG.g[a] ? PG.g[a] - 1 : v);
}

__global__ void k_grid_zero(Dev D, int ncell) { GRID_STRIDE(i, ncell) D.gridCount[i] = 0; }

__global__ void k_grid_count(Dev D, PGrid PG) {
    GRID_STRIDE(P, D.np) {
        const double *x = D.ptab + (long long)P * P_STRIDE;
        int cell = pgrid_cell(PG, x, 0) + PG.g[0] * (pgrid_cell(PG, x, 1) + PG.g[1] * pgrid_cell(PG, x, 2));
        atomicAdd(D.gridCount + cell, 1);
    }
}

// exclusive scan of the grid counts by one block; gridCount becomes the fill cursor
// exclusive prefix sum of the per-cell counts into gridStart (and the fill cursors
// in gridCount), over many blocks: block sums, a scan of the block sums (at most
// 1,024), then each block scans its own range from its offset
__global__ __launch_bounds__(256) void k_gscan_sum(Dev D, int ncell, int chunk, int *bsum) {
    __shared__ int red[256];
    const int lo = blockIdx.x * chunk, hi = min(ncell, lo + chunk);
    int s = 0;
    for (int i = lo + (int)threadIdx.x; i < hi; i += 256) s += D.gridCount[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}
__global__ __launch_bounds__(1024) void k_gscan_top(Dev D, int ncell, int nb, int *bsum) {
    __shared__ int v[1024];
    const int t = threadIdx.x;
    const int x = t < nb ? bsum[t] : 0;
    v[t] = x;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int y = t >= o ? v[t - o] : 0;
        __syncthreads();
        v[t] += y;
        __syncthreads();
    }
    if (t < nb) bsum[t] = v[t] - x;
    if (t == 1023) D.gridStart[ncell] = v[t];
}
__global__ __launch_bounds__(256) void k_gscan_apply(Dev D, int ncell, int chunk, const int *bsum) {
    __shared__ int v[256];
    const int lo = blockIdx.x * chunk, hi = min(ncell, lo + chunk);
    const int t = threadIdx.x;
    int carry = bsum[blockIdx.x];
    for (int base = lo; base < hi; base += 256) {
        const int i = base + t;
        const int x = i < hi ? D.gridCount[i] : 0;
        v[t] = x;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            const int y = t >= o ? v[t - o] : 0;
            __syncthreads();
            v[t] += y;
            __syncthreads();
        }
        if (i < hi) {
            const int st = carry + v[t] - x;
            D.gridStart[i] = st;
            D.gridCount[i] = st;
        }
        carry += v[255];
        __syncthreads();
    }
}

__global__ void k_grid_fill(Dev D, PGrid PG) {
    GRID_STRIDE(P, D.np) {
        const double *x = D.ptab + (long long)P * P_STRIDE;
        int cell = pgrid_cell(PG, x, 0) + PG.g[0] * (pgrid_cell(PG, x, 1) + PG.g[1] * pgrid_cell(PG, x, 2));
        int s = atomicAdd(D.gridCount + cell, 1);
        D.gridIdx[s] = P;
    }
}

// append the pair (a, b) of every active lane with pred to a list of pairs: one
// atomic per wave (the ballot sees the active lanes only, so divergent callers are fine)
__device__ __forceinline__ void wave_push2(bool pred, int a, int b, int *list, int *counter, int cap,
                                           unsigned *err) {
    const unsigned long long mask = __ballot(pred);
    if (!mask) return;
    const int leader = __ffsll((long long)mask) - 1;
    int base = 0;
    if ((int)lane_id() == leader) base = atomicAdd(counter, __popcll(mask));
    base = __shfl(base, leader);
    if (pred) {
        const int slot = base + __popcll(mask & ((1ull << lane_id()) - 1ull));
        if (slot < cap) {
            list[2 * slot] = a;
            list[2 * slot + 1] = b;
        } else {
            atomicOr(err, ERR_CAP);
        }
    }
}

// one thread per particle and neighbouring grid cell (27 per particle), so that the
// dependent loads of the cell lists overlap across many threads.  Pairs are sparse
// (about one per wave), so they are gathered per block in LDS and appended with one
// atomic per block: one atomic per pair on the same counter serialises.
constexpr int PAIR_BUF = 1024;
struct PairLds {
    int2 buf[PAIR_BUF];
    int cnt, base;
};

// the pair (P, Qp) to the block's buffer when the surfaces are closer than the reach
__device__ __forceinline__ void pair_test(const Dev &D, const PGrid &PG, PairLds &L, int P, const double *x, int Qp,
                                          const double *y, int pcap) {
    const double d0 = min_img(y[0] - x[0], PG.n[0], PG.per[0]), d1 = min_img(y[1] - x[1], PG.n[1], PG.per[1]),
                 d2 = min_img(y[2] - x[2], PG.n[2], PG.per[2]);
    const double gap = sqrt(d0 * d0 + d1 * d1 + d2 * d2) - x[P_R] - y[P_R];
    if (gap >= PG.reach) return;
    const int k = atomicAdd(&L.cnt, 1);
    if (k < PAIR_BUF) {
        L.buf[k] = make_int2(P, Qp);
    } else {  // the block's buffer is full: straight to the list
        const int g = atomicAdd(D.counters + C_NPAIRS, 1);
        if (g < pcap) D.pairs[g] = make_int2(P, Qp);
        else atomicOr(D.err, ERR_CAP);
    }
}
// the block's pairs to the list; every thread of the block
__device__ __forceinline__ void pairs_flush(const Dev &D, PairLds &L, int pcap) {
    __syncthreads();
    const int n = min(L.cnt, PAIR_BUF);
    if (threadIdx.x == 0) L.base = n ? atomicAdd(D.counters + C_NPAIRS, n) : 0;
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        if (L.base + k < pcap) D.pairs[L.base + k] = L.buf[k];
        else atomicOr(D.err, ERR_CAP);
    }
}

__global__ __launch_bounds__(256) void k_pairs(Dev D, PGrid PG, int pcap) {
    __shared__ PairLds L;
    if (threadIdx.x == 0) L.cnt = 0;
    __syncthreads();
    const int total = D.np * 27;
    // whole blocks take the same rounds, so every thread reaches the barriers below
    for (int r = blockIdx.x * blockDim.x; r < total; r += gridDim.x * blockDim.x) {
        const int idx = r + threadIdx.x;
        if (idx >= total) continue;
        const int P = idx / 27, d = idx - 27 * P;
        const double *x = D.ptab + (long long)P * P_STRIDE;
        const int off[3] = {d % 3 - 1, (d / 3) % 3 - 1, d / 9 - 1};
        int cc[3];
        bool skip = false;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            int v = pgrid_cell(PG, x, k) + off[k];
            if (PG.per[k]) {
                // a periodic axis of one or two grid cells holds each neighbour once
                if ((PG.g[k] == 1 && off[k] != 0) || (PG.g[k] == 2 && off[k] < 0)) skip = true;
                v = v < 0 ? v + PG.g[k] : (v >= PG.g[k] ? v - PG.g[k] : v);
            } else if (v < 0 || v >= PG.g[k]) {
                skip = true;
            }
            cc[k] = v;
        }
        if (skip) continue;
        const int cell = cc[0] + PG.g[0] * (cc[1] + PG.g[1] * cc[2]);
        for (int s = D.gridStart[cell]; s < D.gridStart[cell + 1]; ++s) {
            const int Qp = D.gridIdx[s];
            if (Qp > P) pair_test(D, PG, L, P, x, Qp, D.ptab + (long long)Qp * P_STRIDE, pcap);
        }
    }
    pairs_flush(D, L, pcap);
}

// Small tables (up to PAIRS_DIRECT spheres): every pair tested, in one launch instead of the
// seven that build and walk the grid (4.6 us each whatever the size).  A block takes
// PDIR_P spheres against 256 later ones, one per thread, so that the launch is one
// round of loads deep.  A first test in FP32 on the axes' distances (pair_near.hpp, on boxes
// up to PAIRS_AXIS cells an axis) leaves the distance itself to the near ones.
constexpr int PAIRS_DIRECT = 2048, PDIR_P = 16;
struct PairsDirect {
    PGrid PG;
    int pcap, nx, n;  // blocks: nx along the spheres, n in all
};
inline PairsDirect pairs_direct_of(const PGrid &PG, int pcap, int np) {
    const int nx = (np + PDIR_P - 1) / PDIR_P;
    return {PG, pcap, nx, nx * ((np + 255) / 256)};
}
__device__ __forceinline__ void pairs_direct(const Dev &D, const PairsDirect &A, int b) {
    __shared__ PairLds L;
    __shared__ float c[PDIR_P][4];
    const PGrid &PG = A.PG;
    const int P0 = b % A.nx * PDIR_P, n = min(PDIR_P, D.np - P0);
    const int Q0 = b / A.nx * 256;
    if (Q0 + 255 <= P0) return;  // every sphere of the chunk comes before
    if (threadIdx.x == 0) L.cnt = 0;
    if ((int)threadIdx.x < 4 * n) {
        const int p = threadIdx.x >> 2, k = threadIdx.x & 3;
        c[p][k] = (float)D.ptab[(long long)(P0 + p) * P_STRIDE + (k < 3 ? P_X + k : P_R)];
    }
    const int Qp = Q0 + (int)threadIdx.x;
    const double *y = D.ptab + (long long)min(Qp, D.np - 1) * P_STRIDE;
    const float y0 = (float)y[P_X], y1 = (float)y[P_X + 1], y2 = (float)y[P_X + 2], yr = reach_of(y[P_R], PG.reach);
    __syncthreads();
    for (int p = 0; p < n; ++p) {
        const float d0 = axis_apart(y0, c[p][0], PG.n[0], PG.per[0]), d1 = axis_apart(y1, c[p][1], PG.n[1], PG.per[1]),
                    d2 = axis_apart(y2, c[p][2], PG.n[2], PG.per[2]);
        if (P0 + p < Qp && Qp < D.np && pair_near(d0, d1, d2, c[p][3] + yr))
            pair_test(D, PG, L, P0 + p, D.ptab + (long long)(P0 + p) * P_STRIDE, Qp, y, A.pcap);
    }
    pairs_flush(D, L, A.pcap);
}

// tables of up to INT_BLOCK_MAX spheres take the particle update in one launch (integrate)
constexpr int INT_BLOCK_MAX = 2048;

// Momentum exchange between two particles (Sec. 2.3): a node inside particle P'
// with a link into particle P contributes with equilibrium populations at rho = 1
// and the rigid velocity of P' at the node, Delta j = 2 c_q e^+_q(1, u_P'(x)), to
// P's force and torque.  Such nodes exist only for pairs closer than sqrt(2), all
// of which are in the candidate list; one wave per pair and direction (of P' towards P)
// scans the nodes of P' that lie within one cell of P's bounding box.  A node's links are
// decided by the inside tests first, which coverage takes as well, so that only nodes
// with such a link read cell types and owners.
// nodes of one sphere next to nodes of the other need the centres closer than the radii
// plus the longest link (sqrt 2); margin 1.5
__device__ __forceinline__ bool pair_links(const Geom &G, const Dev &D, int2 pr) {
    const double *ta = D.ptab + (long long)pr.x * P_STRIDE, *tb = D.ptab + (long long)pr.y * P_STRIDE;
    const double d0 = min_img(ta[P_X] - tb[P_X], G.nx, G.per[0]), d1 = min_img(ta[P_X + 1] - tb[P_X + 1], G.ny, G.per[1]),
                 d2 = min_img(ta[P_X + 2] - tb[P_X + 2], G.nz, G.per[2]);
    const double reach = ta[P_R] + tb[P_R] + 1.5;
    return !(d0 * d0 + d1 * d1 + d2 * d2 > reach * reach);
}
__device__ __forceinline__ void solid_pair(const Geom &G, const Dev &D, int Pp, int Po, int copy) {
    const int lane = threadIdx.x & 63;
    const double *tp = D.ptab + (long long)Pp * P_STRIDE, *tq = D.ptab + (long long)Po * P_STRIDE;
    // the other sphere's centre at its image nearest to this one (node coordinates
    // below stay in this sphere's frame; node_at wraps them)
    double to[3];
    image_near(G, tq + P_X, tp + P_X, to);
    const double Ro = tq[P_R], Rp = tp[P_R];
    const double xp[3] = {tp[P_X], tp[P_X + 1], tp[P_X + 2]};
    const double ro = (Ro + 1.5) * (Ro + 1.5);
    int lo[3], hi[3], lo2[3], hi2[3];
    sphere_box(G, xp, Rp, lo, hi);
    sphere_box(G, to, Ro + 1.0, lo2, hi2);
    for (int a = 0; a < 3; ++a) { lo[a] = max(lo[a], lo2[a]); hi[a] = min(hi[a], hi2[a]); }
    if (lo[0] > hi[0] || lo[1] > hi[1] || lo[2] > hi[2]) return;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    bool some = false;
    const int ex = hi[0] - lo[0] + 1, ey = hi[1] - lo[1] + 1, ez = hi[2] - lo[2] + 1;
    const int tot = ex * ey * ez;
    for (int s = lane; s < tot; s += 64) {
        const int i = lo[0] + s % ex, j = lo[1] + (s / ex) % ey, k = lo[2] + s / (ex * ey);
        const double ox = i - to[0], oy = j - to[1], oz = k - to[2];
        // only nodes within a link of the other sphere can have such links
        if (ox * ox + oy * oy + oz * oz > ro || !inside(i, j, k, xp, Rp)) continue;
        unsigned links = 0u;
#pragma unroll
        for (int q = 1; q < Q; ++q) links |= (unsigned)inside(i + cx(q), j + cy(q), k + cz(q), to, Ro) << q;
        if (!links) continue;
        // the node and the far ends of its links in one batch of loads
        const int c = node_at(G, i, j, k);
        int iw, jw, kw;
        cell_xyz(G, c, iw, jw, kw);
        unsigned real = 0u;
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            const int nb = (links >> q) & 1u ? nbr_idx(G, iw, jw, kw, q, 1) : -1;
            const uint8_t f = D.flags[nb < 0 ? c : nb];
            const int o = D.pid[nb < 0 ? c : nb];
            real |= (unsigned)((nb >= 0) & (f == SOL) & (o == Po)) << q;
        }
        if ((D.flags[c] != SOL) | (D.pid[c] != Pp)) continue;
        const double rx = i - xp[0], ry = j - xp[1], rz = k - xp[2];
        const double ur0 = tp[P_U] + (tp[P_W + 1] * rz - tp[P_W + 2] * ry);
        const double ur1 = tp[P_U + 1] + (tp[P_W + 2] * rx - tp[P_W] * rz);
        const double ur2 = tp[P_U + 2] + (tp[P_W] * ry - tp[P_W + 1] * rx);
        const double uu = ur0 * ur0 + ur1 * ur1 + ur2 * ur2;
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            if (!((real >> q) & 1u)) continue;
            const double cu = cx(q) * ur0 + cy(q) * ur1 + cz(q) * ur2;
            const double e2 = 2.0 * wqd(q) * (1.0 + 4.5 * cu * cu - 1.5 * uu);
            const double j0 = cx(q) * e2, j1 = cy(q) * e2, j2 = cz(q) * e2;
            acc[0] += j0;
            acc[1] += j1;
            acc[2] += j2;
            acc[3] += oy * j2 - oz * j1;
            acc[4] += oz * j0 - ox * j2;
            acc[5] += ox * j1 - oy * j0;
            some = true;
        }
    }
    if (!__ballot(some)) return;
    double *dst = D.pacc + acc_at(Po, copy & (ACC_COPIES - 1));
    for (int a = 0; a < 6; ++a) {
        const double v = wave_sum_halves(acc[a]);
        if (lane == 0 && v != 0.0) unsafeAtomicAdd(dst + a, v);
    }
}

// Links into a particle's nodes from beyond the faces of the box (Eq. momentum_transfer).
// Reading: the far end is taken as a node inside another particle is, with
// equilibrium populations at rho = 1, here at the velocity of the first no-slip face
// the link crosses (at rest when it crosses free-slip faces only): Delta j = 2 c_q
// e^+_q(1, u_w), and that no-slip face takes -Delta j.  The constant parts 2 w_q c_q
// of the links into a closed node set cancel exactly; without these links a sphere
// that covers nodes of a face layer would miss them over the cut and be pulled into
// the face by the lattice pressure 1/3.  One wave per particle walks the face-layer
// nodes of its node box; the torque arm runs from the centre to the far end of the
// link.
// the node box of particle P reaches a face layer of a walled axis
__device__ __forceinline__ bool touches_face(const Geom &G, const Dev &D, int P) {
    const double *t = D.ptab + (long long)P * P_STRIDE;
    const int n[3] = {G.nx, G.ny, G.nz};
    int lo[3], hi[3];
    sphere_box(G, t + P_X, t[P_R], lo, hi);
    bool touch = false;
    for (int a = 0; a < 3; ++a)
        if (!G.per[a] && lo[a] <= hi[a] && (lo[a] == 0 || hi[a] == n[a] - 1)) touch = true;
    return touch;
}
__device__ __forceinline__ void face_links(const Geom &G, const Phys &Ph, const Dev &D, int P) {
    const int lane = threadIdx.x & 63;
    const double *t = D.ptab + (long long)P * P_STRIDE;
    const int n[3] = {G.nx, G.ny, G.nz};
    int lo[3], hi[3];
    sphere_box(G, t + P_X, t[P_R], lo, hi);
    double acc[6] = {0, 0, 0, 0, 0, 0};
    float wu[18];
#pragma unroll
    for (int k = 0; k < 18; ++k) wu[k] = D.wallu[k];
    // the face layers of the walled axes that the node box reaches; a node on the
    // layers of two axes is taken with the lower axis
    for (int a = 0; a < 3; ++a) {
        if (G.per[a]) continue;
        const int b = a == 0 ? 1 : 0, d = a == 2 ? 1 : 2;  // the other two axes
        const int eb = hi[b] - lo[b] + 1, ed = hi[d] - lo[d] + 1;
        for (int side = 0; side < 2; ++side) {
            const int layer = side ? n[a] - 1 : 0;
            if (layer < lo[a] || layer > hi[a] || (side && n[a] == 1)) continue;
            for (int s = lane; s < eb * ed; s += 64) {
                int p[3];
                p[a] = layer;
                p[b] = lo[b] + s % eb;
                p[d] = lo[d] + s / eb;
                bool lower = false;
                for (int k = 0; k < a; ++k)
                    if (!G.per[k] && (p[k] == 0 || p[k] == n[k] - 1)) lower = true;
                if (lower || !inside(p[0], p[1], p[2], t + P_X, t[P_R])) continue;
                const int c = node_at(G, p[0], p[1], p[2]);
                if ((D.flags[c] != SOL) | (D.pid[c] != P)) continue;
                for (int q = 1; q < Q; ++q) {
                    const int f[3] = {p[0] - cx(q), p[1] - cy(q), p[2] - cz(q)};  // far end
                    int fa = -1;
                    bool crossed = false;
                    for (int k = 0; k < 3; ++k) {
                        if (G.per[k] || (f[k] >= 0 && f[k] < n[k])) continue;
                        crossed = true;
                        if (fa < 0 && !Ph.slip[k]) fa = k;
                    }
                    if (!crossed) continue;
                    const int sd = fa >= 0 && f[fa] >= 0 ? 1 : 0;
                    double u0 = 0.0, u1 = 0.0, u2 = 0.0;
                    if (fa >= 0) {
                        const int f6 = fa * 2 + sd;
#pragma unroll
                        for (int k = 0; k < 6; ++k)
                            if (k == f6) {
                                u0 = wu[3 * k];
                                u1 = wu[3 * k + 1];
                                u2 = wu[3 * k + 2];
                            }
                    }
                    const double cu = cx(q) * u0 + cy(q) * u1 + cz(q) * u2;
                    const double e2 = 2.0 * wqd(q) * (1.0 + 4.5 * cu * cu - 1.5 * (u0 * u0 + u1 * u1 + u2 * u2));
                    const double j0 = cx(q) * e2, j1 = cy(q) * e2, j2 = cz(q) * e2;
                    const double r0 = f[0] - t[P_X], r1 = f[1] - t[P_X + 1], r2 = f[2] - t[P_X + 2];
                    acc[0] += j0;
                    acc[1] += j1;
                    acc[2] += j2;
                    acc[3] += r1 * j2 - r2 * j1;
                    acc[4] += r2 * j0 - r0 * j2;
                    acc[5] += r0 * j1 - r1 * j0;
                    if (fa >= 0 && D.wallF) {
                        double *w = D.wallF + 3 * (2 * fa + sd);
                        if (j0 != 0.0) unsafeAtomicAdd(w, -j0);
                        if (j1 != 0.0) unsafeAtomicAdd(w + 1, -j1);
                        if (j2 != 0.0) unsafeAtomicAdd(w + 2, -j2);
                    }
                }
            }
        }
    }
    double *dst = D.pacc + acc_at(P, P & (ACC_COPIES - 1));
    for (int a = 0; a < 6; ++a) {
        const double v = wave_sum_halves(acc[a]);
        if (lane == 0 && v != 0.0) unsafeAtomicAdd(dst + a, v);
    }
}

// Both kinds of links that the lattice update does not see, in one launch: the first
// pair_blocks blocks take the pairs, the others the particles for the box faces.  A wave
// takes `chunk` of them at a time (at most 64), a lane testing each, and works those that
// have such links in turn: one on small tables, where the waves are few and a chain of
// several is latency; eight on large ones, where few of the 1e5 spheres touch anything.
struct SolidArgs {
    int pcap, pair_blocks, chunk, n;  // n: blocks in all
};
inline SolidArgs solid_args(int pcap, int np, bool faces) {
    const int chunk = np <= INT_BLOCK_MAX ? 1 : 8;
    // two waves per group of listed pairs (a few per sphere as a rule), a wave per group of
    // spheres
    const int pb = np < 1 ? 0 : std::min(8192, std::max(1, (int)((4LL * np + 2 * chunk - 1) / (2 * chunk))));
    return {pcap, pb, chunk, pb + (faces ? (np + 4 * chunk - 1) / (4 * chunk) : 0)};
}
__device__ __forceinline__ void solid_links(const Geom &G, const Phys &Ph, const Dev &D, const SolidArgs &A, int b) {
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, chunk = A.chunk;
    if (b < A.pair_blocks) {
        const int n = min(D.counters[C_NPAIRS], A.pcap);
        // two waves per group of pairs, one for each direction of their links
        for (int k0 = (b * 2 + (wv >> 1)) * chunk; k0 < n; k0 += A.pair_blocks * 2 * chunk) {
            const int k = k0 + lane;
            const bool has = lane < chunk && k < n;
            const int2 pr = has ? D.pairs[k] : make_int2(0, 0);
            unsigned long long m = __ballot(has && pair_links(G, D, pr));
            while (m) {
                const int l = __ffsll((long long)m) - 1;
                m &= m - 1ull;
                const int a = __builtin_amdgcn_readlane(pr.x, l), b2 = __builtin_amdgcn_readlane(pr.y, l);
                if (wv & 1) solid_pair(G, D, b2, a, k0 + l);
                else solid_pair(G, D, a, b2, k0 + l);
            }
        }
        return;
    }
    const int P0 = ((b - A.pair_blocks) * 4 + wv) * chunk;
    const int P = P0 + lane;
    unsigned long long m = __ballot(lane < chunk && P < D.np && touches_face(G, D, min(P, D.np - 1)));
    while (m) {
        const int l = __ffsll((long long)m) - 1;
        m &= m - 1ull;
        face_links(G, Ph, D, P0 + l);
    }
}
__global__ __launch_bounds__(256) void k_solid_links(Geom G, Phys Ph, Dev D, SolidArgs A) {
    solid_links(G, Ph, D, A, blockIdx.x);
}

// Pair force of one candidate pair (x, u of each sphere; f: force on sphere 1, sphere 2
// takes -f).  Contact (the paper gives no contact model; reading): overlapping spheres
// repel by a linear spring of stiffness kc along the line of centres, -kc (R1 + R2 -
// |d|) d/|d|.  Eq. (lubrication): only for gaps below Delta_c = 2/3, the gap limited
// from below by 0.2 Delta_c.  The partner is taken at its nearest periodic image.
// Returns false when there is no force.  sR: R1 + R2; lub(): lub_factor of the radii, taken
// only where the force acts.
__device__ __forceinline__ double lub_factor(double R1, double R2, double mu) {
    const double rr = R1 * R2, sR = R1 + R2;
    return -6.0 * M_PI * mu * (rr * rr) / (sR * sR);
}
template <typename Lub>
__device__ __forceinline__ bool pair_force(const Geom &G, const double *x1, const double *u1, const double *x2,
                                           const double *u2, double sR, Lub lub, double kc, double f[3]) {
    const double dc = 2.0 / 3.0;
    const double d0 = min_img(x2[0] - x1[0], G.nx, G.per[0]), d1 = min_img(x2[1] - x1[1], G.ny, G.per[1]),
                 d2 = min_img(x2[2] - x1[2], G.nz, G.per[2]);
    const double dd = d0 * d0 + d1 * d1 + d2 * d2;
    f[0] = f[1] = f[2] = 0.0;
    if (dd > (sR + dc) * (sR + dc) * (1.0 + 1e-12)) return false;  // beyond Delta_c: no root taken
    const double dist = sqrt(dd);
    double gap = dist - sR;
    if (kc > 0.0 && dist < sR && dist > 0.0) {
        const double s = -kc * (sR - dist) / dist;
        f[0] = s * d0;
        f[1] = s * d1;
        f[2] = s * d2;
    }
    if (gap < dc && dist > 0.0) {
        if (gap < 0.2 * dc) gap = 0.2 * dc;
        const double n0 = d0 / dist, n1 = d1 / dist, n2 = d2 / dist;
        const double coef = lub() * (1.0 / gap - 1.0 / dc);
        const double vn = n0 * (u1[0] - u2[0]) + n1 * (u1[1] - u2[1]) + n2 * (u1[2] - u2[2]);
        f[0] += coef * vn * n0;
        f[1] += coef * vn * n1;
        f[2] += coef * vn * n2;
    }
    return f[0] != 0.0 || f[1] != 0.0 || f[2] != 0.0;
}

// Force of the no-slip faces (axes with bit a of wmask; faces at -1/2 and n - 1/2) on
// one sphere, added to f.  Eq. (lubrication) and contact are stated for particle
// pairs; reading: a face is a resting sphere of infinite radius touching the face
// plane, so (R1 R2)^2/(R1 + R2)^2 becomes R^2, the pair normal the face normal and
// the gap h - R (h: distance of the centre from the face).  For a gap below Delta_c,
// limited from below by 0.2 Delta_c, that leaves a drag -6 pi mu R^2 (1/gap -
// 1/Delta_c) on the velocity component normal to the face, whichever the side; an
// overlapping sphere (h < R) is pushed off the face by kc (R - h).
__device__ __forceinline__ void face_force(const Geom &G, int wmask, const double *x, const double *u, double R,
                                           double mu, double kc, double f[3]) {
    const double dc = 2.0 / 3.0;
    const int n[3] = {G.nx, G.ny, G.nz};
    for (int a = 0; a < 3; ++a) {
        if (!((wmask >> a) & 1)) continue;
        const double hl = x[a] + 0.5, hh = (n[a] - 0.5) - x[a];
        const double gl = hl - R, gh = hh - R;
        if (!(fmin(gl, gh) < dc)) continue;  // neither face is near
        if (kc > 0.0) {
            if (hl < R) f[a] += kc * (R - hl);
            if (hh < R) f[a] -= kc * (R - hh);
        }
        const double c = 6.0 * M_PI * mu * R * R;
        if (gl < dc) f[a] -= c * (1.0 / fmax(gl, 0.2 * dc) - 1.0 / dc) * u[a];
        if (gh < dc) f[a] -= c * (1.0 / fmax(gh, 0.2 * dc) - 1.0 / dc) * u[a];
    }
}

__global__ void k_lub(Geom G, Dev D, double mu, double kc, int pcap) {
    int n = min(D.counters[C_NPAIRS], pcap);
    GRID_STRIDE(k, n) {
        const int a = D.pairs[k].x, b = D.pairs[k].y;
        const double *p1 = D.ptab + (long long)a * P_STRIDE, *p2 = D.ptab + (long long)b * P_STRIDE;
        double f[3];
        const double R1 = p1[P_R], R2 = p2[P_R];
        if (!pair_force(G, p1 + P_X, p1 + P_U, p2 + P_X, p2 + P_U, R1 + R2, [&] { return lub_factor(R1, R2, mu); }, kc, f))
            continue;
        unsafeAtomicAdd(D.pFl + 3 * a, f[0]);
        unsafeAtomicAdd(D.pFl + 3 * a + 1, f[1]);
        unsafeAtomicAdd(D.pFl + 3 * a + 2, f[2]);
        unsafeAtomicAdd(D.pFl + 3 * b, -f[0]);
        unsafeAtomicAdd(D.pFl + 3 * b + 1, -f[1]);
        unsafeAtomicAdd(D.pFl + 3 * b + 2, -f[2]);
    }
}

// What a sphere keeps through the substeps of one lattice step: F_hyd, T_hyd are the mean of
// this and the previous step's momentum exchange (two-step average that removes the
// period-two oscillation of explicit coupling), or this step's alone after a reset.
// F: F_hyd + m g, du: the change of velocity in a substep without pair and face forces, dw:
// that of the angular velocity.
struct SubstepConst {
    double R, mP, F[3], du[3];
};
__device__ __forceinline__ SubstepConst substep_const(const Dev &D, int P, int have_prev, double dt, const double gg[3]) {
    const double *t = D.ptab + (long long)P * P_STRIDE;
    const double *FTn = D.pFT + (long long)P * 6, *FTp = D.pFTp + (long long)P * 6;
    SubstepConst c;
    c.R = t[P_R];
    c.mP = t[P_RHO] * (4.0 / 3.0) * M_PI * c.R * c.R * c.R;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double Fh = have_prev ? 0.5 * (FTn[d] + FTp[d]) : FTn[d];
        c.F[d] = Fh + c.mP * gg[d];
        c.du[d] = dt * c.F[d] / c.mP;
    }
    return c;
}
// n substeps of the angular velocity
__device__ __forceinline__ void substep_spin(const Dev &D, int P, const SubstepConst &c, int have_prev, double dt, int n,
                                             double w[3]) {
    const double *FTn = D.pFT + (long long)P * 6, *FTp = D.pFTp + (long long)P * 6;
    const double IP = 0.4 * c.mP * c.R * c.R;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double Th = have_prev ? 0.5 * (FTn[3 + d] + FTp[3 + d]) : FTn[3 + d];
        const double dw = dt * Th / IP;
        for (int s = 0; s < n; ++s) w[d] += dw;
    }
}

// one semi-implicit Euler substep of a sphere: velocity from F_hyd + m g + F_pair (fl,
// consumed), then position; the no-slip faces act through face_force at the position and
// velocity the substep starts from; normal velocity reversed when closer than R to a wall
// face and moving towards it; along a periodic axis the centre kept in [0, n)
__device__ __forceinline__ void substep_one(const Geom &G, const SubstepConst &c, double *x, double *u, double *fl,
                                            double dt, double mu, double kc, int wmask) {
    if (wmask) face_force(G, wmask, x, u, c.R, mu, kc, fl);
    const int n[3] = {G.nx, G.ny, G.nz};
    double du[3] = {c.du[0], c.du[1], c.du[2]};
    if (fl[0] != 0.0 || fl[1] != 0.0 || fl[2] != 0.0) {  // the divisions only where a force acts
#pragma unroll
        for (int d = 0; d < 3; ++d)
            if (fl[d] != 0.0) du[d] = dt * (c.F[d] + fl[d]) / c.mP;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        u[d] += du[d];
        x[d] += dt * u[d];
        if (G.per[d]) x[d] = wrap_coord(x[d], n[d]);
        if (!G.per[d]) {
            if (x[d] < c.R - 0.5 && u[d] < 0) u[d] = -u[d];
            if (x[d] > n[d] - 0.5 - c.R && u[d] > 0) u[d] = -u[d];
        }
        fl[d] = 0.0;
    }
}

__global__ void k_substep(Dev D, Geom G, double dt, double g0, double g1, double g2, int have_prev, double mu,
                          double kc, int wmask) {
    GRID_STRIDE(P, D.np) {
        double *t = D.ptab + (long long)P * P_STRIDE;
        const double gg[3] = {g0, g1, g2};
        const SubstepConst c = substep_const(D, P, have_prev, dt, gg);
        substep_spin(D, P, c, have_prev, dt, 1, t + P_W);
        substep_one(G, c, t + P_X, t + P_U, D.pFl + (long long)P * 3, dt, mu, kc, wmask);
        const int n[3] = {G.nx, G.ny, G.nz};
        if (!sphere_supported(t + P_X, t[P_R], n, G.per)) atomicOr(D.err, ERR_PART);
    }
}

// half a cell or more in one step (see k_cov_flag_init)
__device__ __forceinline__ bool moved_far(const Geom &G, const double *x, const double *xo) {
    return fmax(fabs(min_img(x[0] - xo[0], G.nx, G.per[0])),
                fmax(fabs(min_img(x[1] - xo[1], G.ny, G.per[1])), fabs(min_img(x[2] - xo[2], G.nz, G.per[2])))) >= 0.5;
}
// nodes of the two spheres may lie inside both (see k_cov_flag_init); sR: sum of the radii
__device__ __forceinline__ bool may_overlap(const Geom &G, const double *a, const double *b, double sR) {
    const double d0 = min_img(a[0] - b[0], G.nx, G.per[0]), d1 = min_img(a[1] - b[1], G.ny, G.per[1]),
                 d2 = min_img(a[2] - b[2], G.nz, G.per[2]);
    const double r = sR + 1.0;
    return d0 * d0 + d1 * d1 + d2 * d2 < r * r;
}

// The particle update of a step, for tables of up to INT_BLOCK_MAX spheres: the ns substeps,
// the coverage flags and the mirror, in one launch of int_blocks(np) blocks.  Spheres of
// no listed pair are on their own through all substeps: INT_LONE of them to a block, one per
// lane of its first wave, all in registers.  The others are block 0's: centres and velocities
// in LDS, where the pair forces are summed, their constants and those of the first pairs in
// registers, so that a substep reads no global memory; what bounds it is the chain of one
// substep (0.9 us without, 1.7 us with acting pairs).  Every block marks the paired spheres from the
// list for itself.  20 launches, one per half substep, took 110 us for 1,400 spheres
// with 174 pairs, one block for all of them 48 us, this 23 us.  The same arithmetic as k_lub
// and k_substep.
constexpr int INT_LONE = 64;
// tables above this report a centre outside the box after any substep, as with a launch per
// substep; smaller ones after the last
constexpr int INT_WATCH = 512;
inline int int_blocks(int np) { return 1 + (np + INT_LONE - 1) / INT_LONE; }
struct IntArgs {
    int ns;
    double mu, kc;
    int pcap;
    double g[3];
    int have_prev, wmask;
};
template <int NPT>  // up to 1,024 NPT spheres
struct IntLds {
    unsigned mark[NPT * 32];
    short before[NPT * 32], slot[NPT * 1024], id[NPT * 1024];
    double x[NPT * 1024][3], u[NPT * 1024][3], f[NPT * 1024][3];
};
// what a sphere's substeps start from, with the angular velocity (which nothing in them
// reads) taken over all of them
__device__ __forceinline__ SubstepConst integrate_load(const Dev &D, int P, const IntArgs &A, double dt, double *x,
                                                       double *u, double *w) {
    const double *t = D.ptab + (long long)P * P_STRIDE;
    const SubstepConst c = substep_const(D, P, A.have_prev, dt, A.g);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        x[d] = t[P_X + d];
        u[d] = t[P_U + d];
        w[d] = t[P_W + d];
    }
    substep_spin(D, P, c, A.have_prev, dt, A.ns, w);
    return c;
}
__device__ __forceinline__ void integrate_store(const Geom &G, const Dev &D, int P, double R, const double *x,
                                                const double *u, const double *w) {
    double *t = D.ptab + (long long)P * P_STRIDE;
    const int n[3] = {G.nx, G.ny, G.nz};
    const double xo[3] = {t[P_X], t[P_X + 1], t[P_X + 2]};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        t[P_XOLD + d] = xo[d];
        t[P_X + d] = x[d];
        t[P_U + d] = u[d];
        t[P_W + d] = w[d];
    }
    t[P_OVL] = 0.0;
    if (moved_far(G, x, xo)) atomicOr(D.counters + C_COVALL, 1);
    if (!sphere_supported(x, R, n, G.per)) atomicOr(D.err, ERR_PART);
    mirror_store(D, P, x, u, w);
}
template <int NPT>
__device__ __forceinline__ void integrate(const Geom &G, const Dev &D, const IntArgs &A, int blk) {
    __shared__ IntLds<NPT> L;
    const int np = D.np, npair = min(D.counters[C_NPAIRS], A.pcap);
    const int tid = threadIdx.x;
    const double dt = 1.0 / A.ns;
    const int n[3] = {G.nx, G.ny, G.nz};
    bool left = false;  // a centre left the box between two substeps (and may be back)
    auto watch = [&](const double *x, double R) { left |= np > INT_WATCH && !sphere_supported(x, R, n, G.per); };
    for (int i = tid; i < NPT * 32; i += 1024) L.mark[i] = 0u;
    __syncthreads();
    constexpr int NPR = 2;  // pairs that a thread of block 0 keeps in registers
    int2 pr[NPR];
    double Ra[NPR], Rb[NPR];
    auto mark = [&](int2 q) {
        atomicOr(&L.mark[q.x >> 5], 1u << (q.x & 31));
        atomicOr(&L.mark[q.y >> 5], 1u << (q.y & 31));
    };
#pragma unroll
    for (int j = 0; j < NPR; ++j) {
        const int k = tid + 1024 * j;
        pr[j] = make_int2(-1, -1);
        if (k >= npair) continue;
        pr[j] = D.pairs[k];
        if (blk == 0) {
            Ra[j] = D.ptab[(long long)pr[j].x * P_STRIDE + P_R];
            Rb[j] = D.ptab[(long long)pr[j].y * P_STRIDE + P_R];
        }
        mark(pr[j]);
    }
    for (int k = tid + 1024 * NPR; k < npair; k += 1024) mark(D.pairs[k]);
    __syncthreads();
    if (blk > 0) {
        const int P = (blk - 1) * INT_LONE + tid;
        if (tid >= INT_LONE || P >= np || ((L.mark[P >> 5] >> (P & 31)) & 1u)) return;
        double x[3], u[3], w[3], f[3] = {0.0, 0.0, 0.0};
        const SubstepConst c = integrate_load(D, P, A, dt, x, u, w);
        for (int s = 0; s < A.ns; ++s) {
            substep_one(G, c, x, u, f, dt, A.mu, A.kc, A.wmask);
            watch(x, c.R);
        }
        integrate_store(G, D, P, c.R, x, u, w);
        if (left) atomicOr(D.err, ERR_PART);
        return;
    }
    if (npair == 0) return;
    // the marked spheres' places in LDS
    if (tid < 64) {
        const int n = tid < NPT * 32 ? __popc(L.mark[tid]) : 0;
        int sum = n;
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(sum, o);
            if (tid >= o) sum += v;
        }
        if (tid < NPT * 32) L.before[tid] = (short)(sum - n);
    }
    __syncthreads();
    for (int P = tid; P < np; P += 1024)
        if ((L.mark[P >> 5] >> (P & 31)) & 1u) {
            const int s = L.before[P >> 5] + __popc(L.mark[P >> 5] & ((1u << (P & 31)) - 1u));
            L.slot[P] = (short)s;
            L.id[s] = (short)P;
        }
    const int last = NPT * 32 - 1, nm = L.before[last] + __popc(L.mark[last]);
    __syncthreads();
    int pa[NPR], pb[NPR];  // their places, sum of radii and lub_factor
    double sR[NPR], lub[NPR];
#pragma unroll
    for (int j = 0; j < NPR; ++j) {
        pa[j] = -1;
        if (pr[j].x < 0) continue;
        pa[j] = L.slot[pr[j].x];
        pb[j] = L.slot[pr[j].y];
        sR[j] = Ra[j] + Rb[j];
        lub[j] = lub_factor(Ra[j], Rb[j], A.mu);
    }
    // the constants of the first 1,024 spheres too; the few beyond, on crowded tables, form
    // theirs again in each substep
    SubstepConst c;
    double x[3], u[3], w[3];
    for (int i = tid; i < nm; i += 1024) {
        double wi[3];
        const SubstepConst ci = integrate_load(D, L.id[i], A, dt, L.x[i], L.u[i], wi);
        if (i == tid) {
            c = ci;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                w[d] = wi[d];
                x[d] = L.x[i][d];
                u[d] = L.u[i][d];
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) L.f[i][d] = 0.0;
    }
    __syncthreads();
    auto pair_add = [&](int a, int b, double s, auto l) {
        double f[3];
        if (!pair_force(G, L.x[a], L.u[a], L.x[b], L.u[b], s, l, A.kc, f)) return;
        for (int d = 0; d < 3; ++d) {
            atomicAdd(&L.f[a][d], f[d]);
            atomicAdd(&L.f[b][d], -f[d]);
        }
    };
    for (int s = 0; s < A.ns; ++s) {
#pragma unroll
        for (int j = 0; j < NPR; ++j)
            if (pa[j] >= 0) pair_add(pa[j], pb[j], sR[j], [&] { return lub[j]; });
        for (int k = tid + 1024 * NPR; k < npair; k += 1024) {
            const int2 q = D.pairs[k];
            const double Ra = D.ptab[(long long)q.x * P_STRIDE + P_R], Rb = D.ptab[(long long)q.y * P_STRIDE + P_R];
            pair_add(L.slot[q.x], L.slot[q.y], Ra + Rb, [&] { return lub_factor(Ra, Rb, A.mu); });
        }
        __syncthreads();
        for (int i = tid; i < nm; i += 1024) {
            if (i == tid) {
                double f[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    f[d] = L.f[i][d];
                    L.f[i][d] = 0.0;
                }
                substep_one(G, c, x, u, f, dt, A.mu, A.kc, A.wmask);
                watch(x, c.R);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    L.x[i][d] = x[d];
                    L.u[i][d] = u[d];
                }
                continue;
            }
            const SubstepConst ci = substep_const(D, L.id[i], A.have_prev, dt, A.g);
            substep_one(G, ci, L.x[i], L.u[i], L.f[i], dt, A.mu, A.kc, A.wmask);
            watch(L.x[i], ci.R);
        }
        __syncthreads();
    }
    for (int i = tid; i < nm; i += 1024) {
        if (i >= 1024) {
            double xi[3], ui[3];
            c = integrate_load(D, L.id[i], A, dt, xi, ui, w);
        }
        integrate_store(G, D, L.id[i], c.R, L.x[i], L.u[i], w);
    }
    if (left) atomicOr(D.err, ERR_PART);
    block_phase();
    auto flag = [&](int2 q, double s) {
        if (may_overlap(G, L.x[L.slot[q.x]], L.x[L.slot[q.y]], s))
            D.ptab[(long long)q.x * P_STRIDE + P_OVL] = D.ptab[(long long)q.y * P_STRIDE + P_OVL] = 1.0;
    };
#pragma unroll
    for (int j = 0; j < NPR; ++j)
        if (pr[j].x >= 0) flag(pr[j], sR[j]);
    for (int k = tid + 1024 * NPR; k < npair; k += 1024) {
        const int2 q = D.pairs[k];
        flag(q, D.ptab[(long long)q.x * P_STRIDE + P_R] + D.ptab[(long long)q.y * P_STRIDE + P_R]);
    }
}
template <int NPT>
__global__ __launch_bounds__(1024) void k_integrate(Geom G, Dev D, IntArgs A) {
    integrate<NPT>(G, D, A, blockIdx.x);
}
// ... beside the conversions of the step, which neither read nor write the sphere table (the
// first nconv blocks; apart 18 and 23 us on a bed of 128^3, together 34)
template <int ST, int NPT>
__global__ __launch_bounds__(1024) void k_conv_integrate(Geom G, Phys Ph, Dev D, IntArgs A, int nconv) {
    if ((int)blockIdx.x < nconv) conversions<ST>(G, Ph, D, nconv);
    else integrate<NPT>(G, D, A, blockIdx.x - nconv);
}

// ---- coverage update --------------------------------------------------------------
// Which spheres resolve their coverage through claims (lowest index wins an
// overlap): those with a candidate partner whose centre is closer than the radii
// plus one cell at the new positions, and those that moved half a cell or more.
// For every other sphere no node can be inside it and another sphere at once, so
// its cover and uncover events follow from the inside tests at the old and new
// positions alone.
__global__ void k_cov_flag_init(Geom G, Dev D) {
    GRID_STRIDE(P, D.np) {
        double *t = D.ptab + (long long)P * P_STRIDE;
        t[P_OVL] = 0.0;
        // a sphere that moved half a cell or more in one step may meet partners that
        // the pair list (taken at the old positions) does not hold: then every
        // sphere takes the claim path this step
        if (moved_far(G, t + P_X, t + P_XOLD)) atomicOr(D.counters + C_COVALL, 1);
    }
}
__device__ __forceinline__ bool cov_claims(const Dev &D, const double *t) {
    return t[P_OVL] != 0.0 || D.counters[C_COVALL] != 0;
}
__global__ void k_cov_flag_pairs(Geom G, Dev D, int pcap) {
    const int n = min(D.counters[C_NPAIRS], pcap);
    GRID_STRIDE(k, n) {
        const int a = D.pairs[k].x, b = D.pairs[k].y;
        double *ta = D.ptab + (long long)a * P_STRIDE, *tb = D.ptab + (long long)b * P_STRIDE;
        if (may_overlap(G, ta + P_X, tb + P_X, ta[P_R] + tb[P_R])) ta[P_OVL] = tb[P_OVL] = 1.0;
    }
}

// The threads that walk one sphere's nodes: 2^sh of them (a wave or more; blocks of
// max(256, 2^sh)).  With a wave a sphere of R = 8 takes 77 rounds of dependent loads, so
// small tables, which leave the device idle, give a sphere up to 1,024 threads (333
// spheres: claims 49 -> 8 us, scan 84 -> 14 us); large ones fill it with a wave each.
struct Team {
    int P, lane, n;
    __device__ __forceinline__ Team(int block, int sh) {
        const int t = block * (int)blockDim.x + (int)threadIdx.x;
        P = t >> sh;
        n = 1 << sh;
        lane = t & (n - 1);
    }
};

// the node box of every sphere (all = 0: of those flagged above) is walked and its nodes
// claimed
__global__ void k_cov_claim(Geom G, Dev D, int all, int sh) {
    const Team T(blockIdx.x, sh);
    if (T.P >= D.np) return;
    const double *t = D.ptab + (long long)T.P * P_STRIDE;
    if (!all && !cov_claims(D, t)) return;
    int lo[3], hi[3];
    sphere_box(G, t + P_X, t[P_R], lo, hi);
    int ex = hi[0] - lo[0] + 1, ey = hi[1] - lo[1] + 1, ez = hi[2] - lo[2] + 1;
    int tot = ex * ey * ez;
    for (int s = T.lane; s < tot; s += T.n) {
        int i = lo[0] + s % ex, j = lo[1] + (s / ex) % ey, k = lo[2] + s / (ex * ey);
        if (inside(i, j, k, t + P_X, t[P_R])) atomicMin(D.claim + node_at(G, i, j, k), T.P);
    }
}

__device__ __forceinline__ int event_len(const Dev &D, int which) {
    int n = D.counters[which];
    return n < D.capEv ? n : D.capEv;
}

__device__ __forceinline__ void push_event(const Dev &D, int *list, int which, int cell, int P) {
    int s = atomicAdd(D.counters + which, 1);
    if (s < D.capEv) { list[2 * s] = cell; list[2 * s + 1] = P; }
    else atomicOr(D.err, ERR_CAP);
}

// cell c becomes a node of sphere P; returns the mass it hands to the ledger.  Only the
// sphere that takes a node (the lowest index inside, see k_cov_flag_init) calls this, and a
// scan that meets the cell before or after decides the same: a fluid cell has no owner.
template <int ST>
__device__ __forceinline__ double cover_cell(const Geom &G, const Phys &Ph, const Dev &D, int c, int P, double *phi) {
    const uint8_t f = D.flags[c];
    double led = 0.0;
    if (f == LIQ) led = cell_rho<ST>(G, D, Ph, D.fB, c);
    else if (f == IFC) led = D.m[c];
    else if (f == GAS) D.cv[c] = CV_GRM;  // left the gas: for the splitting test
    // the relabelling after a merge sees gas and interface cells only
    if ((f == GAS || f == IFC) && D.counters[C_MERGED]) D.bub[c] = (uint16_t)bubble_root(D, D.bub[c]);
    D.flags[c] = SOL;
    D.pid[c] = P;
    phi[c] = 0.0;
    return led;
}

// Walks the union of the old and new bounding boxes: nodes that the sphere covers become
// its nodes at once (apply) or are listed for k_cov_apply, nodes that it leaves are marked
// (CV_UNC) and listed for k_unc.  The ledger takes the covered mass summed per wave.  Covering
// at once saves small tables a launch; on large ones the populations of a covered cell are read
// by a few lanes of each wave in turn (23,328 spheres, 99,000 cells a step: 2.71 ms against 1.28
// and 0.07 apart).
template <int ST>
__global__ void k_cov_scan(Geom G, Phys Ph, Dev D, double *phi, int sh, int apply) {
    const Team T(blockIdx.x, sh);
    const int P = T.P;
    if (P >= D.np) return;
    const double *t = D.ptab + (long long)P * P_STRIDE;
    // the old centre at its image nearest the new one: both boxes in one frame
    double xo[3];
    image_near(G, t + P_XOLD, t + P_X, xo);
    int lo[3], hi[3], lo2[3], hi2[3];
    const bool inNew = sphere_box(G, t + P_X, t[P_R], lo, hi);
    const bool inOld = sphere_box(G, xo, t[P_R], lo2, hi2);
    if (!inNew && !inOld) return;
    for (int a = 0; a < 3; ++a) {
        lo[a] = !inNew ? lo2[a] : !inOld ? lo[a] : min(lo[a], lo2[a]);
        hi[a] = !inNew ? hi2[a] : !inOld ? hi[a] : max(hi[a], hi2[a]);
    }
    double led = 0.0;
    auto events = [&](bool cov, bool unc, int c) {
        wave_push2(cov, c, P, D.lCov, D.counters + C_NCOVER, D.capEv, D.err);
        wave_push2(unc, c, P, D.lUnc, D.counters + C_NUNCOVER, D.capEv, D.err);
        if (cov && apply) led += cover_cell<ST>(G, Ph, D, c, P, phi);
        if (unc) D.cv[c] = CV_UNC;
    };
    if (cov_claims(D, t)) {
        // by cell index: along a periodic axis n consecutive nodes hold every cell once
        const int n[3] = {G.nx, G.ny, G.nz};
        for (int a = 0; a < 3; ++a)
            if (G.per[a]) hi[a] = min(hi[a], lo[a] + n[a] - 1);
        const int ex = hi[0] - lo[0] + 1, ey = hi[1] - lo[1] + 1, ez = hi[2] - lo[2] + 1;
        const int tot = ex * ey * ez;
        for (int s = T.lane; s < tot; s += T.n) {
            const int i = lo[0] + s % ex, j = lo[1] + (s / ex) % ey, k = lo[2] + s / (ex * ey);
            const int c = node_at(G, i, j, k);
            const int cl = D.claim[c];
            const uint8_t f = D.flags[c];
            const bool owned = f == SOL && D.pid[c] == P;
            const bool mine = cl == P && !owned;
            if (mine && f == SOL) D.pid[c] = P;  // owner changes to the lower index
            events(mine && f != SOL, owned && cl == CLAIM_NONE, c);
        }
    } else {
        const int ex = hi[0] - lo[0] + 1, ey = hi[1] - lo[1] + 1;
        // a sphere alone (it moved less than half a cell): only nodes whose inside test
        // changed between the old and new positions can change owner.  Walked as (x, y) columns: the in-plane part of
        // both squared distances is formed once per column, in the order of inside(), and
        // a column outside both circles is skipped (adding dz^2 cannot bring it inside);
        // cov_column_ranges gives the candidates of the others, and every candidate
        // still takes the exact test.
        const double *xn = t + P_X;
        const double R2 = __dmul_rn(t[P_R], t[P_R]);
        for (int s = T.lane; s < ex * ey; s += T.n) {
            const int i = lo[0] + s % ex, j = lo[1] + s / ex;
            const double a0 = i - xn[0], a1 = j - xn[1], b0 = i - xo[0], b1 = j - xo[1];
            const double sn = __dadd_rn(__dmul_rn(a0, a0), __dmul_rn(a1, a1));
            const double so = __dadd_rn(__dmul_rn(b0, b0), __dmul_rn(b1, b1));
            if (sn > R2 && so > R2) continue;
            int r[4];  // candidate ranges of k
            cov_column_ranges(sn, so, R2, xn[2], xo[2], lo[2], hi[2], r);
            const int r1lo = r[0], r2lo = r[2];
            const int n1 = max(r[1] - r1lo + 1, 0), n2 = max(r[3] - r2lo + 1, 0);
            for (int m = 0; m < n1 + n2; ++m) {
                const int k = m < n1 ? r1lo + m : r2lo + (m - n1);
                const double a2 = k - xn[2], b2 = k - xo[2];
                const bool in_new = __dadd_rn(sn, __dmul_rn(a2, a2)) <= R2;
                const bool in_old = __dadd_rn(so, __dmul_rn(b2, b2)) <= R2;
                if (in_new == in_old) continue;
                const int c = node_at(G, i, j, k);
                const uint8_t f = D.flags[c];
                events(in_new && f != SOL, !in_new && f == SOL && D.pid[c] == P, c);
            }
        }
    }
    led = wave_sum(led);
    if (lane_id() == 0 && led != 0.0) unsafeAtomicAdd(D.ledger, led);
}

// full-box variant used when the table is replaced (no previous positions)
__global__ void k_cov_scan_dense(Geom G, Dev D) {
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < G.N;
         c += (long long)gridDim.x * blockDim.x) {
        int cl = D.claim[c];
        uint8_t f = D.flags[c];
        if (f == SOL) {
            if (cl == CLAIM_NONE) {
                push_event(D, D.lUnc, C_NUNCOVER, (int)c, D.pid[c]);
                D.cv[c] = CV_UNC;
            } else {
                D.pid[c] = cl;
            }
        } else if (cl != CLAIM_NONE) {
            push_event(D, D.lCov, C_NCOVER, (int)c, cl);
        }
    }
}

// the listed covered nodes; the ledger takes the mass summed per wave (one atomic per wave):
// every wave of the block takes the same rounds, so the sums see whole waves
template <int ST>
__global__ void k_cov_apply(Geom G, Phys Ph, Dev D, double *phi) {
    const int n = event_len(D, C_NCOVER);
    for (int base = blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
        const int e = base + threadIdx.x;
        double led = 0.0;
        if (e < n) led = cover_cell<ST>(G, Ph, D, D.lCov[2 * e], D.lCov[2 * e + 1], phi);
        led = wave_sum(led);
        if (lane_id() == 0 && led != 0.0) unsafeAtomicAdd(D.ledger, led);
    }
}

// Uncovered nodes (32 lanes each, lane q the neighbour along q): the decision with the cell
// types after covering, every uncovered node still solid (its mark says so, whatever type
// it shows by then), and the cell's new state.  When all are decided, uncover_finish makes
// interface cells of those that came to lie next to gas uncovered in this step (the
// closure; only if there is any) and clears the marks.
// the new state of node c, left by its sphere in event e, with nli liquid or interface neighbours
// of densities rs in sum and the bubble of its first gas neighbour (-1: none)
template <int ST>
__device__ __forceinline__ void uncover_cell(const Geom &G, const Phys &Ph, const Dev &D, double *phi, int e, int c,
                                             int nli, double rs, int bub) {
    const int type = nli > 0 ? (bub >= 0 ? IFC : LIQ) : (bub >= 0 ? GAS : LIQ);
    const double rb = nli > 0 ? rs / nli : 1.0;
    D.uncDec[e] = type;
    D.uncRho[e] = rb;
    D.pid[c] = -1;
    D.flags[c] = (uint8_t)type;
    if (type == GAS) {
        D.bub[c] = (uint16_t)bub;
        phi[c] = 0.0;
        __hip_atomic_store(D.counters + C_NUGAS, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    const int P = D.lUnc[2 * e + 1];
    float u0 = 0.f, u1 = 0.f, u2 = 0.f;
    if ((unsigned)P < (unsigned)D.np) {
        int x, y, z;
        cell_xyz(G, c, x, y, z);
        const double *t = D.ptab + (long long)P * P_STRIDE;
        double rx = min_img(x - t[P_X], G.nx, G.per[0]), ry = min_img(y - t[P_X + 1], G.ny, G.per[1]),
               rz = min_img(z - t[P_X + 2], G.nz, G.per[2]);
        u0 = (float)(t[P_U] + (t[P_W + 1] * rz - t[P_W + 2] * ry));
        u1 = (float)(t[P_U + 1] + (t[P_W + 2] * rx - t[P_W] * rz));
        u2 = (float)(t[P_U + 2] + (t[P_W] * ry - t[P_W + 1] * rx));
    }
    store_equilibrium<ST>(G, Ph, D.fB, c, rb - 1.0, u0, u1, u2);
    // the density of the stored populations, for rho_w (Eq. bbrule) in the next launch
    if (D.rhow != nullptr && D.st_cur >= 0)
        D.rhow[c] = rhow_word((float)cell_rho<ST>(G, D, Ph, D.fB, c), D.st_cur);
    unsafeAtomicAdd(D.ledger, -rb);
    phi[c] = 1.0;
    if (type == IFC) {
        D.m[c] = rb;
        D.bub[c] = (uint16_t)bub;
    }
}

template <int ST>
__device__ __forceinline__ void uncover(const Geom &G, const Phys &Ph, const Dev &D, double *phi, const Items &W) {
    const int n = event_len(D, C_NUNCOVER);
    ITEM_LOOP(W, e, n) {
        const bool has = e < n;
        const int c = has ? D.lUnc[2 * e] : 0;
        const int nb = lane_nbr(G, c, W.q, has);
        const uint8_t f = nb < 0 ? WALL : (D.cv[nb] & CV_UNC) ? SOL : D.flags[nb];
        const bool li = f == LIQ || f == IFC;
        const double r = li ? cell_rho<ST>(G, D, Ph, D.fB, nb) : 0.0;
        const unsigned ml = W.any(li), mg = W.any(f == GAS);
        const int bub = W.from(f == GAS ? (int)D.bub[nb] : 0, mg ? __ffs(mg) - 1 : 0);
        // mean density of the neighbours, summed in direction order
        double rs = 0.0;
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            const double rq = W.from(r, q);
            if ((ml >> q) & 1u) rs += rq;
        }
        if (has && W.q == 0) uncover_cell<ST>(G, Ph, D, phi, e, c, __popc(ml), rs, mg ? bub : -1);
    }
}
// ... a thread to a node, for lists that fill the device several times over: 32 lanes have one
// neighbour each, most of them without populations to read (the 12.2 M nodes of a replaced table:
// 27 ms against 76)
template <int ST>
__device__ __forceinline__ void uncover_each(const Geom &G, const Phys &Ph, const Dev &D, double *phi, int thread,
                                             int nthreads) {
    const int n = event_len(D, C_NUNCOVER);
    for (int e = thread; e < n; e += nthreads) {
        const int c = D.lUnc[2 * e];
        int x, y, z, nli = 0, bub = -1;
        cell_xyz(G, c, x, y, z);
        double rs = 0.0;
        for (int q = 1; q < Q; ++q) {
            const int nb = nbr_idx(G, x, y, z, q, 1);
            if (nb < 0 || (D.cv[nb] & CV_UNC)) continue;
            const uint8_t f = D.flags[nb];
            if (f == LIQ || f == IFC) {
                rs += cell_rho<ST>(G, D, Ph, D.fB, nb);
                ++nli;
            } else if (f == GAS && bub < 0) {
                bub = D.bub[nb];
            }
        }
        uncover_cell<ST>(G, Ph, D, phi, e, c, nli, rs, bub);
    }
}

// an uncovered liquid cell next to gas becomes interface
__device__ __forceinline__ void uncover_closure(const Geom &G, const Dev &D, double *phi, const Items &W) {
    const int n = event_len(D, C_NUNCOVER);
    ITEM_LOOP(W, e, n) {
        const bool has = e < n && D.uncDec[e < n ? e : 0] == LIQ;
        const int c = has ? D.lUnc[2 * e] : 0;
        const int nb = lane_nbr(G, c, W.q, has);
        const unsigned mg = W.any(nb >= 0 && D.flags[nb < 0 ? 0 : nb] == GAS);
        if (!has || !mg || W.q != __ffs(mg) - 1) continue;
        D.flags[c] = IFC;
        D.m[c] = D.uncRho[e];
        phi[c] = 1.0;
        D.bub[c] = D.bub[nb];
    }
}

// closure and marks, by the blocks of W together; neither touches what the other reads
__device__ __forceinline__ void uncover_finish(const Geom &G, const Dev &D, double *phi, const Items &W, int block,
                                               int nblk) {
    const int n = event_len(D, C_NUNCOVER);
    if (__hip_atomic_load(D.counters + C_NUGAS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0)
        uncover_closure(G, D, phi, W);
    // new gas stays marked for the splitting test
    for (int e = block * blockDim.x + threadIdx.x; e < n; e += nblk * blockDim.x)
        D.cv[D.lUnc[2 * e]] = D.uncDec[e] == GAS ? CV_GAD : 0;
}
// A launch of its own where the nodes may be many (large tables, a table that is replaced):
// 23,328 spheres of radius 5 moving at 0.05 through the surface of a 512 x 512 x 256 pool take
// 1.6 ms of coverage a step, and replacing the table (12.2 M nodes) 27 ms; 11.4 ms and 1.3 s when
// the block that finished last did this for all nodes.
__global__ __launch_bounds__(256) void k_unc_finish(Geom G, Dev D, double *phi) {
    uncover_finish(G, D, phi, Items(blockIdx.x, gridDim.x), blockIdx.x, gridDim.x);
}

// The first unc_blocks blocks take the uncovered nodes, the others (threads by sphere as
// in k_cov_claim) take back the claims, which the scan before was the last to read.
// finish: as many of the former as the nodes fill, one to a half wave, go on to uncover_finish
// after a grid barrier (small tables); else k_unc_finish follows.
template <int ST>
__global__ __launch_bounds__(1024) void k_unc(Geom G, Phys Ph, Dev D, double *phi, int unc_blocks, int sh, int finish) {
    if ((int)blockIdx.x < unc_blocks) {
        const int per = (int)(blockDim.x >> 5);
        const int nblk = min(unc_blocks, max(1, (event_len(D, C_NUNCOVER) + per - 1) / per));
        if ((int)blockIdx.x >= nblk) return;
        const Items W(blockIdx.x, nblk);
        if (!finish && event_len(D, C_NUNCOVER) > 4 * W.ngrp) {
            uncover_each<ST>(G, Ph, D, phi, blockIdx.x * blockDim.x + threadIdx.x, nblk * blockDim.x);
            return;
        }
        uncover<ST>(G, Ph, D, phi, W);
        if (!finish) return;
        GridBarrier{D.counters + C_BARU, nblk, 0, D.err}.wait();
        uncover_finish(G, D, phi, W, blockIdx.x, nblk);
        return;
    }
    const Team T(blockIdx.x - unc_blocks, sh);
    if (T.P >= D.np) return;
    const double *t = D.ptab + (long long)T.P * P_STRIDE;
    if (!cov_claims(D, t)) return;
    int lo[3], hi[3];
    sphere_box(G, t + P_X, t[P_R], lo, hi);
    int ex = hi[0] - lo[0] + 1, ey = hi[1] - lo[1] + 1, ez = hi[2] - lo[2] + 1;
    int tot = ex * ey * ez;
    for (int s = T.lane; s < tot; s += T.n) {
        int i = lo[0] + s % ex, j = lo[1] + (s / ex) % ey, k = lo[2] + s / (ex * ey);
        D.claim[node_at(G, i, j, k)] = CLAIM_NONE;
    }
}

}  // namespace fsl
