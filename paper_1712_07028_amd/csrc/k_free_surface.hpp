// k_free_surface.hpp -- list-driven cell conversions (Sec. 2.2, Fig.
// cellConversions) and the bubble model (end of Sec. 2.2).
//
// The stream-collide kernel leaves two lists of interface cells, filled (phi >= 1 -
// eps_c) and emptied (phi <= eps_c), and marks them (CV_F, CV_E0).  Three phases follow:
//   closure : conflict rule (an emptied cell next to a filled one stays interface);
//             gas neighbours of filled cells and liquid neighbours of emptied cells
//             become new interface cells (one winner per cell by an atomic OR), the
//             former with m = 0, the latter with m = rho
//   change  : new interface cells from gas take the equilibrium at the mean density and
//             velocity of their liquid/interface neighbours; those from liquid the
//             bubble id of their first emptied neighbour; cell types; excess mass (m -
//             rho, or m) shared equally by the neighbours that are interface now (FP64
//             atomics), or paid into the ledger
//   fill    : fill levels of the recipients, marks cleared, invariant checked, bubble
//             merges recorded and carried out
// Every phase touches only the listed cells and their neighbours.  Cell types change in
// the phase that also needs the old and the new types of neighbours: both follow from
// the type a neighbour shows, old or new, and its mark, which that phase does not change.
//
// A listed cell is worked by 32 lanes, lane q taking the neighbour along direction q: the
// lists are short (tens of cells on a 128^3 pool, thousands on a 500 x 500 surface), so
// a phase costs the latency of its dependent loads, which one thread per cell paid 18
// times over (128^3 pool with 1,400 spheres: 19 to 22 us per phase, six phases).
#pragma once

#include "fsl_device.hpp"

namespace fsl {

__device__ __forceinline__ void cell_xyz(const Geom &G, int c, int &x, int &y, int &z) {
    x = c % G.nx;
    int r = c / G.nx;
    y = r % G.ny;
    z = r / G.ny;
}

// neighbour index of c along q, -1 beyond a wall
__device__ __forceinline__ int nbr_idx(const Geom &G, int x, int y, int z, int q, int sign) {
    int a = x + sign * cx(q), b = y + sign * cy(q), d = z + sign * cz(q);
    if (a < 0 || a >= G.nx) { if (!G.per[0]) return -1; a = wrapc(a, G.nx); }
    if (b < 0 || b >= G.ny) { if (!G.per[1]) return -1; b = wrapc(b, G.ny); }
    if (d < 0 || d >= G.nz) { if (!G.per[2]) return -1; d = wrapc(d, G.nz); }
    return a + G.nx * (b + G.ny * d);
}

template <int ST>
__device__ __forceinline__ double cell_rho(const Geom &G, const Dev &D, const Phys &Ph, const void *F, int c) {
    using SS = Store<ST>;
    const typename SS::T *p = (const typename SS::T *)F;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) s += (double)SS::ld(p + q * G.S + c, Ph.inv);
    return 1.0 + s;
}

// density deviation drho = rho - 1 and velocity of the post-collision populations
// (first moment minus half the Guo force)
template <int ST>
__device__ __forceinline__ void cell_rho_u(const Geom &G, const Phys &Ph, const void *F, int c,
                                           float &drho, float &u0, float &u1, float &u2) {
    using SS = Store<ST>;
    const typename SS::T *p = (const typename SS::T *)F;
    float d = 0.f, j0 = 0.f, j1 = 0.f, j2 = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        float h = SS::ld(p + q * G.S + c, Ph.inv);
        d += h;
        j0 += cx(q) * h;
        j1 += cy(q) * h;
        j2 += cz(q) * h;
    }
    drho = d;
    const float rho = 1.0f + d;
    u0 = j0 / rho - 0.5f * Ph.g[0];
    u1 = j1 / rho - 0.5f * Ph.g[1];
    u2 = j2 / rho - 0.5f * Ph.g[2];
}

// shifted equilibrium e_q(rho,u) - w_q written to cell c; drho = rho - 1 is passed
// separately so that it keeps its own precision
template <int ST>
__device__ __forceinline__ void store_equilibrium(const Geom &G, const Phys &Ph, void *F, int c,
                                                  double drho_d, float u0, float u1, float u2) {
    using SS = Store<ST>;
    typename SS::T *p = (typename SS::T *)F;
    const float drho = (float)drho_d;
    const float rho = 1.0f + drho;
    float uu = u0 * u0 + u1 * u1 + u2 * u2;
    // moving populations in FP32; the rest population carries the exact mass balance
    // sum_q h_q = rho - 1 (the equilibrium's zeroth moment), so that the rounded
    // weights do not bias the mass of the cell
    double s = 0.0;
#pragma unroll
    for (int q = 1; q < Q; ++q) {
        float cu = cx(q) * u0 + cy(q) * u1 + cz(q) * u2;
        float h = wq(q) * (drho + rho * (3.0f * cu + 4.5f * cu * cu - 1.5f * uu));
        const typename SS::T v = SS::enc(h, Ph.scale);
        s += (double)SS::dec(v, Ph.inv);
        p[q * G.S + c] = v;
    }
    SS::st(p + c, (float)(drho_d - s), Ph.scale);
}

__device__ __forceinline__ uint8_t cv_or(uint8_t *cv, int c, uint8_t bits) {
    unsigned *w = (unsigned *)(cv + (c & ~3));
    int sh = 8 * (c & 3);
    unsigned old = atomicOr(w, (unsigned)bits << sh);
    return (uint8_t)(old >> sh);
}

__device__ __forceinline__ int list_len(const Dev &D, int which) {
    int n = D.counters[which];
    return n < D.cap ? n : D.cap;
}

#define GRID_STRIDE(i, n) for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += gridDim.x * blockDim.x)

// root of a bubble id through the merge table; ids outside the table map to 0
__device__ __forceinline__ int bubble_root(const Dev &D, int b) {
    for (int it = 0; it < 64; ++it) {
        if (b < 0 || b >= D.maxB) return 0;
        int r = D.broot[b];
        if (r == b) return b;
        b = r;
    }
    return b < 0 || b >= D.maxB ? 0 : b;
}

// item i of a phase is worked by 32 lanes; grp and ngrp: this half wave's number and how
// many there are.  The loop runs the same rounds in both halves of a wave.
struct Items {
    int grp, ngrp, q, half;
    __device__ __forceinline__ Items(int block, int nblocks) {
        q = (int)(threadIdx.x & 31u);
        half = (int)((threadIdx.x >> 5) & 1u);
        const int per = (int)(blockDim.x >> 5);
        grp = block * per + (int)(threadIdx.x >> 5);
        ngrp = nblocks * per;
    }
    // the lanes of this half wave with pred, as a 32-bit set (bit q: lane q)
    __device__ __forceinline__ unsigned any(bool pred) const { return (unsigned)(__ballot(pred) >> (32 * half)); }
    __device__ __forceinline__ int from(int v, int lane) const { return __shfl(v, 32 * half + lane); }
    __device__ __forceinline__ float from(float v, int lane) const { return __shfl(v, 32 * half + lane); }
    __device__ __forceinline__ double from(double v, int lane) const { return __shfl(v, 32 * half + lane); }
};
#define ITEM_LOOP(W, i, n) for (int i = (W).grp, i##0 = (W).grp - (W).half; i##0 < (n); i += (W).ngrp, i##0 += (W).ngrp)

// neighbour of cell c along the lane's direction q (-1 beyond a wall; lanes whose q is
// no direction, or without a cell: -1)
__device__ __forceinline__ int lane_nbr(const Geom &G, int c, int q, bool has) {
    if (!has || q < 1 || q >= Q) return -1;
    int x, y, z;
    cell_xyz(G, c, x, y, z);
    int a = x + dir_comp<0>(q), b = y + dir_comp<1>(q), d = z + dir_comp<2>(q);
    if (a < 0 || a >= G.nx) { if (!G.per[0]) return -1; a = wrapc(a, G.nx); }
    if (b < 0 || b >= G.ny) { if (!G.per[1]) return -1; b = wrapc(b, G.ny); }
    if (d < 0 || d >= G.nz) { if (!G.per[2]) return -1; d = wrapc(d, G.nz); }
    return a + G.nx * (b + G.ny * d);
}

// the lists that the closure phase makes
enum { L_E, L_NL, L_NG, L_N };
__device__ __forceinline__ int *conv_list(const Dev &D, int k) { return k == L_E ? D.lE : k == L_NL ? D.lNL : D.lNG; }
__device__ __forceinline__ int *conv_count(const Dev &D, int k) {
    return D.counters + (k == L_E ? C_NE : k == L_NL ? C_NNL : C_NNG);
}
// The entries of a block gathered in LDS, for launches of many blocks: one atomic per wave and
// round on three counters of one line queues (tens of thousands of listed cells on a 512 x 512
// surface that 23,328 spheres cross: 611 us a launch against 50).
struct ListBuf {
    static constexpr int CAP = 512;
    int n[L_N], base[L_N], buf[L_N][CAP];
    __device__ __forceinline__ void open() {
        if (threadIdx.x < L_N) n[threadIdx.x] = 0;
        __syncthreads();
    }
    __device__ __forceinline__ void push(const Dev &D, int k, bool pred, int value) {
        const unsigned long long mask = __ballot(pred);
        if (!mask) return;
        const int leader = __ffsll((long long)mask) - 1;
        int at = 0;
        if ((int)lane_id() == leader) at = atomicAdd(&n[k], __popcll(mask));
        at = __shfl(at, leader) + __popcll(mask & ((1ull << lane_id()) - 1ull));
        if (pred && at < CAP) buf[k][at] = value;
        wave_append(pred && at >= CAP, value, conv_list(D, k), conv_count(D, k), D.cap, D.err);
    }
    __device__ __forceinline__ void close(const Dev &D) {
        __syncthreads();
        if (threadIdx.x < L_N) {
            const int m = min(n[threadIdx.x], CAP);
            base[threadIdx.x] = m ? atomicAdd(conv_count(D, threadIdx.x), m) : 0;
        }
        __syncthreads();
        for (int k = 0; k < L_N; ++k)
            for (int i = threadIdx.x; i < min(n[k], CAP); i += blockDim.x) {
                if (base[k] + i < D.cap) conv_list(D, k)[base[k] + i] = buf[k][i];
                else atomicOr(D.err, ERR_CAP);
            }
    }
};

// push(k, pred, value): appends to list k; every lane of the wave calls it
template <int ST, typename Push>
__device__ __forceinline__ void conv_closure(const Geom &G, const Phys &Ph, const Dev &D, const Items &W, Push &&push) {
    const int nF = list_len(D, C_NF), nE = list_len(D, C_NE0);
    ITEM_LOOP(W, i, nE) {
        const bool has = i < nE;
        const int c = has ? D.lE0[i] : 0;
        const int n = lane_nbr(G, c, W.q, has);
        const uint8_t nm = n >= 0 ? D.cv[n] : 0, nf = n >= 0 ? D.flags[n] : WALL;
        const bool keep = has && W.any(nm == CV_F) == 0u;
        if (keep && W.q == 0) cv_or(D.cv, c, CV_E);
        push(L_E, keep && W.q == 0, c);
        const bool won = keep && nf == LIQ && !(cv_or(D.cv, n, CV_NEWL) & CV_NEWL);
        push(L_NL, won, n);
        if (won) D.m[n] = cell_rho<ST>(G, D, Ph, D.fB, n);
    }
    ITEM_LOOP(W, j, nF) {
        const bool has = j < nF;
        const int c = has ? D.lF[j] : 0;
        const int n = lane_nbr(G, c, W.q, has);
        const bool won = n >= 0 && D.flags[n] == GAS && !(cv_or(D.cv, n, CV_NEWG) & CV_NEWG);
        push(L_NG, won, n);
        if (won) D.m[n] = 0.0;
    }
}

// a neighbour's type before and after the change phase, from the type it shows and its mark
__device__ __forceinline__ bool was_fluid(uint8_t f, uint8_t m) {  // liquid or interface before
    return (m & (CV_F | CV_E0 | CV_NEWL)) ? true : (m & CV_NEWG) ? false : f == LIQ || f == IFC;
}
__device__ __forceinline__ bool is_interface(uint8_t f, uint8_t m) {  // interface after
    return (m & (CV_NEWG | CV_NEWL)) ? true : (m & (CV_F | CV_E)) ? false : f == IFC;
}

// excess mass of cell c (the value of the half wave's lane 0) to its neighbours
__device__ __forceinline__ void share_excess(const Geom &G, const Dev &D, const Items &W, int c, bool has, double ex) {
    const int n = lane_nbr(G, c, W.q, has);
    const bool to = n >= 0 && is_interface(D.flags[n], D.cv[n]);
    const int k = __popc(W.any(to));
    ex = W.from(ex, 0);
    if (!has) return;
    if (k == 0) {
        if (W.q == 0) unsafeAtomicAdd(D.ledger, ex);
        return;
    }
    const double part = ex / k;
    if (to) unsafeAtomicAdd(D.m + n, part);
}

template <int ST>
__device__ __forceinline__ void conv_change(const Geom &G, const Phys &Ph, const Dev &D, const Items &W) {
    const int nG = list_len(D, C_NNG), nL = list_len(D, C_NNL), nF = list_len(D, C_NF), nE = list_len(D, C_NE);
    ITEM_LOOP(W, i, nG) {
        const bool has = i < nG;
        const int c = has ? D.lNG[i] : 0;
        const int n = lane_nbr(G, c, W.q, has);
        const bool src = n >= 0 && was_fluid(D.flags[n], D.cv[n]);
        float r = 0.f, a = 0.f, b = 0.f, e = 0.f;
        if (src) cell_rho_u<ST>(G, Ph, D.fB, n, r, a, b, e);
        const unsigned m = W.any(src);
        // the mean over the neighbours, summed in direction order
        float rs = 0.f, s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            const float rq = W.from(r, q), aq = W.from(a, q), bq = W.from(b, q), eq = W.from(e, q);
            if ((m >> q) & 1u) {
                rs += rq;
                s0 += aq;
                s1 += bq;
                s2 += eq;
            }
        }
        if (has && W.q == 0) {
            const float inv = 1.0f / (float)__popc(m);
            store_equilibrium<ST>(G, Ph, D.fB, c, (double)(rs * inv), s0 * inv, s1 * inv, s2 * inv);
            D.flags[c] = IFC;
        }
    }
    ITEM_LOOP(W, j, nL) {
        const bool has = j < nL;
        const int c = has ? D.lNL[j] : 0;
        const int n = lane_nbr(G, c, W.q, has);
        const unsigned m = W.any(n >= 0 && (D.cv[n] & CV_E));
        if (has && m && W.q == __ffs(m) - 1) D.bub[c] = D.bub[n];
        if (has && W.q == 0) D.flags[c] = IFC;
    }
    ITEM_LOOP(W, k, nF) {
        const bool has = k < nF;
        const int c = has ? D.lF[k] : 0;
        double ex = 0.0;
        if (has && W.q == 0) {
            ex = D.m[c] - cell_rho<ST>(G, D, Ph, D.fB, c);
            D.m[c] = 0.0;
            D.flags[c] = LIQ;
        }
        share_excess(G, D, W, c, has, ex);
    }
    ITEM_LOOP(W, l, nE) {
        const bool has = l < nE;
        const int c = has ? D.lE[l] : 0;
        double ex = 0.0;
        if (has && W.q == 0) {
            ex = D.m[c];
            D.m[c] = 0.0;
            D.flags[c] = GAS;
        }
        share_excess(G, D, W, c, has, ex);
    }
}

template <int ST>
__device__ __forceinline__ void conv_fill(const Geom &G, const Phys &Ph, const Dev &D, const Items &W, int thread,
                                          int nthreads) {
    const int nF = list_len(D, C_NF), nE = list_len(D, C_NE);
    const int nE0 = list_len(D, C_NE0), nG = list_len(D, C_NNG), nL = list_len(D, C_NNL);
    ITEM_LOOP(W, i, nF + nE) {
        const bool has = i < nF + nE, filled = i < nF;
        const int c = !has ? 0 : filled ? D.lF[i] : D.lE[i - nF];
        if (has && W.q == 0) D.phi_nxt[c] = filled ? 1.0 : 0.0;
        const int n = lane_nbr(G, c, W.q, has);
        if (n < 0) continue;
        const uint8_t f = D.flags[n];
        if (f == IFC) {
            D.phi_nxt[n] = D.m[n] / cell_rho<ST>(G, D, Ph, D.fB, n);
        } else if (filled ? f == GAS : f == LIQ) {
            atomicOr(D.err, ERR_LG);
        } else if (!filled && f == GAS) {
            const int a = bubble_root(D, D.bub[c]), b = bubble_root(D, D.bub[n]);
            if (a != b) {
                const int s = atomicAdd(D.counters + C_NMERGE, 1);
                if (s < D.cap) D.merges[s] = make_int2(a, b);
                else atomicOr(D.err, ERR_CAP);
            }
        }
    }
    for (int i = thread; i < nF; i += nthreads) D.cv[D.lF[i]] = 0;
    // emptied cells are new gas: marked for the splitting test
    for (int i = thread; i < nE0; i += nthreads) D.cv[D.lE0[i]] = (D.cv[D.lE0[i]] & CV_E) ? CV_GAD : 0;
    for (int i = thread; i < nG; i += nthreads) D.cv[D.lNG[i]] = CV_GRM;  // left the gas: for the splitting test
    for (int i = thread; i < nL; i += nthreads) D.cv[D.lNL[i]] = 0;
}

// serial union of merged bubbles: the lower root id survives, gas masses add.  The cells
// of merged bubbles are relabelled to their root by the bubble pass of the step.
__device__ __forceinline__ void merge_bubbles(const Dev &D) {
    int n = __hip_atomic_load(D.counters + C_NMERGE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n > D.cap) n = D.cap;
    for (int i = 0; i < n; ++i) {
        int a = bubble_root(D, D.merges[i].x), b = bubble_root(D, D.merges[i].y);
        if (a == b) continue;
        int lo = a < b ? a : b, hi = a < b ? b : a;
        D.broot[hi] = lo;
        D.btab[lo * B_STRIDE + B_M] += D.btab[hi * B_STRIDE + B_M];
        D.balive[hi] = 0;
        D.counters[C_MERGED] = 1;
    }
}

// The phases as one launch each (large boxes: any number of listed cells) ...
template <int ST>
__global__ __launch_bounds__(256) void k_conv_closure(Geom G, Phys Ph, Dev D) {
    __shared__ ListBuf L;
    L.open();
    conv_closure<ST>(G, Ph, D, Items(blockIdx.x, gridDim.x),
                     [&](int k, bool pred, int value) { L.push(D, k, pred, value); });
    L.close(D);
}
template <int ST>
__global__ __launch_bounds__(256) void k_conv_change(Geom G, Phys Ph, Dev D) {
    conv_change<ST>(G, Ph, D, Items(blockIdx.x, gridDim.x));
}
template <int ST>
__global__ __launch_bounds__(256) void k_conv_fill(Geom G, Phys Ph, Dev D) {
    conv_fill<ST>(G, Ph, D, Items(blockIdx.x, gridDim.x), blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
    if (last_block(D.counters + C_DONEC, gridDim.x) && threadIdx.x == 0) merge_bubbles(D);
}
// ... or all of them in one launch (small boxes): a launch costs 4.5 us, a barrier of the
// block a fraction of one and a grid barrier about three.  As many blocks take part as the
// lists fill, two cells per half wave; the others leave.
template <int ST>
__device__ __forceinline__ void conversions(const Geom &G, const Phys &Ph, const Dev &D, int nmax) {
    const int n = list_len(D, C_NF) + list_len(D, C_NE0);
    const int nblk = min(nmax, (n + 63) / 64);
    if ((int)blockIdx.x >= nblk) return;
    GridBarrier B{D.counters + C_BAR, nblk, 0, D.err};
    const Items W(blockIdx.x, nblk);
    conv_closure<ST>(G, Ph, D, W, [&](int k, bool pred, int value) {
        wave_append(pred, value, conv_list(D, k), conv_count(D, k), D.cap, D.err);
    });
    B.wait();
    conv_change<ST>(G, Ph, D, W);
    B.wait();
    conv_fill<ST>(G, Ph, D, W, blockIdx.x * blockDim.x + threadIdx.x, nblk * blockDim.x);
    if (last_block(D.counters + C_DONEC, nblk) && threadIdx.x == 0) merge_bubbles(D);
}
template <int ST>
__global__ __launch_bounds__(1024) void k_conversions(Geom G, Phys Ph, Dev D) {
    conversions<ST>(G, Ph, D, gridDim.x);
}

// ---- bubble volumes: dense pass over the cell types ------------------------------
struct BubbleLds {
    double acc[64 * BACC_STRIDE];
    int root[64];
};

// V_b = #gas cells + sum over interface cells of (1 - phi), with centroid moments;
// per-block LDS accumulation (FP64), one global atomic per block and component.  The cells
// of a bubble merged away in this step take their root's id on the way (relabel), so that
// merged ids hold no cells and a split can take them again.  A thread takes 16
// consecutive cells (one 16-byte load of types); 16 gas cells of one bubble in one row,
// which is nearly every chunk with gas, add in closed form (counts and coordinate sums
// are integers, exact in FP64).
__device__ __forceinline__ void bubble_accum(const Geom &G, const Dev &D, const double *phi, BubbleLds &L, bool relabel) {
    const int nb = D.nb;
    for (int i = threadIdx.x; i < nb * BACC_STRIDE; i += blockDim.x) L.acc[i] = 0.0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) L.root[i] = bubble_root(D, i);
    __syncthreads();
    const long long N = G.N;
    const long long nchunk = (N + 15) / 16;
    // the thread's sums for the bubble of the cells it is walking; they go to the
    // block's table only when the bubble changes (the cells of one region mostly
    // belong to one bubble)
    int bc = -1;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0, a4 = 0.0, a5 = 0.0;
    auto flush = [&]() {
        if (bc >= 0) {
            double *a = L.acc + bc * BACC_STRIDE;
            atomicAdd(a + 0, a0);
            atomicAdd(a + 1, a1);
            atomicAdd(a + 2, a2);
            atomicAdd(a + 3, a3);
            atomicAdd(a + 4, a4);
            atomicAdd(a + 5, a5);
        }
        a0 = a1 = a2 = a3 = a4 = a5 = 0.0;
    };
    for (long long ch = blockIdx.x * (long long)blockDim.x + threadIdx.x; ch < nchunk;
         ch += (long long)gridDim.x * blockDim.x) {
        const long long c0 = ch * 16;
        const uint4 f4 = *(const uint4 *)(D.flags + c0);
        // gas (0) and interface (2) are the even types
        if (((f4.x & f4.y & f4.z & f4.w) & 0x01010101u) == 0x01010101u) continue;
        int x = (int)(c0 % G.nx);
        const int yz = (int)(c0 / G.nx);
        int y = yz % G.ny, z = yz / G.ny;
        if ((f4.x | f4.y | f4.z | f4.w) == 0u && c0 + 16 <= N && x + 16 <= G.nx && !relabel) {
            const uint4 u = *(const uint4 *)(D.bub + c0), v = *(const uint4 *)(D.bub + c0 + 8);
            const unsigned id2 = (u.x & 0xffffu) * 0x10001u;
            if (((u.x ^ id2) | (u.y ^ id2) | (u.z ^ id2) | (u.w ^ id2) | (v.x ^ id2) | (v.y ^ id2) | (v.z ^ id2) |
                 (v.w ^ id2)) == 0u) {
                const int id = (int)(id2 & 0xffffu);
                const int b = id < nb ? L.root[id] : 0;
                if (b != bc) {
                    flush();
                    bc = b;
                }
                a0 += 16.0;
                a1 += 16.0 * x + 120.0;
                a2 += 16.0 * y;
                a3 += 16.0 * z;
                a4 += 16.0;
                continue;
            }
        }
        // all loads of the chunk first (the fields reach beyond the last cell to a multiple
        // of 256), then the cells in turn
        const uint32_t wds[4] = {f4.x, f4.y, f4.z, f4.w};
        const uint4 u = *(const uint4 *)(D.bub + c0), v = *(const uint4 *)(D.bub + c0 + 8);
        const uint32_t ids[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
        double ph[16];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            ph[k] = ((wds[k >> 2] >> (8 * (k & 3))) & 0xffu) == IFC && c0 + k < N ? phi[c0 + k] : 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k, ++x) {
            if (x == G.nx) {
                x = 0;
                if (++y == G.ny) {
                    y = 0;
                    ++z;
                }
            }
            const long long c = c0 + k;
            if (c >= N) break;
            const uint32_t f = (wds[k >> 2] >> (8 * (k & 3))) & 0xffu;
            if (f != GAS && f != IFC) continue;
            const int id = (int)((ids[k >> 1] >> (16 * (k & 1))) & 0xffffu);
            const int b = id < nb ? L.root[id] : 0;
            if (relabel && id != b) D.bub[c] = (uint16_t)b;
            if (b != bc) {
                flush();
                bc = b;
            }
            const double w = (f == GAS) ? 1.0 : 1.0 - ph[k];
            a0 += w;
            a1 += w * x;
            a2 += w * y;
            a3 += w * z;
            if (f == GAS) a4 += 1.0;
            else a5 += 1.0;
        }
    }
    // a wave whose lanes ended on one bubble sums first (64 lanes on one LDS address would
    // queue)
    const unsigned long long holds = __ballot(bc >= 0);
    if (holds) {
        const int b0 = __builtin_amdgcn_readlane(bc, __ffsll((long long)holds) - 1);
        if (__ballot(bc >= 0 && bc != b0) == 0ull) {
            a0 = wave_sum(a0);
            a1 = wave_sum(a1);
            a2 = wave_sum(a2);
            a3 = wave_sum(a3);
            a4 = wave_sum(a4);
            a5 = wave_sum(a5);
            bc = lane_id() == 0 ? b0 : -1;
        }
    }
    flush();
    __syncthreads();
    for (int i = threadIdx.x; i < nb * BACC_STRIDE; i += blockDim.x)
        if (L.acc[i] != 0.0) unsafeAtomicAdd(D.bacc + i, L.acc[i]);
}

// rho_g = M / V for every root bubble; per-id FP32 mirror for the boundary condition.
// With init set, the gas densities of the initial state are read from the table's density
// slot and the constant gas masses M = rho_g V(0) are fixed.  open: bubble 0 is a pressure
// outlet, held at the density in its table slot (the initial rho_g0) with its mass
// following its volume.  One block; the sums are cleared for the next pass.
__device__ __forceinline__ void bubble_finalize(const Dev &D, int init, int open) {
    for (int b = threadIdx.x; b < D.nb; b += blockDim.x) {
        double *t = D.btab + b * B_STRIDE;
        double a[BACC_STRIDE];
#pragma unroll
        for (int k = 0; k < BACC_STRIDE; ++k) {
            a[k] = __hip_atomic_load(D.bacc + b * BACC_STRIDE + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            D.bacc[b * BACC_STRIDE + k] = 0.0;
        }
        if (init) {
            t[B_M] = t[B_RHO] * a[0];
            t[B_V0] = a[0];
            D.balive[b] = a[0] > 0.0;
            D.broot[b] = b;
        }
        if (D.broot[b] != b) continue;
        t[B_V] = a[0];
        t[B_NGAS] = a[4];
        t[B_NIF] = a[5];
        if (!D.balive[b]) continue;
        const bool outlet = b == 0 && open;
        if (outlet) t[B_M] = t[B_RHO] * a[0];
        if (a[0] > 0.0) {
            if (!outlet) t[B_RHO] = t[B_M] / a[0];
            t[B_C] = a[1] / a[0];
            t[B_C + 1] = a[2] / a[0];
            t[B_C + 2] = a[3] / a[0];
        } else if (t[B_M] > 0.0) {
            // a bubble whose gas volume has vanished no longer exists; its gas mass
            // leaves (the liquid mass ledger is not involved)
            D.balive[b] = 0;
            t[B_M] = 0.0;
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < D.nb; b += blockDim.x)
        D.rhog[b] = (float)D.btab[bubble_root(D, b) * B_STRIDE + B_RHO];
}

// ---- surface tension: interface curvature (end of Sec. 2.2) ----------------------
// The fill level as the curvature sees it: liquid and particle nodes 1 (perfect
// wetting), gas 0, interface cells their fill level; a position beyond a wall takes
// the nearest cell inside the box, a periodic one wraps (k_curv_tiles).

// Parker-Youngs weighted central differences over the 3x3x3 block: a cell displaced
// along the axis of the derivative counts 4, 2 or 1 for 0, 1 or 2 nonzero
// transverse offsets (sum 16, distance 2)
__device__ __forceinline__ double st_w(int a, int b) {
    return (a == 0 && b == 0) ? 4.0 : ((a == 0 || b == 0) ? 2.0 : 1.0);
}
// kappa = -(1/2) div(n/|n|) at every interface cell: the mean curvature, so that
// 2 sigma kappa is the Laplace jump (a gas bubble of radius R has kappa = -1/R).
//
// Worked in tiles of KTX x KTY cells of one plane.  A marking pass lists the tiles
// that hold interface cells; the curvature pass stages the fill levels of a listed
// tile with a two-cell halo in LDS, forms the gradient of every cell of the tile
// and a one-cell halo once, and takes the divergence at the tile's interface cells
// (in the order of the per-cell definition, so the result is the same).
constexpr int KTX = 32, KTY = 8;
constexpr int KFX = KTX + 4, KFY = KTY + 4, KFZ = 5;  // staged fill levels
constexpr int KNX = KTX + 2, KNY = KTY + 2, KNZ = 3;  // gradients and their norms

// every tile with an interface cell enters the list once (tflag is zero for all
// tiles on entry; the curvature pass clears the flags of the tiles it takes)
__global__ __launch_bounds__(256) void k_curv_mark(Geom G, Dev D, unsigned *tflag, int *tlist, int *count,
                                                   int ktx, int kty) {
    const long long N = G.N;
    const long long nchunk = (N + 15) / 16;
    for (long long ch = blockIdx.x * (long long)blockDim.x + threadIdx.x; ch < nchunk;
         ch += (long long)gridDim.x * blockDim.x) {
        const long long c0 = ch * 16;
        const uint4 f4 = *(const uint4 *)(D.flags + c0);
        const uint32_t wds[4] = {f4.x, f4.y, f4.z, f4.w};
        uint32_t any = 0;  // interface is the type with bit 1 set and bit 0 clear
#pragma unroll
        for (int k = 0; k < 4; ++k) any |= (wds[k] >> 1) & ~wds[k] & 0x01010101u;
        if (!any) continue;
        int x = (int)(c0 % G.nx);
        const int yz = (int)(c0 / G.nx);
        int y = yz % G.ny, z = yz / G.ny;
        int last = -1;
        for (int e = 0; e < 16 && c0 + e < N; ++e, ++x) {
            if (x == G.nx) {
                x = 0;
                if (++y == G.ny) {
                    y = 0;
                    ++z;
                }
            }
            if (((wds[e >> 2] >> (8 * (e & 3))) & 0xffu) != IFC) continue;
            const int t = (z * kty + y / KTY) * ktx + x / KTX;
            if (t == last) continue;
            last = t;
            if (atomicExch(tflag + t, 1u) == 0u) tlist[atomicAdd(count, 1)] = t;
        }
    }
}

// a staged coordinate: wrapped on a periodic axis (the halo may reach past the box
// more than once in a short axis), the nearest cell inside beyond a wall
__device__ __forceinline__ int kc_wrap(int v, int n, int per) {
    if (per) {
        v %= n;
        return v < 0 ? v + n : v;
    }
    return v < 0 ? 0 : (v >= n ? n - 1 : v);
}

// LDS index of the point whose gradient stands for position v of the one-cell halo:
// beyond a wall the nearest cell inside (the per-cell definition clamps the
// position first); on a periodic axis v itself, since the staged fill levels are
// already wrapped
__device__ __forceinline__ int kc_pos(int v, int n, int per, int origin) {
    if (!per) v = v < 0 ? 0 : (v >= n ? n - 1 : v);
    return v - origin;
}

__global__ __launch_bounds__(256) void k_curv_tiles(Geom G, Dev D, const double *phi, unsigned *tflag,
                                                    const int *tlist, const int *count, int ktx, int kty) {
    __shared__ double F[KFZ][KFY][KFX];
    __shared__ double NG[4][KNZ][KNY][KNX];  // gradient components and norm
    const int nt = *count;
    for (int it = blockIdx.x; it < nt; it += gridDim.x) {
        const int t = tlist[it];
        const int x0 = (t % ktx) * KTX, y0 = ((t / ktx) % kty) * KTY, z = t / (ktx * kty);
        // the tile's cell types in one batch of loads, the interface cells' fill levels in a
        // second (a loop over the elements paid both latencies nine times)
        constexpr int NF = KFX * KFY * KFZ, K = (NF + 255) / 256;
        int ce[K];
        uint8_t fe[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = min((int)threadIdx.x + 256 * k, NF - 1);
            const int ex = e % KFX, ey = (e / KFX) % KFY, ez = e / (KFX * KFY);
            ce[k] = kc_wrap(x0 - 2 + ex, G.nx, G.per[0]) +
                    G.nx * (kc_wrap(y0 - 2 + ey, G.ny, G.per[1]) + G.ny * kc_wrap(z - 2 + ez, G.nz, G.per[2]));
            fe[k] = D.flags[ce[k]];
        }
        double ve[K];
#pragma unroll
        for (int k = 0; k < K; ++k) ve[k] = fe[k] == GAS ? 0.0 : fe[k] == IFC ? phi[ce[k]] : 1.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = (int)threadIdx.x + 256 * k;
            if (e < NF) (&F[0][0][0])[e] = ve[k];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < KNX * KNY * KNZ; e += blockDim.x) {
            const int ex = e % KNX, ey = (e / KNX) % KNY, ez = e / (KNX * KNY);
            const int px = kc_pos(x0 - 1 + ex, G.nx, G.per[0], x0 - 2);
            const int py = kc_pos(y0 - 1 + ey, G.ny, G.per[1], y0 - 2);
            const int pz = kc_pos(z - 1 + ez, G.nz, G.per[2], z - 2);
            double n0 = 0.0, n1 = 0.0, n2 = 0.0;
            for (int dz = -1; dz <= 1; ++dz)
                for (int dy = -1; dy <= 1; ++dy)
                    for (int dx = -1; dx <= 1; ++dx) {
                        if (!dx && !dy && !dz) continue;
                        const double v = F[pz + dz][py + dy][px + dx];
                        if (dx) n0 += dx * st_w(dy, dz) * v;
                        if (dy) n1 += dy * st_w(dx, dz) * v;
                        if (dz) n2 += dz * st_w(dx, dy) * v;
                    }
            n0 *= 1.0 / 32.0;
            n1 *= 1.0 / 32.0;
            n2 *= 1.0 / 32.0;
            NG[0][ez][ey][ex] = n0;
            NG[1][ez][ey][ex] = n1;
            NG[2][ez][ey][ex] = n2;
            NG[3][ez][ey][ex] = sqrt(n0 * n0 + n1 * n1 + n2 * n2);
        }
        __syncthreads();
        for (int e = threadIdx.x; e < KTX * KTY; e += blockDim.x) {
            const int lx = e % KTX, ly = e / KTX;
            const int x = x0 + lx, y = y0 + ly;
            if (x >= G.nx || y >= G.ny) continue;
            const long long c = x + (long long)G.nx * (y + (long long)G.ny * z);
            if (D.flags[c] != IFC) continue;
            double div = 0.0;
            for (int dz = -1; dz <= 1; ++dz)
                for (int dy = -1; dy <= 1; ++dy)
                    for (int dx = -1; dx <= 1; ++dx) {
                        if (!dx && !dy && !dz) continue;
                        const int a = 1 + lx + dx, b = 1 + ly + dy, d = 1 + dz;
                        const double nn = NG[3][d][b][a];
                        if (nn == 0.0) continue;
                        if (dx) div += dx * st_w(dy, dz) * NG[0][d][b][a] / nn;
                        if (dy) div += dy * st_w(dx, dz) * NG[1][d][b][a] / nn;
                        if (dz) div += dz * st_w(dx, dy) * NG[2][d][b][a] / nn;
                    }
            D.kappa[c] = (float)(-0.5 * div / 32.0);
        }
        if (threadIdx.x == 0) tflag[t] = 0u;
        __syncthreads();
    }
}

}  // namespace fsl
