// Bubble splitting (bubble model, end of Sec. 2.2): a bubble is a connected region of
// gas, so a bubble whose gas falls apart becomes several bubbles.
//
// Two gas cells are connected when they are D3Q19 neighbours (the neighbourhood of
// the merge rule) and belong to the same root bubble.  Where the gas of a root falls
// into several parts, the part holding the lowest cell index keeps the bubble and
// the others, in order of their lowest cell index, take the lowest ids that are not
// alive (merges relabel the cells to their roots, so merged ids are free); an
// interface cell goes with the part of its gas neighbours (the lowest when they
// differ) and stays with the bubble without any; the gas mass is shared in
// proportion to the parts' volumes (gas cells plus 1 - phi of their interface
// cells), so that every part starts at the density of its bubble.
//
// The gas of a bubble can only come apart in a step where gas cells leave the gas
// phase (new interface cells, cells covered by a particle), where cells enter it
// (emptied cells, cells uncovered as gas) or where bubbles merge.  A cell that left
// is tested on its 3x3x3 block, a cell that entered must touch older gas of its
// bubble, and a merge always asks for labelling; only then does a union-find
// labelling of all gas cells run.  The tests are exact given that every root's gas
// was connected before the step, which the labelling establishes at initialisation
// and whenever tables or particles are set.
#pragma once

#include "k_particles.hpp"
#include "split_block.hpp"

namespace fsl {

constexpr int SPLIT_MAXC = 1024;  // gas components one labelling may list

struct SplitBuf {
    int *lab;     // per gas cell: union-find link, then the part's lowest cell index;
                  // at that cell, -(slot + 2) once the parts are numbered
    int *comp;    // lowest cell index of each part, in discovery order
    int *cid;     // per slot (parts by lowest cell index): new bubble id, -1 = keeps its id
    int *parent;  // per slot: root bubble
    double *vol;  // per slot: volume of a part that takes a new id
};

// ---- local test on the 3x3x3 block ------------------------------------------------
__device__ __forceinline__ int blk_cell(const Geom &G, int x, int y, int z, int dx, int dy, int dz) {
    int a = x + dx, b = y + dy, d = z + dz;
    if (a < 0 || a >= G.nx) { if (!G.per[0]) return -1; a = wrapc(a, G.nx); }
    if (b < 0 || b >= G.ny) { if (!G.per[1]) return -1; b = wrapc(b, G.ny); }
    if (d < 0 || d >= G.nz) { if (!G.per[2]) return -1; d = wrapc(d, G.nz); }
    return a + G.nx * (b + G.ny * d);
}

// the step's cells that left the gas (new interface cells from gas, covered gas
// cells: CV_GRM) and that entered it (emptied cells, cells uncovered as gas: CV_GAD),
// taken from the step's lists in that order
__device__ __forceinline__ int split_cell(const Dev &D, int i, int nG, int nC, int nE) {
    if (i < nG) return D.lNG[i];
    i -= nG;
    if (i < nC) return D.lCov[2 * i];
    i -= nC;
    if (i < nE) return D.lE[i];
    return D.lUnc[2 * (i - nE)];
}

// A failed test or a merge in this step asks for labelling.  A cell is worked by 32 lanes,
// lane b taking cell b of its 3x3x3 block (one thread per cell paid the latency of 26
// neighbours in turn: 40 us on the 384 x 256 surface).  Cell left the gas phase: its
// block's gas and removed cells of its root, tested by split_block_ok.  Cell entered it: it
// joins the older gas of its root (gas before the step and still gas) through a D3Q19
// neighbour.  root: the block's table of bubble roots.
__device__ __forceinline__ void split_test(const Geom &G, const Dev &D, const int *root, const Items &W) {
    const int nG = list_len(D, C_NNG), nC = event_len(D, C_NCOVER);
    const int nE = list_len(D, C_NE), nU = event_len(D, C_NUNCOVER);
    // a periodic axis shorter than the block folds it onto itself: always label
    const bool fold = (G.per[0] && G.nx < 3) || (G.per[1] && G.ny < 3) || (G.per[2] && G.nz < 3);
    if (blockIdx.x == 0 && threadIdx.x == 0 && D.counters[C_NMERGE] > 0) atomicOr(D.counters + C_SPLIT, 1);
    const int n = nG + nC + nE + nU;
    auto root_of = [&](int c) {
        const int id = D.bub[c];
        return id < D.nb ? root[id] : 0;
    };
    ITEM_LOOP(W, i, n) {
        const bool has = i < n;
        const int c = has ? split_cell(D, i, nG, nC, nE) : 0;
        const uint8_t m = has ? D.cv[c] : 0;
        const int q = W.q;
        int nb = -1;
        if ((m & (CV_GRM | CV_GAD)) && q < 27 && q != 13) {
            int x, y, z;
            cell_xyz(G, c, x, y, z);
            nb = blk_cell(G, x, y, z, q % 3 - 1, (q / 3) % 3 - 1, q / 9 - 1);
        }
        bool gas = false, old = false, rem = false;
        if (nb >= 0) {
            const uint8_t f = D.flags[nb], v = D.cv[nb];
            if ((f == GAS || (v & CV_GRM)) && root_of(nb) == root_of(c)) {
                gas = f == GAS;
                old = gas && !(v & CV_GAD);
                rem = !gas;
            }
        }
        const unsigned mg = W.any(gas), mo = W.any(old), mr = W.any(rem);
        bool ok = true;
        if (m & CV_GRM) ok = !fold && split_block_ok(mg, mr);
        else if (m & CV_GAD) ok = (mo & blk_step(1u << 13)) != 0u;
        if (has && !ok && q == 0) atomicOr(D.counters + C_SPLIT, 1);
    }
}

// The bubble pass of a step in one launch: volumes, the splitting test, and in the block
// that finishes last the gas densities.  (Clearing, summing and finishing the table took
// three launches, the test a fourth.)
__global__ __launch_bounds__(256) void k_bubbles(Geom G, Dev D, const double *phi, int init, int test, int open) {
    __shared__ BubbleLds L;
    bubble_accum(G, D, phi, L, D.counters[C_MERGED] != 0);
    if (test) split_test(G, D, L.root, Items(blockIdx.x, gridDim.x));
    if (last_block<false>(D.counters + C_DONEB, gridDim.x)) bubble_finalize(D, init, open);
}

// ---- labelling: union-find over the gas cells -------------------------------------
// Links only ever point to a lower cell index, so every part ends at its lowest cell.
__device__ __forceinline__ int lab_get(const int *lab, int x) {
    return __hip_atomic_load(lab + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int lab_find(const int *lab, int x) {
    for (;;) {
        const int p = lab_get(lab, x);
        if (p == x) return x;
        x = p;
    }
}

// join the parts of a and b: the higher root is linked below the lower one; a root
// relinked by another thread meanwhile is followed and joined in turn (the larger of
// the two indices falls every round, so this ends)
__device__ void lab_unite(int *lab, int a, int b) {
    for (;;) {
        a = lab_find(lab, a);
        b = lab_find(lab, b);
        if (a == b) return;
        if (a < b) {
            const int t = a;
            a = b;
            b = t;
        }
        const int old = atomicMin(lab + a, b);
        if (old == a) return;
        a = old;
    }
}

// a range of cells for thread `thread` of `nthreads`
#define CELL_RANGE(c, n) for (long long c = T.thread; c < (n); c += T.nthreads)
struct Threads {
    long long thread, nthreads;
};

// clears the marks the test read (cv is zero outside the conversion phase)
__device__ __forceinline__ void split_clear(const Dev &D, const Threads &T) {
    const int nG = list_len(D, C_NNG), nC = event_len(D, C_NCOVER);
    const int nE = list_len(D, C_NE), nU = event_len(D, C_NUNCOVER);
    CELL_RANGE(i, nG + nC + nE + nU) D.cv[split_cell(D, (int)i, nG, nC, nE)] = 0;
}

// starts the labelling: every gas cell its own part
__device__ __forceinline__ void ccl_init(const Geom &G, const Dev &D, const SplitBuf &B, const Threads &T) {
    CELL_RANGE(c, G.N) if (D.flags[c] == GAS) B.lab[c] = (int)c;
}

__device__ __forceinline__ void ccl_union(const Geom &G, const Dev &D, const SplitBuf &B, const Threads &T) {
    CELL_RANGE(c, G.N) {
        if (D.flags[c] != GAS) continue;
        int x, y, z;
        cell_xyz(G, (int)c, x, y, z);
        const int r = bubble_root(D, D.bub[c]);
        for (int q = 1; q < Q; ++q) {
            if (opp(q) < q) continue;  // one direction of each pair
            const int n = nbr_idx(G, x, y, z, q, 1);
            if (n < 0 || D.flags[n] != GAS || bubble_root(D, D.bub[n]) != r) continue;
            lab_unite(B.lab, (int)c, n);
        }
    }
}

// every gas cell links straight to its part's lowest cell (a concurrent find only
// ever sees a link to an ancestor); the parts' lowest cells are listed
__device__ __forceinline__ void ccl_flatten(const Geom &G, const Dev &D, const SplitBuf &B, const Threads &T) {
    CELL_RANGE(c, G.N) {
        if (D.flags[c] != GAS) continue;
        const int root = lab_find(B.lab, (int)c);
        if (root != (int)c) {
            __hip_atomic_store(B.lab + c, root, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            continue;
        }
        const int s = atomicAdd(D.counters + C_NCOMP, 1);
        if (s < SPLIT_MAXC) B.comp[s] = (int)c;
        else atomicOr(D.err, ERR_CAP);
    }
}

struct PlanLds {
    int sorted[SPLIT_MAXC];
    unsigned char seen[64], taken[64];
};

// parts in order of their lowest cell index: the first part of each root keeps it,
// the others take the lowest ids that are not alive.  One block.
__device__ __forceinline__ void split_plan(const Dev &D, const SplitBuf &B, PlanLds &P, int open) {
    const int n = __hip_atomic_load(D.counters + C_NCOMP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n > SPLIT_MAXC) {  // not every part listed: no split, error set
        if (threadIdx.x == 0) D.counters[C_SPLIT] = 1;
        return;
    }
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const int v = B.comp[k];
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += B.comp[j] < v;
        P.sorted[rank] = v;
    }
    for (int i = threadIdx.x; i < 64; i += blockDim.x) P.seen[i] = P.taken[i] = 0;
    __syncthreads();
    if (threadIdx.x) return;
    int used = *D.bused, any = 0;
    for (int k = 0; k < n; ++k) {
        const int c = P.sorted[k];
        const int r = bubble_root(D, D.bub[c]);
        int id = -1;
        if (r == 0 && open) {
            // every part of an open atmosphere stays at the outlet
        } else if (!P.seen[r]) {
            P.seen[r] = 1;
        } else {
            // the lowest id that is not alive: never used, or merged away (merges
            // relabel the cells to their roots)
            int b = 1;
            while (b < D.maxB && (D.balive[b] || P.taken[b])) ++b;
            if (b < D.maxB) {
                id = b;
                P.taken[b] = 1;
                used = max(used, b + 1);
                any = 1;
            } else {
                atomicOr(D.err, ERR_CAP);
            }
        }
        B.cid[k] = id;
        B.parent[k] = r;
        B.vol[k] = 0.0;
        B.lab[c] = -(k + 2);
    }
    *D.bused = used;
    D.counters[C_SPLIT] = any ? 2 : 1;
}

__device__ __forceinline__ int lab_slot(const int *lab, int c) {
    const int l = lab[c];
    return l < 0 ? -l - 2 : -lab[l] - 2;
}

// interface cells first: they find their part through the ids of their gas
// neighbours, which the next phase changes
__device__ __forceinline__ void split_ifc(const Geom &G, const Dev &D, const SplitBuf &B, const double *phi,
                                          const Threads &T) {
    CELL_RANGE(c, G.N) {
        if (D.flags[c] != IFC) continue;
        int x, y, z;
        cell_xyz(G, (int)c, x, y, z);
        const int r = bubble_root(D, D.bub[c]);
        int best = -1;
        for (int q = 1; q < Q; ++q) {
            const int n = nbr_idx(G, x, y, z, q, 1);
            if (n < 0 || D.flags[n] != GAS || bubble_root(D, D.bub[n]) != r) continue;
            const int l = B.lab[n];
            const int rep = l < 0 ? n : l;
            if (best < 0 || rep < best) best = rep;
        }
        if (best < 0) continue;
        const int k = -B.lab[best] - 2;
        const int id = B.cid[k];
        if (id < 0) continue;
        D.bub[c] = (uint16_t)id;
        unsafeAtomicAdd(B.vol + k, 1.0 - phi[c]);
    }
}

// gas cells: 16 consecutive cells per thread, their count summed per part
__device__ __forceinline__ void split_gas(const Geom &G, const Dev &D, const SplitBuf &B, const Threads &T) {
    const long long nchunk = (G.N + 15) / 16;
    int ks = -1;
    double acc = 0.0;
    CELL_RANGE(ch, nchunk) {
        for (long long c = ch * 16; c < ch * 16 + 16 && c < G.N; ++c) {
            if (D.flags[c] != GAS) continue;
            const int k = lab_slot(B.lab, (int)c);
            const int id = B.cid[k];
            if (id < 0) continue;
            D.bub[c] = (uint16_t)id;
            if (k != ks) {
                if (ks >= 0) unsafeAtomicAdd(B.vol + ks, acc);
                ks = k;
                acc = 0.0;
            }
            acc += 1.0;
        }
    }
    if (ks >= 0) unsafeAtomicAdd(B.vol + ks, acc);
}

struct MassLds {
    double Mr[64], taken[64];
};

// gas masses of the new bubbles: M_part = M_root V_part / V_root, the root keeps
// the rest (the root volumes are those of the state before the split).  One thread.
__device__ __forceinline__ void split_mass(const Dev &D, const SplitBuf &B, MassLds &S) {
    for (int r = 0; r < D.maxB; ++r) {
        S.Mr[r] = D.btab[r * B_STRIDE + B_M];
        S.taken[r] = 0.0;
    }
    const int n = min(__hip_atomic_load(D.counters + C_NCOMP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), SPLIT_MAXC);
    for (int k = 0; k < n; ++k) {
        const int id = B.cid[k];
        if (id < 0) continue;
        const int r = B.parent[k];
        double *t = D.btab + id * B_STRIDE;
        const double v = __hip_atomic_load(B.vol + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        t[B_M] = S.Mr[r] * v / D.btab[r * B_STRIDE + B_V];
        t[B_V0] = v;
        D.broot[id] = id;
        D.balive[id] = 1;
        S.taken[r] += t[B_M];
    }
    for (int r = 0; r < D.maxB; ++r)
        if (S.taken[r] != 0.0) D.btab[r * B_STRIDE + B_M] = S.Mr[r] - S.taken[r];
}

// The labelling and the split in one launch (small boxes, where six more launches cost more
// than the step has to spare): the blocks return after clearing the marks when there is
// nothing to do.
__global__ __launch_bounds__(256) void k_split(Geom G, Dev D, SplitBuf B, const double *phi, int open) {
    __shared__ union {
        PlanLds P;
        MassLds S;
        BubbleLds V;
    } L;
    const Threads T{blockIdx.x * (long long)blockDim.x + threadIdx.x, (long long)gridDim.x * blockDim.x};
    const bool run = D.counters[C_SPLIT] != 0;
    split_clear(D, T);
    if (!run) return;
    GridBarrier GB{D.counters + C_BARS, (int)gridDim.x, 0, D.err};
    ccl_init(G, D, B, T);
    GB.wait();
    ccl_union(G, D, B, T);
    GB.wait();
    ccl_flatten(G, D, B, T);
    GB.wait();
    if (blockIdx.x == 0) split_plan(D, B, L.P, open);
    GB.wait();
    if (__hip_atomic_load(D.counters + C_SPLIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 2) return;
    split_ifc(G, D, B, phi, T);
    GB.wait();
    split_gas(G, D, B, T);
    GB.wait();
    if (blockIdx.x == 0 && threadIdx.x == 0) split_mass(D, B, L.S);
    GB.wait();
    bubble_accum(G, D, phi, L.V, false);
    if (last_block(D.counters + C_DONES, gridDim.x)) bubble_finalize(D, 0, open);
}

// The same as a launch per phase, for boxes where the labelling wants the whole device (a
// phase of a few values goes to the block that finishes the one before it); each returns
// at once when there is nothing to do.  force: label regardless of the test (initial state,
// new tables or particles).
__global__ void k_split_start(Geom G, Dev D, SplitBuf B, int force) {
    const Threads T{blockIdx.x * (long long)blockDim.x + threadIdx.x, (long long)gridDim.x * blockDim.x};
    split_clear(D, T);
    if (force || D.counters[C_SPLIT] != 0) ccl_init(G, D, B, T);
}
__global__ void k_ccl_union(Geom G, Dev D, SplitBuf B, int force) {
    if (!force && D.counters[C_SPLIT] == 0) return;
    ccl_union(G, D, B, Threads{blockIdx.x * (long long)blockDim.x + threadIdx.x, (long long)gridDim.x * blockDim.x});
}
__global__ __launch_bounds__(256) void k_ccl_flatten(Geom G, Dev D, SplitBuf B, int force, int open) {
    __shared__ PlanLds P;
    if (!force && D.counters[C_SPLIT] == 0) return;
    ccl_flatten(G, D, B, Threads{blockIdx.x * (long long)blockDim.x + threadIdx.x, (long long)gridDim.x * blockDim.x});
    if (last_block(D.counters + C_DONES, gridDim.x)) split_plan(D, B, P, open);
}
__global__ void k_split_ifc(Geom G, Dev D, SplitBuf B, const double *phi) {
    if (D.counters[C_SPLIT] != 2) return;
    split_ifc(G, D, B, phi, Threads{blockIdx.x * (long long)blockDim.x + threadIdx.x, (long long)gridDim.x * blockDim.x});
}
__global__ __launch_bounds__(256) void k_split_gas(Geom G, Dev D, SplitBuf B) {
    __shared__ MassLds S;
    if (D.counters[C_SPLIT] != 2) return;
    split_gas(G, D, B, Threads{blockIdx.x * (long long)blockDim.x + threadIdx.x, (long long)gridDim.x * blockDim.x});
    if (last_block(D.counters + C_DONES, gridDim.x) && threadIdx.x == 0) split_mass(D, B, S);
}
__global__ __launch_bounds__(256) void k_split_volumes(Geom G, Dev D, const double *phi, int open) {
    __shared__ BubbleLds L;
    if (D.counters[C_SPLIT] != 2) return;
    bubble_accum(G, D, phi, L, false);
    if (last_block(D.counters + C_DONES, gridDim.x)) bubble_finalize(D, 0, open);
}

}  // namespace fsl
