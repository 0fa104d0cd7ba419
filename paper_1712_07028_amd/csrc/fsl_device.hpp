// fsl_device.hpp -- device-side definitions of the free-surface LBM library:
// D3Q19 velocity set, population storage formats, workspace pointers and the
// wave-level helpers shared by the kernels.  gfx950 (CDNA4), wave64.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fsl {

// ---- D3Q19 (Sec. 2.1): rest, six axis directions, twelve diagonals -------------
// Order: 0 rest; 1..6 +x,-x,+y,-y,+z,-z; 7..18 (+-1,+-1,0),(+-1,0,+-1),(0,+-1,+-1)
// with sign pairs (+,+),(+,-),(-,+),(-,-).
constexpr int Q = 19;
__host__ __device__ constexpr int cx(int q) {
    constexpr int v[Q] = {0, 1, -1, 0, 0, 0, 0, 1, 1, -1, -1, 1, 1, -1, -1, 0, 0, 0, 0};
    return v[q];
}
__host__ __device__ constexpr int cy(int q) {
    constexpr int v[Q] = {0, 0, 0, 1, -1, 0, 0, 1, -1, 1, -1, 0, 0, 0, 0, 1, 1, -1, -1};
    return v[q];
}
__host__ __device__ constexpr int cz(int q) {
    constexpr int v[Q] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1};
    return v[q];
}
__host__ __device__ constexpr int opp(int q) {
    constexpr int v[Q] = {0, 2, 1, 4, 3, 6, 5, 10, 9, 8, 7, 14, 13, 12, 11, 18, 17, 16, 15};
    return v[q];
}

__host__ __device__ constexpr float wq(int q) {
    return q == 0 ? 1.0f / 3.0f : (q <= 6 ? 1.0f / 18.0f : 1.0f / 36.0f);
}
__host__ __device__ constexpr double wqd(int q) {
    return q == 0 ? 1.0 / 3.0 : (q <= 6 ? 1.0 / 18.0 : 1.0 / 36.0);
}

// cell types
constexpr uint8_t GAS = 0, LIQ = 1, IFC = 2, SOL = 3, WALL = 4;

// device error bits (latched, reported by the host at the next sync)
constexpr unsigned ERR_LG = 1u, ERR_NAN = 2u, ERR_CAP = 4u, ERR_VOL = 8u;
// a sphere centre left the box, or came closer than R + 1 to a periodic face (the
// coverage, pair search and lever arms do not wrap)
constexpr unsigned ERR_PART = 16u;
// a grid barrier gave up (the blocks of one launch did not come to run together)
constexpr unsigned ERR_SYNC = 32u;

// conversion marks (one byte per cell, zero outside the conversion phase)
constexpr uint8_t CV_F = 1, CV_E0 = 2, CV_E = 4, CV_NEWG = 8, CV_NEWL = 16;
// a gas cell that left the gas phase in this step (became interface or was covered);
// set until the splitting test at the end of the step
constexpr uint8_t CV_GRM = 32;
// a cell that entered the gas phase in this step (emptied or uncovered as gas)
constexpr uint8_t CV_GAD = 64;
// a node that its sphere leaves in this step, until its new state is decided
constexpr uint8_t CV_UNC = 128;

// counters in the control block
enum Counter {
    C_NF = 0, C_NE0, C_NE, C_NNG, C_NNL, C_NMERGE, C_NCOVER, C_NUNCOVER, C_NPAIRS, C_COVALL,
    C_SPLIT,  // splitting pass: 1 = label the gas, 2 = some bubble splits
    C_NCOMP,  // gas components listed by the splitting pass
    C_MERGED, // some bubbles merged in this step: cells are relabelled to their roots
    C_NGEN,   // tiles listed for the general path of the stream-collide step
    C_NKT,    // tiles listed for the curvature
    C_BAR,    // arrivals at the grid barriers of the fused conversion phases
    C_BARS,   // ... of the fused labelling
    C_BARU,   // ... of the uncover pass
    C_DONEC,  // blocks of the last conversion phase that are done
    C_DONEB,  // blocks of the bubble pass that are done
    C_NUGAS,  // some node was uncovered as gas
    C_DONES,  // blocks of a splitting phase that are done
    C_COUNT
};
// Two sets of counters take turns: a step uses one and its first kernel clears the
// other for the next step, so that clearing costs no launch.  The persistent word after
// them (not cleared per step) is the number of bubble ids in use.
constexpr int C_SET = 48, C_BUSED = 127, C_WORDS = 128;
static_assert(C_COUNT <= C_SET && 2 * C_SET <= C_BUSED, "counter sets");

// particle table: 16 doubles per particle
// P_OVL: 1 when the coverage update must resolve overlaps through claims (a sphere
// within one cell of another, or one that moved half a cell or more in a step)
enum PSlot { P_X = 0, P_U = 3, P_W = 6, P_R = 9, P_RHO = 10, P_XOLD = 11, P_OVL = 14, P_STRIDE = 16 };
// particle accumulators: F(3) T(3) dm(1) pad -> 8 doubles
constexpr int ACC_STRIDE = 8;
// copies of each particle's accumulator: the waves that touch one sphere add into
// different copies (by block), so their FP64 atomics do not queue on one cache line;
// the force pass sums the copies in a fixed order
constexpr int ACC_COPIES = 8;
__host__ __device__ constexpr long long acc_at(int P, int copy) {
    return ((long long)P * ACC_COPIES + copy) * ACC_STRIDE;
}
// bubble table: 16 doubles per id
enum BSlot { B_M = 0, B_V = 1, B_RHO = 2, B_C = 3, B_V0 = 6, B_NGAS = 7, B_NIF = 8, B_STRIDE = 16 };
// bubble accumulators: V, Vx, Vy, Vz, n_gas, n_iface
constexpr int BACC_STRIDE = 6;

// ---- population storage (form 1) ----------------------------------------------
// Populations are always stored shifted, h_q = f_q - w_q, so that density
// deviations of O(1e-3) never round at O(1).  FP32 stores h directly; the 16-bit
// formats store h * scale (a power of two) with round-to-nearest-even.
enum { ST_F32 = 0, ST_F16 = 1, ST_BF16 = 2 };

template <int S> struct Store;
// enc() gives the stored word, dec() the value it represents, so that the
// value a kernel will read back is known when it writes (rnd = dec(enc(v))).
template <> struct Store<ST_F32> {
    using T = float;
    static __device__ __forceinline__ T enc(float v, float) { return v; }
    static __device__ __forceinline__ float dec(T w, float) { return w; }
    static __device__ __forceinline__ float ld(const T *p, float inv) { return dec(*p, inv); }
    static __device__ __forceinline__ void st(T *p, float v, float sc) { *p = enc(v, sc); }
};
template <> struct Store<ST_F16> {
    using T = _Float16;
    static __device__ __forceinline__ T enc(float v, float sc) { return (_Float16)(v * sc); }
    static __device__ __forceinline__ float dec(T w, float inv) { return (float)w * inv; }
    static __device__ __forceinline__ float ld(const T *p, float inv) { return dec(*p, inv); }
    static __device__ __forceinline__ void st(T *p, float v, float sc) { *p = enc(v, sc); }
};
template <> struct Store<ST_BF16> {
    using T = uint16_t;
    static __device__ __forceinline__ T enc(float v, float sc) {
        uint32_t u = __float_as_uint(v * sc);
        if ((u & 0x7f800000u) != 0x7f800000u) u += 0x7fffu + ((u >> 16) & 1u);  // RNE
        return (uint16_t)(u >> 16);
    }
    static __device__ __forceinline__ float dec(T w, float inv) {
        return __uint_as_float(((uint32_t)w) << 16) * inv;
    }
    static __device__ __forceinline__ float ld(const T *p, float inv) { return dec(*p, inv); }
    static __device__ __forceinline__ void st(T *p, float v, float sc) { *p = enc(v, sc); }
};

// ---- geometry / parameters passed by value ------------------------------------
struct Geom {
    int nx, ny, nz;
    int per[3];
    long long N;  // cells
    long long S;  // plane stride of one population (>= N, multiple of 256)
};

struct Phys {
    float lp, lm;      // lambda_+, lambda_-
    float g[3];
    double eps;        // conversion threshold slack
    float scale, inv;  // 16-bit storage scale and its inverse
    float s6;          // 6 sigma: density form of the Laplace jump 2 sigma kappa (rho = 3 p)
    int moving_walls;  // some face moves (velocities in Dev::wallu) or slips: wall links
                       // then take the general path
    int slip[3];       // the faces of axis a are free-slip
    int open_atm;      // bubble 0 is held at its density (pressure outlet)
    int wide;          // offsets that leave 32 bits: 0 none, 1 the byte offset within a pair of
                       // opposite planes (below four planes; that of one plane and the pair's in
                       // elements fit), 2 the pair's in elements as well
};

struct Dev {
    void *fA, *fB;            // post-collision populations at t (A), next (B)
    uint8_t *flags, *cv;
    double *phi_cur, *phi_nxt, *m;
    uint16_t *bub;
    int *pid, *claim;
    int *lF, *lE0, *lE, *lNG, *lNL;  // conversion lists
    int *lCov, *lUnc;                // coverage events (cell, particle) pairs
    double *uncRho;                  // per uncover event: decided density
    int *uncDec;                     // per uncover event: the type decided
    int2 *merges, *pairs;
    int *counters, *counters_nxt;    // this step's set of counters and the next step's
    int *bused;                      // number of bubble ids in use
    unsigned *err;
    double *ledger;                  // [0] ledger
    double *wallF, *wallF_nxt;       // force on each no-slip face in this step [18], and the
                                     // next step's accumulator
    double *ptab, *pacc, *pFT, *pFTp, *pFl; // particles (pFTp: previous step's F, T)
    float4 *pmir;                    // FP32 mirror per particle (PMir: anchor, fraction, u, omega)
    int *gridStart, *gridCount, *gridIdx;
    double *btab, *bacc;
    int *broot, *balive;
    float *rhog;                     // FP32 gas density per bubble id (through root)
    float *kappa;                    // interface curvature (null without surface tension)
    float *wallu;                    // face velocities [axis][low, high][component]
    // density of every liquid and interface cell as computed from its populations by
    // the last launch (null without particles), for Eq. bbrule's rho_w in the next
    // launch: see rhow_word; a launch reads words of stamp st_prev and writes words of
    // stamp st_cur (< 0: none)
    unsigned *rhow;
    int st_prev, st_cur;
    int cap;                         // conversion list capacity
    int capEv;                       // coverage event list capacity
    int maxP, maxB;
    int np, nb;
};

// FP32 mirror of a particle for the kernels that need its rigid-body velocity at a node:
// anchor a = floor(x_P) (exact integers), fraction x_P - a, u_P, omega_P; 12 floats in
// the first three float4 of the particle's 64-byte record
struct PMir {
    float ax, ay, az, fx, fy, fz, ux, uy, uz, wx, wy, wz;
};
__device__ __forceinline__ PMir pmir_load(const float4 *pmir, int P) {
    const float4 *m = pmir + 4LL * P;
    const float4 a = m[0], b = m[1], c = m[2];
    return PMir{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w};
}

// The sphere positions the library handles: every component finite; on a
// non-periodic axis the centre inside the box (faces at -1/2 and n - 1/2); on a
// periodic axis anywhere (the centre is kept in [0, n) and the sphere acts through its
// nearest images), the axis longer than 2R + 4, so that every node within a link of
// the sphere lies less than n/2 from its centre and the sphere never meets its own
// image.
__host__ __device__ inline bool sphere_supported(const double x[3], double R, const int n[3], const int per[3]) {
    for (int a = 0; a < 3; ++a) {
        const double v = x[a];
        if (!(v == v) || v - v != 0.0) return false;  // NaN or infinite
        if (per[a]) {
            if (!(n[a] > 2.0 * R + 4.0)) return false;
        } else if (!(v >= -0.5 && v <= n[a] - 0.5)) {
            return false;
        }
    }
    return true;
}

// a coordinate along a periodic axis taken into [0, n)
__host__ __device__ inline double wrap_coord(double v, int n) {
    if (v >= 0.0 && v < n) return v;  // no division on the common path
    v -= n * floor(v / n);
    return v < n ? v : 0.0;  // v just below 0 can round up to n
}

// a displacement along an axis, the nearest image along a periodic one: [-n/2, n/2)
__host__ __device__ inline double min_img(double d, int n, int per) {
    if (!per || fabs(d) < 0.49 * n) return d;  // no division on the common path
    return d - n * floor(d / n + 0.5);
}

// lever arm x - x_P along one axis from the FP32 mirror: the integer part x - anchor
// taken to its nearest image along a periodic axis (exactly: it is an integer below n
// in size), minus the fraction
__device__ __forceinline__ float mirror_arm(int x, float anchor, float frac, int n, int per) {
    float d = (float)x - anchor;
    if (per) d -= (float)n * rintf(d / (float)n);
    return d - frac;
}

// Stored density word: the FP32 density with its lowest mantissa bit replaced by the
// parity of the stamp of the launch that wrote it (a change of at most one unit in the
// last place); RHOW_NONE (a NaN) where no density is held.  A reader takes the word
// only with the parity of the stamp it expects.
constexpr unsigned RHOW_NONE = 0x7fc00000u;
__device__ __forceinline__ unsigned rhow_word(float rho, int stamp) {
    return (__float_as_uint(rho) & ~1u) | (unsigned)(stamp & 1);
}
__device__ __forceinline__ bool rhow_valid(unsigned w, int stamp) {
    return stamp >= 0 && (w & 0x7f800000u) != 0x7f800000u && (w & 1u) == (unsigned)(stamp & 1);
}

// ---- small helpers ---------------------------------------------------------------
__device__ __forceinline__ int wrapc(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

__device__ __forceinline__ unsigned lane_id() { return __lane_id(); }

// append the lanes with pred to a list: one atomic per wave
__device__ __forceinline__ void wave_append(bool pred, int value, int *list, int *counter,
                                            int cap, unsigned *err) {
    unsigned long long mask = __ballot(pred);
    if (!mask) return;
    int n = __popcll(mask);
    int leader = __ffsll((long long)mask) - 1;
    int base = 0;
    if ((int)lane_id() == leader) base = atomicAdd(counter, n);
    base = __shfl(base, leader);
    if (pred) {
        int off = __popcll(mask & ((1ull << lane_id()) - 1ull));
        int slot = base + off;
        if (slot < cap) list[slot] = value;
        else atomicOr(err, ERR_CAP);
    }
}

// the D3Q19 components of a direction that differs between lanes: two bits each
// (value + 1) in a 64-bit constant, where the arrays of cx, cy, cz would be loads
constexpr unsigned long long pack_dirs(int a) {
    unsigned long long m = 0;
    for (int q = 0; q < Q; ++q) m |= (unsigned long long)((a == 0 ? cx(q) : a == 1 ? cy(q) : cz(q)) + 1) << (2 * q);
    return m;
}
template <int A> __device__ __forceinline__ int dir_comp(int q) {
    constexpr unsigned long long m = pack_dirs(A);
    return (int)((m >> (2 * q)) & 3ull) - 1;
}

// a barrier between two phases of one block that hand each other global memory, atomics
// among it: the loads that follow see what every wave of the block wrote before
__device__ __forceinline__ void block_phase() {
    __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// A barrier between two phases over the first nblk blocks of a launch.  The callers launch
// at most SYNC_BLOCKS blocks of 256 threads (or SYNC_BIG of 1,024), and no more than an eighth of
// what the device holds of that kernel (sync_rule.hpp, from its occupancy), so the blocks come
// to run together whatever else is running; one block needs no device barrier.  bar counts arrivals since the step's counters were cleared, target the
// arrivals the next barrier waits for.  Every wave's stores have left the wave before its
// block arrives; one thread releases them to the device and acquires the others'.  The
// wait is bounded: a launch that lost a block reports an error instead of hanging.
constexpr int SYNC_BLOCKS = 128, SYNC_BIG = 32;  // blocks of 256 threads, of 1,024
struct GridBarrier {
    int *bar;
    int nblk, target;
    unsigned *err;
    __device__ __forceinline__ void wait() {
        if (nblk == 1) {
            block_phase();
            return;
        }
        target += nblk;
        __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence();
            __hip_atomic_fetch_add(bar, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int spin = 0; __hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target; ++spin) {
                __builtin_amdgcn_s_sleep(1);
                if (spin > (1 << 23)) {
                    atomicOr(err, ERR_SYNC);
                    break;
                }
            }
            __threadfence();
        }
        __syncthreads();
    }
};

// true in every thread of the block that finishes last of nblk (its reads then see what
// the others wrote); done counts the blocks and is left at zero.  STORES: the others hand
// over plain stores; without, atomics only, which need no release (a release writes a
// whole L2 back: 40 us of the 84 of the 2,048 blocks of the bubble pass)
template <bool STORES = true>
__device__ __forceinline__ bool last_block(int *done, int nblk) {
    __shared__ int last;
    __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        if (STORES) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        last = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nblk - 1;
        if (last) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    return last != 0;
}

// FP64 sum over the wave with DPP on the two 32-bit halves: pairs, quads, half-row and row
// mirrors leave every lane of a row of 16 with the row sum; row_bcast:15 on rows 1 and 3
// then adds the row before, row_bcast:31 on rows 2 and 3 lane 31, so that lane 63 holds
// the whole wave.  Every lane of the wave must be active; all get the sum.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_d(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xF, false);
    return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add_d<0xB1, 0xF>(v);
    v = dpp_add_d<0x4E, 0xF>(v);
    v = dpp_add_d<0x141, 0xF>(v);
    v = dpp_add_d<0x140, 0xF>(v);
    v = dpp_add_d<0x142, 0xA>(v);
    v = dpp_add_d<0x143, 0xC>(v);
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Seven such sums at once, each in the tree of wave_sum (lanes pairwise by bit 0, 1, ... 5 of
// their number; the order of a pair does not matter).  In the first three rounds a lane
// keeps half of what it holds and hands the other half to its partner, so that four, two and
// one additions stand for seven each; lane ln ends with the sum of component wave_part(ln) (7: none).
// Every lane of the wave must be active.
__device__ __forceinline__ int wave_part(int ln) { return 4 * (ln & 1) + (ln & 2) + ((ln >> 2) & 1); }
template <typename X> __device__ __forceinline__ double wave_swap(double v, X &&x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)x((int)(unsigned)b), hi = (unsigned)x((int)(unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sums7(const double (&v)[7]) {
    const int ln = (int)lane_id();
    auto dpp1 = [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false); };   // quad_perm [1,0,3,2]
    auto dpp2 = [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false); };   // quad_perm [2,3,0,1]
    auto swz4 = [](int x) { return __builtin_amdgcn_ds_swizzle(x, 0x101F); };                     // lane ^ 4
    auto dpp8 = [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, false); };  // row_ror:8
    auto swz16 = [](int x) { return __builtin_amdgcn_ds_swizzle(x, 0x401F); };                    // lane ^ 16
    const bool b0 = ln & 1, b1 = ln & 2, b2 = ln & 4;
    double r[4], s[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double h = k < 3 ? v[k < 3 ? k + 4 : 0] : 0.0;
        r[k] = (b0 ? h : v[k]) + wave_swap(b0 ? v[k] : h, dpp1);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) s[k] = (b1 ? r[k + 2] : r[k]) + wave_swap(b1 ? r[k] : r[k + 2], dpp2);
    double t = (b2 ? s[1] : s[0]) + wave_swap(b2 ? s[0] : s[1], swz4);
    t += wave_swap(t, dpp8);
    t += wave_swap(t, swz16);
    t += __shfl_xor(t, 32);
    return t;
}
// One sum by halves of the wave (32, 16, ... 1).  The links between spheres and at faces take
// this tree: the last bits of a force depend on it.
__device__ __forceinline__ double wave_sum_halves(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

}  // namespace fsl
