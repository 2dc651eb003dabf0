// Batched solver: many independent non-negative QPs (Sec. 2.1.3, eq.
// non-negative) advanced together.
//
// Each member runs the single-problem method (the same steps, constants and
// tests: gradient and KKT test, Cauchy search, Jacobi-PCG on the free face,
// projected search, trust-region update), but the members do not move in
// lockstep: every member carries its own phase in a device-resident state
// machine, and one global step advances every member by one step of its own
// phase.  A global step is two launches over all members, each block working
// on some slices of one member:
//
//   row pass     per slice, by the member's phase: gradient g = K c - f,
//                Cauchy trial along -g, CG matrix pass, or projected-search
//                trial along the CG step (one matrix pass each);
//   vector pass  per slice, by the operation chosen: Cauchy step with CG
//                set-up, CG vector update, breakpoint search, or step along w.
//
// Each pass begins with the member's transition: every block of the member
// combines the slice partials the pass before left (the same fixed order, the
// same bits) and takes the decision the host takes in the single-problem
// solver (convergence, trial accepted, CG step length, next phase).  The
// member's first block writes the new state to the other of two state arrays,
// which the next pass reads.  (As launches of their own, one block per member,
// the two transitions took 4.2 us each and two launch gaps of 2.4 us, of the
// 32.6 us of a step of 64 members.)
//
// A member that needs many iterations therefore does not hold the others
// back: while it is in a long CG, the others run their own Cauchy searches,
// gradients and CGs in the same launches.  The host only replays chunks of
// global steps (captured once per size class as hipGraphs) and, between
// chunks, drops finished members from the device lists the launches walk.
//
// Layout: the members keep their own sliced-ELL matrices, reached through
// per-member pointer tables.  The batch numbers their 64-row slices
// consecutively (a slice never spans two members) and concatenates the work
// vectors over those slices, so global row s*64 + lane is local row
// (s - first slice of its member)*64 + lane.  Every reduction leaves one
// partial per slice, and a member's partials are combined by its own block
// in a fixed order: a member's arithmetic depends only on its own data, so
// its result is bitwise the same in any batch and for any launch shape.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <vector>

#include "diag.hpp"

// 1: chunks of global steps replayed as captured graphs; 0: launched one by one
#ifndef NNQP_BATCH_GRAPH
#define NNQP_BATCH_GRAPH 1
#endif

namespace nnqp {

namespace {

constexpr int kBNV = 5;          // values per slice partial
constexpr int kFinBlock = 256;   // threads of a block
constexpr int kBWaves = kFinBlock / 64;
// Blocks the running slices are spread over, eight per CU of 256 CUs (64
// members: 188 ms a solve, 195 with half as many, 205-219 with two to four
// times as many), and a block's slices at most above that.
constexpr int kBGrid = 2048;
constexpr int kBMost = 32;
// Slices above which a launch of its own forms the shares of a member's partials
// (kb_share).  Without it each of the member's blocks (one per kBMost slices)
// adds up every partial, which grows with the square: one member of 127^3 rows,
// 31,256 slices, 445 -> 189 ms a solve and 69.3 -> 24.1 a backward-Euler step,
// 3,907 slices (two of 64^3) 40.2 -> 37.1 and 25.0 -> 20.1.  Below the line the
// two launches a step cost more than they save: 3,151 slices 227 -> 239 and
// 33.5 -> 31.3, 1,623 slices 13.2 -> 15.8 and 4.0 -> 4.5.
constexpr int kBLarge = 3584;
constexpr double kMu0 = 0.01;    // sufficient-decrease constant
constexpr double kExtrap = 10.0; // Cauchy extrapolation factor
constexpr double kInterp = 0.1;  // Cauchy interpolation factor
constexpr double kBack = 0.5;    // projected-search backtracking factor
constexpr int kMaxTrials = 60;

// member phases: what the next row pass does for the member
enum : int {
    PH_DONE = 0,    // finished (status set)
    PH_GRAD = 1,    // gradient and convergence test
    PH_CAUCHY = 2,  // Cauchy search trial along -g
    PH_CG = 3,      // CG iteration
    PH_BREAK = 4,   // breakpoint of the step along w (vector pass only)
    PH_SEARCH = 5,  // projected-search trial along w
    PH_APPLYW = 6   // take the step along w (vector pass only)
};
// vector-pass operations chosen by the first transition
enum : int { VO_NONE = 0, VO_SETUP = 1, VO_UPDATE = 2, VO_BREAK = 3, VO_APPLYW = 4 };
// Cauchy search sub-states
enum : int { CS_FIRST = 0, CS_EXT = 1, CS_INT = 2 };

// Per-member state, in device memory (mirrored on the host between chunks).
struct BState {
    // control
    int phase, vop, status, outer;
    int cst, cur, ksbuf, ntrial;     // Cauchy sub-state, accepted K s buffer, trial buffer, trials
    int it, cgdone, nsearch, max_outer;
    int max_cg, pad0;
    double t, tcau, ttrial;          // accepted Cauchy step, its start value, signed trial step
    double gs, sks, ss;              // accepted Cauchy trial: g.s, s.Ks, s.s
    double delta, normf, tol, rtol2;
    double rz, rr_stop, alpha, beta, n_free, nnz_free;   // CG
    double bmin, wn, ts, stepn;      // projected search along w, step length of the iteration
    double n, nnz, eb, eg, vb;       // rows, nonzeros, bytes per nonzero of the search and CG
                                     // passes and of the gradient, bytes per vector entry
    // report
    double kkt_rel, kkt_nat, min_c, bytes;
    int n_active, cg_its, spmvs, cauchy_trials, search_trials, refinements, mixed, pad1;
};

// One block's work: slices [s, s + n) of member p (global numbers); first:
// the member's first block, which writes its state.
struct BBlk {
    int p, s, n, first;
};

// The list entry a workgroup takes, of nb: eight neighbouring entries on one
// XCD (workgroups go round-robin to the eight), as the blocks of a member read
// one another's rows and all of its partials.  64 float64 members of 32^2 to
// 256^2 cells: 186.6 -> 183.2 ms, 80 mixed ones 180.3 -> 177.9; a whole eighth
// of the list per XCD took the same there, but leaves XCDs with all of a large
// member, and one step of 60 members went from 47.0 to 48.5 ms.
__device__ __forceinline__ int near_block(int nb)
{
    const int b = blockIdx.x;
    return b < (nb & ~63) ? (b & ~63) | ((b & 7) << 3) | ((b >> 3) & 7) : b;
}

// A member's place in the concatenated vectors and, with the diagonal layout,
// its offsets: the array of offset h[u] starts at b0 + (u + 1) stride counted
// from global row 0 (W = 0: another layout).
struct BTab {
    int s0, nsl, nrow, W;
    int share;      // large members: place in the shares (kb_share), else -1
    DiagReg reg;
};

struct BDev {
    int P, nslices;
    const int *cnt;                 // [2] blocks and members in the current lists
    const int *plist;               // members taking part in the current launches
    const BBlk *blk;                // their blocks, member by member
    const BTab *tab;                // per member
    const int *sprob;               // [nslices] member of each slice
    const int *s0, *nrow;           // per member: first slice, rows
    const int *const *so;           // per member sliced-ELL offsets
    const int *const *sc;           // per member sliced-ELL columns (local)
    const short *const *sd;         // per member int16 offsets col - row (or null)
    const double *const *v64;       // per member float64 values
    const float *const *v32;        // per member float32 values (mixed precision)
    const double *const *diag;      // per member diagonal
    const int *const *rowptr;       // per member CSR row pointers
    double *const *c;               // per member solution vectors (local rows)
    const double *const *f;         // per member loads of the solve
    const double *const *f0;        // per member loads (transient step: f of f + M c/dt)
    const double *const *mv;        // per member capacity values (transient step)
    uint8_t *const *act_out;        // per member active-set outputs (entries may be null)
    BState *st, *st2;               // states before the row pass, before the vector pass
    double *part, *part2;           // [kBNV][nslices]: of the row pass, of the vector pass
    const int *large;               // the large members
    double *shares;                 // [large member][kBNV][kFinBlock] (kb_share)
    double *pres;                   // [P][kBNV] (start-up reductions)
    // the batch as one block-diagonal sliced-ELL matrix and concatenated
    // vectors (global rows s*64 + lane), copied in at the start of a call
    const int *gso;                 // [nslices+1] first entry of each slice
    const int *gcol;                // global column of each entry
    const short *gd16;              // col - row (int16), or null
    const double *gv64;             // float64 values of the solve
    const float *gv32;              // float32 values (mixed precision), or null
    double *cg, *fg;                // solution and load
    const double *dg;               // diagonal of the solve's matrix (1 on rows past the end)
    const int *rlen;                // entries of each row (0 past the end)
    double lo, hi;                  // bounds lo <= c <= hi of every member
};

// Work vectors of the batched solve, concatenated over the slices.
template <class VV>
struct BVec {
    double *g, *ks0, *ks1;
    uint8_t *mask;
    VV *w, *r, *z, *p, *q, *dm;
};

__device__ __forceinline__ double bcomb(int op, double a, double b)
{
    return op == OP_SUM ? a + b : (op == OP_MIN ? fmin(a, b) : fmax(a, b));
}

// combination of one value over the wavefront (every lane active)
__device__ __forceinline__ double bwave(int op, double a)
{
    return op == OP_SUM ? wave_sum(a) : (op == OP_MIN ? wave_min(a) : wave_max(a));
}

__device__ __forceinline__ double bident(int op)
{
    return op == OP_SUM ? 0.0 : (op == OP_MIN ? INFINITY : -INFINITY);
}

// projection on [lo, hi]; NaN maps to lo (+0.0 for lo = 0)
__device__ __forceinline__ double projb(const BDev &B, double x)
{
    const double y = x > B.lo ? x : B.lo;
    return y < B.hi ? y : B.hi;
}

// The calling block's slices, one wavefront each in turn.  For a slice of a
// member with take(p): body(p, s, global row, local row, row exists, a); every
// slice then stores its wave-combined partials (identities when the member did
// not take part).
template <int NV, class Take, class Body>
__device__ __forceinline__ void for_bslices(const BDev &B, const int (&ops)[NV], Take take,
                                            Body body)
{
    if ((int)blockIdx.x >= B.cnt[0]) return;
    const BBlk K = B.blk[near_block(B.cnt[0])];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int s = K.s + wid; s < K.s + K.n; s += kBWaves) {
        double a[NV];
#pragma unroll
        for (int k = 0; k < NV; k++) a[k] = bident(ops[k]);
        if (take(K.p)) {
            const int il = (s - B.s0[K.p]) * kSlice + lane;
            body(K.p, s, s * kSlice + lane, il, il < B.nrow[K.p], a);
        }
#pragma unroll
        for (int k = 0; k < NV; k++) a[k] = bwave(ops[k], a[k]);
        if (lane == 0)
#pragma unroll
            for (int k = 0; k < NV; k++) B.part[(size_t)k * B.nslices + s] = a[k];
    }
}

// Layouts of the concatenated matrix (as in the single-problem kernels):
// diagonal arrays where every member has them in one regular run; else, when
// every member's offsets fit int16, quads of float32 values or pairs of
// float64 values; else int32 columns.  Float64 values load with the non-temporal
// hint, float32 values normally (as in the single-problem kernels).
enum { CM_I32, CM_Q4, CM_P2, CM_DIAG };

// Position of entry k of lane l in a slice of width w of the quad layout
// (CM_Q4), relative to the slice's first entry: entries 4j .. 4j+3 of a row
// side by side at 256 j + 4 l, two left over as a pair at 256 (w / 4) + 2 l,
// an odd last one in its column-major place 64 k + l.  A row of seven
// entries (2D P1) then takes three value loads and three offset loads
// instead of seven of each.
__host__ __device__ __forceinline__ int quad_pos(int k, int l, int w)
{
    const int nq = w >> 2, np = (w - 4 * nq) >> 1;
    if (k < 4 * nq) return 256 * (k >> 2) + 4 * l + (k & 3);
    if (k < 4 * nq + 2 * np) return 256 * nq + 2 * l + (k - 4 * nq);
    return 64 * k + l;
}

// The same for the paired layout (CM_P2): entries 2j, 2j+1 of a row side by
// side at 128 j + 2 l, an odd last one in its column-major place.
__host__ __device__ __forceinline__ int pair_pos(int k, int l, int w)
{
    const int np = w >> 1;
    if (k < 2 * np) return 128 * (k >> 1) + 2 * l + (k & 1);
    return 64 * k + l;
}

// Four (quad) or two (pair) consecutive values of the quad layout, with the
// same load hint as bld_val.
__device__ __forceinline__ void bld_quad(const double *p, double (&v)[4])
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    const d2 a = __builtin_nontemporal_load(reinterpret_cast<const d2 *>(p));
    const d2 b = __builtin_nontemporal_load(reinterpret_cast<const d2 *>(p + 2));
    v[0] = a.x;
    v[1] = a.y;
    v[2] = b.x;
    v[3] = b.y;
}
__device__ __forceinline__ void bld_quad(const float *p, float (&v)[4])
{
    const float4 a = *reinterpret_cast<const float4 *>(p);
    v[0] = a.x;
    v[1] = a.y;
    v[2] = a.z;
    v[3] = a.w;
}
__device__ __forceinline__ void bld_pair(const double *p, double &a, double &b)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    const d2 v = __builtin_nontemporal_load(reinterpret_cast<const d2 *>(p));
    a = v.x;
    b = v.y;
}
__device__ __forceinline__ void bld_pair(const float *p, float &a, float &b)
{
    const float2 v = *reinterpret_cast<const float2 *>(p);
    a = v.x;
    b = v.y;
}

__device__ __forceinline__ double bld_val(const double *p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ float bld_val(const float *p) { return *p; }

// Row sums of slice s of member p: sum_k val(k) x(col(k)), with the same
// wave-uniform load phases (eight entries each) and column order as the
// single-problem kernels.  Padding and rows past the end hold valid columns.
template <int WMAX, class VT, class X>
__device__ __forceinline__ double bsell_row(const BDev &B, const VT *__restrict__ sv, int p, int s,
                                            X x)
{
    const int lane = threadIdx.x & 63;
    const int ls = s - B.s0[p];
    const int *__restrict__ so = B.so[p];
    const int *__restrict__ sc = B.sc[p];
    const int off = so[ls];
    const int w = (so[ls + 1] - off) >> 6;
    double acc = 0.0;
    constexpr int H = WMAX < 8 ? WMAX : 8;
#pragma unroll
    for (int h0 = 0; h0 < WMAX; h0 += H) {
        int cc[H];
        VT vv[H];
#pragma unroll
        for (int k = 0; k < H; k++) {
            if (h0 + k < w) {
                cc[k] = sc[off + (h0 + k) * kSlice + lane];
                vv[k] = bld_val(sv + off + (h0 + k) * kSlice + lane);
            } else {
                cc[k] = 0;
                vv[k] = VT(0);
            }
        }
#pragma unroll
        for (int k = 0; k < H; k++)
            if (h0 + k < w) acc += (double)vv[k] * x(cc[k]);
    }
    for (int k = WMAX; k < w; k++) {
        const int e = off + k * kSlice + lane;
        acc += (double)bld_val(sv + e) * x(sc[e]);
    }
    return acc;
}

#ifndef NNQP_BATCH_FLAT8
#define NNQP_BATCH_FLAT8 1   // slices of width <= 8: every load of the row issued before any use
#endif

// The row sum of gsell_row_at for slices of width w <= 8 (2D P1 rows),
// written so that no load waits for another: every matrix load of the row is
// issued under wave-uniform guards that only move raw bits (no column is
// decoded inside a guard, which would make the compiler wait for that load
// there), then every gather is issued, then the products are added in entry
// order.  A slot past the row's entries keeps offset 0 (column i, a valid
// row) or column i, and value 0, and its product is not added (a select, so
// a non-finite x_i cannot leak in): the sum is bitwise the one of the
// guarded walk, entry by entry with fused multiply-adds.  On the 512-member
// batch the row pass went from 95 to 73 us (float64) and from 76 to 55 us
// (mixed): the guarded walk waited for every pair's offsets and for every
// gather in turn.
template <int CM, class VT, class X>
__device__ __forceinline__ double gsell_row8(const BDev &B, const VT *__restrict__ sv, int i,
                                             int off, int w, X x)
{
    const int lane = threadIdx.x & 63;
    const short *__restrict__ gd = B.gd16;
    double acc = 0.0;
    if constexpr (CM == CM_Q4) {
        // quads 0 and 1 (entries 0-7), the pair left over (two entries
        // after the quads), the odd last entry: the entry order
        const int nq = w >> 2, rem = w & 3;
        VT q[2][4];
        int2 dq[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            if (k < nq) {
                const int e = off + k * 4 * kSlice + 4 * lane;
                bld_quad(sv + e, q[k]);
                dq[k] = *reinterpret_cast<const int2 *>(gd + e);
            } else {
#pragma unroll
                for (int t = 0; t < 4; t++) q[k][t] = VT(0);
                dq[k] = make_int2(0, 0);
            }
        }
        VT pa = VT(0), pb = VT(0), so = VT(0);
        int dp = 0, dso = 0;
        if (rem >= 2) {
            const int e = off + nq * 4 * kSlice + 2 * lane;
            bld_pair(sv + e, pa, pb);
            dp = *reinterpret_cast<const int *>(gd + e);
        }
        if (rem & 1) {
            const int e = off + (w - 1) * kSlice + lane;
            so = bld_val(sv + e);
            dso = gd[e];
        }
        double xv[11];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            xv[4 * k] = x(i + (int)(short)(dq[k].x & 0xffff));
            xv[4 * k + 1] = x(i + (dq[k].x >> 16));
            xv[4 * k + 2] = x(i + (int)(short)(dq[k].y & 0xffff));
            xv[4 * k + 3] = x(i + (dq[k].y >> 16));
        }
        xv[8] = x(i + (int)(short)(dp & 0xffff));
        xv[9] = x(i + (dp >> 16));
        xv[10] = x(i + dso);
#pragma unroll
        for (int k = 0; k < 2; k++)
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const double y = __builtin_fma((double)q[k][t], xv[4 * k + t], acc);
                acc = k < nq ? y : acc;
            }
        const double y8 = __builtin_fma((double)pa, xv[8], acc);
        acc = rem >= 2 ? y8 : acc;
        const double y9 = __builtin_fma((double)pb, xv[9], acc);
        acc = rem >= 2 ? y9 : acc;
        const double y10 = __builtin_fma((double)so, xv[10], acc);
        acc = (rem & 1) ? y10 : acc;
        return acc;
    } else if constexpr (CM == CM_P2) {
        // pairs 0-3 (entries 0-7), the odd last entry
        const int np = w >> 1;
        VT v[4][2];
        int d[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            if (k < np) {
                const int e = off + k * 2 * kSlice + 2 * lane;
                bld_pair(sv + e, v[k][0], v[k][1]);
                d[k] = *reinterpret_cast<const int *>(gd + e);
            } else {
                v[k][0] = v[k][1] = VT(0);
                d[k] = 0;
            }
        }
        VT so = VT(0);
        int dso = 0;
        if (w & 1) {
            const int e = off + (w - 1) * kSlice + lane;
            so = bld_val(sv + e);
            dso = gd[e];
        }
        double xv[9];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            xv[2 * k] = x(i + (int)(short)(d[k] & 0xffff));
            xv[2 * k + 1] = x(i + (d[k] >> 16));
        }
        xv[8] = x(i + dso);
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const double y = __builtin_fma((double)v[k][t], xv[2 * k + t], acc);
                acc = k < np ? y : acc;
            }
        const double y8 = __builtin_fma((double)so, xv[8], acc);
        acc = (w & 1) ? y8 : acc;
        return acc;
    } else {
        // column-major entries 0-7 (int32 global columns)
        const int *__restrict__ gc = B.gcol;
        VT v[8];
        int cc[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            if (k < w) {
                const int e = off + k * kSlice + lane;
                v[k] = bld_val(sv + e);
                cc[k] = gc[e];
            } else {
                v[k] = VT(0);
                cc[k] = i;
            }
        }
        double xv[8];
#pragma unroll
        for (int k = 0; k < 8; k++) xv[k] = x(cc[k]);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const double y = __builtin_fma((double)v[k], xv[k], acc);
            acc = k < w ? y : acc;
        }
        return acc;
    }
}

// Row sums over the concatenated matrix for global row i = s*64 + lane of a
// slice whose first entry (off) and width (w) are known; global columns.
template <int WMAX, int CM, class VT, class X>
__device__ __forceinline__ double gsell_row_at(const BDev &B, const VT *__restrict__ sv, int i,
                                               int off, int w, X x)
{
    if constexpr (WMAX == 8 && NNQP_BATCH_FLAT8) return gsell_row8<CM>(B, sv, i, off, w, x);
    const int lane = threadIdx.x & 63;
    const int *__restrict__ gc = B.gcol;
    const short *__restrict__ gd = B.gd16;
    auto col = [&](int e) {
        if (CM == CM_Q4 || CM == CM_P2) return i + (int)gd[e];
        return gc[e];
    };
    double acc = 0.0;
    if constexpr (CM == CM_P2) {
        // pairs in entry order, then the odd entry: the column-major sum order
        const int np = w >> 1;
        constexpr int HP = (WMAX < 8 ? WMAX : 8) / 2;   // pairs per load phase
#pragma unroll
        for (int h0 = 0; h0 < WMAX / 2; h0 += HP) {
            int cc[2 * HP];
            VT vv[2 * HP];
#pragma unroll
            for (int k = 0; k < HP; k++) {
                if (h0 + k < np) {
                    const int e = off + (h0 + k) * 2 * kSlice + 2 * lane;
                    bld_pair(sv + e, vv[2 * k], vv[2 * k + 1]);
                    const int d2 = *reinterpret_cast<const int *>(gd + e);
                    cc[2 * k] = i + (int)(short)(d2 & 0xffff);
                    cc[2 * k + 1] = i + (d2 >> 16);
                } else {
                    cc[2 * k] = cc[2 * k + 1] = 0;
                    vv[2 * k] = vv[2 * k + 1] = VT(0);
                }
            }
#pragma unroll
            for (int k = 0; k < 2 * HP; k++)
                if (h0 + k / 2 < np) acc += (double)vv[k] * x(cc[k]);
        }
        for (int k = WMAX / 2; k < np; k++) {   // slices wider than the unrolled part
            const int e = off + k * 2 * kSlice + 2 * lane;
            acc += (double)bld_val(sv + e) * x(col(e));
            acc += (double)bld_val(sv + e + 1) * x(col(e + 1));
        }
        if (w & 1) {
            const int e = off + (w - 1) * kSlice + lane;
            acc += (double)bld_val(sv + e) * x(col(e));
        }
        return acc;
    }
    if constexpr (CM == CM_Q4) {
        // quads in entry order, then the left-over pair, then the odd entry:
        // the same sum order as the column-major walk
        const int nq = w >> 2, rem = w & 3;
        constexpr int HQ = (WMAX < 8 ? WMAX : 8) / 4;   // quads per load phase
#pragma unroll
        for (int h0 = 0; h0 < WMAX / 4; h0 += HQ) {
            int cc[4 * HQ];
            VT vv[4 * HQ];
#pragma unroll
            for (int k = 0; k < HQ; k++) {
                if (h0 + k < nq) {
                    const int e = off + (h0 + k) * 4 * kSlice + 4 * lane;
                    VT q[4];
                    bld_quad(sv + e, q);
                    const int2 d = *reinterpret_cast<const int2 *>(gd + e);
                    cc[4 * k] = i + (int)(short)(d.x & 0xffff);
                    cc[4 * k + 1] = i + (d.x >> 16);
                    cc[4 * k + 2] = i + (int)(short)(d.y & 0xffff);
                    cc[4 * k + 3] = i + (d.y >> 16);
#pragma unroll
                    for (int t = 0; t < 4; t++) vv[4 * k + t] = q[t];
                } else {
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        cc[4 * k + t] = 0;
                        vv[4 * k + t] = VT(0);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 4 * HQ; k++)
                if (h0 + k / 4 < nq) acc += (double)vv[k] * x(cc[k]);
        }
        for (int k = WMAX / 4; k < nq; k++) {   // slices wider than the unrolled part
            const int e = off + k * 4 * kSlice + 4 * lane;
#pragma unroll
            for (int t = 0; t < 4; t++) acc += (double)bld_val(sv + e + t) * x(col(e + t));
        }
        if (rem >= 2) {
            const int e = off + nq * 4 * kSlice + 2 * lane;
            VT a, b;
            bld_pair(sv + e, a, b);
            const int d2 = *reinterpret_cast<const int *>(gd + e);
            acc += (double)a * x(i + (int)(short)(d2 & 0xffff));
            acc += (double)b * x(i + (d2 >> 16));
        }
        if (rem & 1) {
            const int e = off + (w - 1) * kSlice + lane;
            acc += (double)bld_val(sv + e) * x(col(e));
        }
        return acc;
    }
    constexpr int H = WMAX < 8 ? WMAX : 8;
#pragma unroll
    for (int h0 = 0; h0 < WMAX; h0 += H) {
        int cc[H];
        VT vv[H];
#pragma unroll
        for (int k = 0; k < H; k++) {
            if (h0 + k < w) {
                cc[k] = col(off + (h0 + k) * kSlice + lane);
                vv[k] = bld_val(sv + off + (h0 + k) * kSlice + lane);
            } else {
                cc[k] = 0;
                vv[k] = VT(0);
            }
        }
#pragma unroll
        for (int k = 0; k < H; k++)
            if (h0 + k < w) acc += (double)vv[k] * x(cc[k]);
    }
    for (int k = WMAX; k < w; k++) {
        const int e = off + k * kSlice + lane;
        acc += (double)bld_val(sv + e) * x(col(e));
    }
    return acc;
}

// Row sum of a diagonal-layout member (see diag.hpp): PH entries per load
// phase; rows whose columns would leave the member's are held inside it.
template <int W, int PH, class VT, class X>
__device__ __forceinline__ double bdiag_row(const BTab &T, const VT *__restrict__ sv, int s, X x)
{
    using XT = decltype(x(0, 0));
    DiagTab<W> t;
    t.b0 = T.reg.b0;
    t.stride = T.reg.stride;
#pragma unroll
    for (int u = 0; u < W / 2; u++) t.h[u] = T.reg.h[u];
    const int ls = s - T.s0, far = t.h[W / 2 - 1];
    auto x1 = [&](int ub, int l, XT (&out)[1]) { out[0] = x(ub, l); };
    double acc[1] = {0.0};
    if (ls * kSlice >= far && ls * kSlice + kSlice - 1 + far < T.nrow) {
        diag_row_reg<W, 1, PH, false, XT>(t, sv, 0, s * kSlice, x1, acc);
    } else {
        // columns counted from the member's first row, held inside its rows
        const int r0 = T.s0 * kSlice;
        auto xl = [&](int, int l, XT (&out)[1]) { out[0] = x(r0, l); };
        diag_row_reg<W, 1, 4, true, XT>(t, sv + r0, T.nrow, ls * kSlice, xl, acc);
    }
    return acc[0];
}

// The same for slice s of a member in the batch's layout; x(ub, l) is the
// gathered value of global row ub + l.
template <int WMAX, int CM, int PH, class VT, class X>
__device__ __forceinline__ double gsell_row(const BDev &B, const BTab &T, const VT *__restrict__ sv,
                                            int s, int i, X x)
{
    if constexpr (CM == CM_DIAG) {
        if constexpr (WMAX > 8)
            if (T.W == 15) return bdiag_row<15, PH>(T, sv, s, x);
        return bdiag_row<7, PH>(T, sv, s, x);
    } else {
        const int off = B.gso[s];
        return gsell_row_at<WMAX, CM>(B, sv, i, off, (B.gso[s + 1] - off) >> 6,
                                      [&](int j) { return x(0, j); });
    }
}

__device__ __forceinline__ bool running(const BDev &B, int p) { return B.st[p].phase != PH_DONE; }

// Slice s of member p into the diagonal arrays: entry k of a row at b_k + row
// for the offsets >= 0 (the others are read through the opposite triangle),
// zero where the row has none, and the zeros in front of the arrays.
__device__ __forceinline__ void gather_diag(const BDev &B, int p, int s, int src,
                                            double *__restrict__ gv64, float *__restrict__ gv32)
{
    const int lane = threadIdx.x & 63;
    const BTab &T = B.tab[p];
    const int ls = s - T.s0, row = ls * kSlice + lane, i = s * kSlice + lane;
    const int H = T.W / 2;
    const int len = row < T.nrow ? B.rowptr[p][row + 1] - B.rowptr[p][row] : 0;
    const int *sc = B.sc[p];
    const double *v64 = B.v64[p];
    const float *v32 = B.v32[p];
    int cur = 0;
    auto offset = [&]() { return cur < len ? sc[src + cur * kSlice + lane] - row : 0x7fffffff; };
    int d = offset();
    while (d < 0) {   // (entries below the diagonal)
        cur++;
        d = offset();
    }
    for (int u = 0; u <= H; u++) {
        const int du = u == 0 ? 0 : T.reg.h[u - 1];
        const ptrdiff_t b = (ptrdiff_t)T.reg.b0 + (ptrdiff_t)u * T.reg.stride;
        const bool has = d == du;
        const int e = src + cur * kSlice + lane;
        gv64[b + i] = has ? v64[e] : 0.0;
        if (gv32) gv32[b + i] = has ? v32[e] : 0.f;
        if (has) {
            cur++;
            d = offset();
        }
        // rows before the member's first one
        const int reach = (T.reg.h[H - 1] + kSlice - 1) / kSlice;
        for (int q = ls; q < reach; q += T.nsl) {
            const ptrdiff_t at = b + (ptrdiff_t)(T.s0 + q - reach) * kSlice + lane;
            gv64[at] = 0.0;
            if (gv32) gv32[at] = 0.f;
        }
    }
}

// Copy the members into the concatenated layout (every slice of the batch):
// c, f, diagonal and row lengths into the global vectors; slice offsets
// (ebase[p] + the member's own offset), global columns, int16 offsets and
// values into the global matrix arrays in the batch's layout.  Rows past a
// member's end get c = 0, f = 0, diagonal 1, length 0; their entries keep their
// valid columns (zeros in the diagonal layout).
__global__ void kb_gather(BDev B, const int64_t *__restrict__ ebase, int *__restrict__ gso,
                          int *__restrict__ gcol, short *__restrict__ gd16,
                          double *__restrict__ gv64, float *__restrict__ gv32,
                          double *__restrict__ dg, int *__restrict__ rlen, int copy_f, int layout)
{
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    for (int s = blockIdx.x * wpb + wid; s < B.nslices; s += nw) {
        const int p = B.sprob[s];
        const int ls = s - B.s0[p];
        const int il = ls * kSlice + lane, i = s * kSlice + lane;
        const int r0 = B.s0[p] * kSlice;
        const bool row = il < B.nrow[p];
        B.cg[i] = row ? B.c[p][il] : 0.0;
        if (copy_f) B.fg[i] = row ? B.f[p][il] : 0.0;
        dg[i] = row ? B.diag[p][il] : 1.0;
        rlen[i] = row ? B.rowptr[p][il + 1] - B.rowptr[p][il] : 0;
        const int *so = B.so[p];
        const int src = so[ls], w = (so[ls + 1] - src) >> 6;
        if (layout == CM_DIAG) {
            gather_diag(B, p, s, src, gv64, gv32);
            continue;
        }
        const int dst = (int)(ebase[p] + src);
        if (lane == 0) gso[s] = dst;
        const int *sc = B.sc[p];
        const short *sd = B.sd[p];
        const double *v64 = B.v64[p];
        const float *v32 = B.v32[p];
        for (int k = 0; k < w; k++) {
            const int es = src + k * kSlice + lane;
            const int ed = dst + (layout == CM_Q4   ? quad_pos(k, lane, w)
                                  : layout == CM_P2 ? pair_pos(k, lane, w)
                                                    : k * kSlice + lane);
            gcol[ed] = sc[es] + r0;
            if (gd16) gd16[ed] = sd[es];
            gv64[ed] = v64[es];
            if (gv32) gv32[ed] = v32[es];
        }
    }
}

// Copy the solution back to the members' vectors, and the active sets.
__global__ void kb_scatter(BDev B)
{
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int nw = gridDim.x * wpb;
    for (int s = blockIdx.x * wpb + wid; s < B.nslices; s += nw) {
        const int p = B.sprob[s];
        const int il = (s - B.s0[p]) * kSlice + lane;
        if (il >= B.nrow[p]) continue;
        const double cv = B.cg[s * kSlice + lane];
        B.c[p][il] = cv;
        uint8_t *out = B.act_out[p];
        if (out) out[il] = cv == B.lo ? 1 : (cv == B.hi ? 2 : 0);
    }
}

// ---------------------------------------------------------------- start-up kernels
// c = c0v (mode 0) or P(c) (mode 1); |f|^2, max f, #non-finite f, #non-finite c
__global__ void kb_init(BDev B, int mode, double c0v)
{
    const int ops[4] = {OP_SUM, OP_MAX, OP_SUM, OP_SUM};
    for_bslices<4>(B, ops, [&](int p) { return running(B, p); },
                   [&](int, int, int i, int, bool row, double (&a)[4]) {
                       if (!row) return;
                       const double fi = B.fg[i];
                       a[0] += fi * fi;
                       a[1] = fmax(a[1], fi);
                       a[2] += isfinite(fi) ? 0.0 : 1.0;
                       double *c = B.cg;
                       if (mode == 0) {
                           c[i] = c0v;
                       } else {
                           const double cv = c[i];
                           a[3] += isfinite(cv) ? 0.0 : 1.0;
                           c[i] = projb(B, cv);
                       }
                   });
}

// Right-hand side of a backward-Euler step, ft = f0 + (M c) / dt, written
// into the concatenated vector ft (the solve's loads point into it).
template <int WMAX>
__global__ void kb_transient_rhs(BDev B, double dt, double *__restrict__ ft)
{
    const int ops[1] = {OP_SUM};
    for_bslices<1>(B, ops, [&](int p) { return running(B, p); },
                   [&](int p, int s, int i, int il, bool row, double (&)[1]) {
                       const double *c = B.c[p];
                       const double mc =
                           bsell_row<WMAX>(B, B.mv[p], p, s, [&](int j) { return c[j]; });
                       if (row) ft[i] = B.f0[p][il] + mc / dt;
                       else ft[i] = 0.0;
                   });
}

// Partials of a member as its transition reads them: value k of place s at
// v[k * ld + s], s = s0 .. s0 + n - 1.
struct BPart {
    const double *v;
    size_t ld;
    int s0, n;
};

// The calling thread's share of the first NV values of a member's partials:
// places t, t + 256, ... in order.
template <int NV>
__device__ __forceinline__ void member_load(const BPart &Q, const int (&ops)[NV], double (&a)[NV])
{
#pragma unroll
    for (int k = 0; k < NV; k++) a[k] = bident(ops[k]);
    for (int s = Q.s0 + threadIdx.x; s < Q.s0 + Q.n; s += kFinBlock)
#pragma unroll
        for (int k = 0; k < NV; k++) a[k] = bcomb(ops[k], a[k], Q.v[(size_t)k * Q.ld + s]);
}

// Combine the threads' shares in a fixed order (a wave butterfly, then the
// four waves in order) into out (LDS); the caller separates it from the reads
// with a barrier, and two calls from each other.
template <int NV>
__device__ __forceinline__ void member_combine(const int (&ops)[NV], double (&a)[NV], double *out)
{
    __shared__ double sh[NV][kBWaves];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int k = 0; k < NV; k++) a[k] = bwave(ops[k], a[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; k++) sh[k][wid] = a[k];
    __syncthreads();
    if (threadIdx.x < NV) {
        const int k = threadIdx.x;
        double v = sh[k][0];
        // (ops is the same constant in every thread; k is not)
        int op = ops[0];
#pragma unroll
        for (int q = 1; q < NV; q++) op = k == q ? ops[q] : op;
        for (int w = 1; w < kBWaves; w++) v = bcomb(op, v, sh[k][w]);
        out[k] = v;
    }
}

// start-up reduction: |f|^2, max f, #non-finite f, #non-finite c into pres
__global__ __launch_bounds__(kFinBlock) void kb_reduce_init(BDev B)
{
    if ((int)blockIdx.x >= B.cnt[1]) return;
    const int p = B.plist[blockIdx.x];
    const int ops[4] = {OP_SUM, OP_MAX, OP_SUM, OP_SUM};
    __shared__ double r[4];
    double a[4];
    member_load<4>(BPart{B.part, (size_t)B.nslices, B.tab[p].s0, B.tab[p].nsl}, ops, a);
    member_combine<4>(ops, a, r);
    __syncthreads();
    if (threadIdx.x < 4) B.pres[(size_t)p * kBNV + threadIdx.x] = r[threadIdx.x];
}

// ---------------------------------------------------------------- global step
__device__ __forceinline__ void radius_update(BState &S)
{
    if (isfinite(S.delta) && S.stepn >= 0.99 * S.delta) S.delta *= 4.0;
}

// First transition: the decision on the row pass's sums a (none when the
// phase had no row work).
__device__ __forceinline__ void transition1(BState &S, const double *a)
{
    const int ph = S.phase;
    const double n = S.n, nnz = S.nnz;
    const double trial_bytes = 4.0 * (n + 1) + S.eb * nnz + 32.0 * n;
    S.vop = VO_NONE;
    if (ph == PH_GRAD) {
        // gradient, KKT report, convergence test
        S.spmvs++;
        S.bytes += 4.0 * (n + 1) + S.eg * nnz + 32.0 * n;
        if (a[1] != 0.0) {
            S.status = NN_ENONFINITE;
            S.phase = PH_DONE;
            return;
        }
        S.kkt_rel = sqrt(a[0]) / S.normf;
        S.kkt_nat = a[2];
        S.min_c = a[3];
        S.n_active = (int)a[4];
        if (S.mixed) S.refinements = S.outer + 1;
        if (S.kkt_rel <= S.tol) {
            S.status = NN_OK;
            S.phase = PH_DONE;
        } else if (S.outer >= S.max_outer) {
            S.status = NN_EMAXIT;
            S.phase = PH_DONE;
        } else {
            // Cauchy search from the previous step length
            S.cst = CS_FIRST;
            S.t = S.tcau;
            S.cur = 0;
            S.ntrial = 0;
            S.ttrial = -S.t;
            S.ksbuf = 0;
            S.phase = PH_CAUCHY;
        }
    } else if (ph == PH_CAUCHY) {
        S.spmvs++;
        S.cauchy_trials++;
        S.bytes += trial_bytes;
        const bool ok = a[0] < 0.0 && a[0] + 0.5 * a[1] <= kMu0 * a[0] && sqrt(a[2]) <= S.delta;
        bool accept = false;
        if (S.cst == CS_FIRST) {
            if (ok) {
                S.gs = a[0], S.sks = a[1], S.ss = a[2];
                S.cst = CS_EXT;
            } else {
                S.cst = CS_INT;
                S.t *= kInterp;
            }
        } else if (S.cst == CS_EXT) {
            if (!ok) {
                accept = true;
            } else {
                const bool same = a[0] == S.gs && a[1] == S.sks;
                S.t *= kExtrap;
                S.cur ^= 1;
                S.gs = a[0], S.sks = a[1], S.ss = a[2];
                // stop when every moving variable has reached its bound
                if (same || ++S.ntrial >= 20) accept = true;
            }
        } else {
            S.gs = a[0], S.sks = a[1], S.ss = a[2];
            if (ok) {
                accept = true;
            } else if (++S.ntrial >= kMaxTrials || !(a[0] < 0.0)) {
                // no decrease along -g at this precision: stationary up to rounding
                S.status = NN_EMAXIT;
                S.phase = PH_DONE;
                return;
            } else {
                S.t *= kInterp;
            }
        }
        if (accept) {
            S.tcau = S.t;
            S.stepn = sqrt(S.ss);
            S.vop = VO_SETUP;   // Cauchy step and CG set-up in the vector pass
            S.phase = PH_CG;
        } else if (S.cst == CS_EXT) {
            S.ttrial = -S.t * kExtrap;
            S.ksbuf = S.cur ^ 1;
        } else {
            S.ttrial = -S.t;
            S.ksbuf = S.cur;
        }
    } else if (ph == PH_CG) {
        // alpha = r.z / p.q; breakdown on non-positive or non-finite curvature
        const double pq = a[0];
        if (S.cgdone != 0) {
            S.phase = PH_BREAK;
        } else if (!isfinite(pq)) {
            S.status = NN_ENONFINITE;
            S.phase = PH_DONE;
        } else if (!(pq > 0.0)) {
            S.status = NN_ENOTSPD;
            S.phase = PH_DONE;
        } else {
            S.alpha = S.rz / pq;
            S.vop = VO_UPDATE;
        }
    } else if (ph == PH_SEARCH) {
        S.spmvs++;
        S.search_trials++;
        S.bytes += trial_bytes;
        bool accept = false;
        if (a[0] < 0.0 && a[0] + 0.5 * a[1] <= kMu0 * a[0]) {
            accept = true;
        } else {
            S.ts *= kBack;
            if (S.ts <= S.bmin) {
                S.ts = S.bmin;   // no bound is crossed: decrease is guaranteed
                accept = true;
            } else if (++S.nsearch >= kMaxTrials) {
                accept = true;
            }
        }
        if (accept) {
            S.vop = VO_APPLYW;
            S.phase = PH_APPLYW;
        }
    } else if (ph == PH_BREAK) {
        S.vop = VO_BREAK;
    } else if (ph == PH_APPLYW) {
        S.vop = VO_APPLYW;
    }
}

// Second transition: the decision on the vector pass's sums a, and the phase of
// the member's next global step.
__device__ __forceinline__ void transition2(BState &S, const double *a)
{
    const int vop = S.vop;
    const double n = S.n;
    if (vop == VO_SETUP) {
        // CG start on the free face: stop before the first iteration when the
        // face is empty or the residual vanishes
        S.bytes += 24.0 * n + 88.0 * n;
        S.rz = a[0];
        S.rr_stop = S.rtol2 * a[1];
        S.n_free = a[2];
        S.nnz_free = a[3];
        S.beta = 0.0;
        S.alpha = 0.0;
        S.it = 0;
        if (!isfinite(a[0]) || !isfinite(a[1])) {
            S.status = NN_ENONFINITE;
            S.phase = PH_DONE;
        } else if (a[1] == 0.0 || a[2] == 0.0 || S.max_cg <= 0 || !(a[0] > 0.0)) {
            S.cgdone = 1;
            S.phase = PH_BREAK;
        } else {
            S.cgdone = 0;
            S.phase = PH_CG;
        }
    } else if (vop == VO_UPDATE) {
        // iteration done: beta for the next one, stopping test on r.r
        const double rz = a[0], rr = a[1];
        const double nf = S.n_free, nzf = S.nnz_free;
        S.bytes += n + 4.0 * nf + S.eb * nzf + 5.0 * S.vb * nf + n + 8.0 * S.vb * nf;
        S.it += 1;
        S.cg_its++;
        S.spmvs++;
        S.beta = rz / S.rz;
        S.rz = rz;
        if (!isfinite(rz) || !isfinite(rr)) {
            S.status = NN_ENONFINITE;
            S.phase = PH_DONE;
        } else if (rr <= S.rr_stop || S.it >= S.max_cg || !(rz > 0.0)) {
            S.cgdone = 1;
            S.phase = PH_BREAK;
        }
    } else if (vop == VO_BREAK) {
        S.bytes += 24.0 * n;
        S.bmin = a[0];
        S.wn = sqrt(a[2]);
        if (S.it > 0 && a[1] < 0.0 && S.wn > 0.0) {
            S.ts = fmin(1.0, S.delta / S.wn);
            S.nsearch = 0;
            S.phase = S.bmin >= S.ts ? PH_APPLYW : PH_SEARCH;
        } else {
            // no step along w: radius update on the Cauchy step, next iteration
            radius_update(S);
            S.outer++;
            S.phase = PH_GRAD;
        }
    } else if (vop == VO_APPLYW) {
        S.bytes += 24.0 * n;
        S.stepn += S.ts * S.wn;
        radius_update(S);
        S.outer++;
        S.phase = PH_GRAD;
    }
    S.vop = VO_NONE;
}

// What a pass needs of the member's new state.
struct BAct {
    int what;       // row pass: phase (PH_DONE: nothing to do); vector pass: operation
    int buf;        // row pass: buffer of K s; vector pass: accepted buffer
    double a, b;    // trial step or beta; alpha, Cauchy step or step along w
};

// The sums of a pass, first NV values of the member's slice partials, into
// sums (LDS), every thread of the block; the caller adds a barrier.
template <int NV>
__device__ __forceinline__ void member_sums(const BPart &Q, const int (&ops)[NV], double *sums)
{
    double a[NV];
    member_load<NV>(Q, ops, a);
    member_combine<NV>(ops, a, sums);
}

// The member's transition on the partials of the pass before (the first one in
// a vector pass, the second in a row pass).  Every block of the member comes to
// the same result; the first one writes the new state to `out`.  The state and
// the partials of a CG iteration (one value, or two) are loaded together, and
// a member that stays in its CG needs no more than them: one barrier, after
// which every thread has the decision.  Anything else goes through the
// transition itself, on the state in LDS.  ahead() runs once those loads are
// issued and issues others.  (Reading the block's first slices there, entries
// and gathers or the update's vectors, measured 1-3 % slower on 64 members:
// the registers cost more waves than the round trip hidden.)
template <bool SECOND, class Ahead>
__device__ __forceinline__ BAct block_transition(const BDev &B, const BBlk &K, const BTab &T,
                                                 const BState *in, BState *out, BState &S,
                                                 double *sums, Ahead ahead)
{
    static_assert(sizeof(BState) % sizeof(int) == 0 && sizeof(BState) / sizeof(int) <= kFinBlock,
                  "one word per thread");
    constexpr int kWords = sizeof(BState) / sizeof(int);
    constexpr int NF = SECOND ? 2 : 1;
    __shared__ double sh[NF][kBWaves];
    const BPart Q = T.share >= 0
                        ? BPart{B.shares + (size_t)T.share * kBNV * kFinBlock, kFinBlock, 0, kFinBlock}
                        : BPart{SECOND ? B.part2 : B.part, (size_t)B.nslices, T.s0, T.nsl};
    const int word = threadIdx.x < kWords ? reinterpret_cast<const int *>(in + K.p)[threadIdx.x] : 0;
    double f[NF], f1[NF];
    const int t1 = Q.s0 + threadIdx.x, te = Q.s0 + Q.n;
#pragma unroll
    for (int k = 0; k < NF; k++) f1[k] = t1 < te ? Q.v[(size_t)k * Q.ld + t1] : 0.0;
    ahead();
#pragma unroll
    for (int k = 0; k < NF; k++) f[k] = 0.0 + f1[k];
    for (int s = t1 + kFinBlock; s < te; s += kFinBlock)
#pragma unroll
        for (int k = 0; k < NF; k++) f[k] += Q.v[(size_t)k * Q.ld + s];
    if (threadIdx.x < kWords) reinterpret_cast<int *>(&S)[threadIdx.x] = word;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int k = 0; k < NF; k++) {
        f[k] = wave_sum(f[k]);
        if (lane == 0) sh[k][wid] = f[k];
    }
    __syncthreads();
    auto total = [&](int k) { return ((sh[k][0] + sh[k][1]) + sh[k][2]) + sh[k][3]; };
    static_assert(kBWaves == 4, "four waves' sums in order");
    BAct r{SECOND ? (int)PH_DONE : (int)VO_NONE, 0, 0.0, 0.0};
    bool fast;
    if constexpr (SECOND) {
        const double rz = total(0), rr = total(1);
        fast = S.vop == VO_UPDATE && isfinite(rz) && isfinite(rr) && rr > S.rr_stop &&
               S.it + 1 < S.max_cg && rz > 0.0;
        r.what = PH_CG;
        r.a = rz / S.rz;   // beta
        if (threadIdx.x == 0) {
            sums[0] = rz;
            sums[1] = rr;
        }
    } else {
        const double pq = total(0);
        fast = S.phase == PH_CG && S.cgdone == 0 && isfinite(pq) && pq > 0.0;
        r.what = VO_UPDATE;
        r.b = S.rz / pq;   // alpha
        if (threadIdx.x == 0) sums[0] = pq;
    }
    if (fast && !K.first) return r;
    __syncthreads();
    if (!fast) {
        if constexpr (SECOND) {
            const int vop = S.vop;
            if (vop == VO_SETUP) {
                const int ops[4] = {OP_SUM, OP_SUM, OP_SUM, OP_SUM};
                member_sums<4>(Q, ops, sums);
            } else if (vop == VO_BREAK) {
                const int ops[3] = {OP_MIN, OP_SUM, OP_SUM};
                member_sums<3>(Q, ops, sums);
            }
        } else {
            const int ph = S.phase;
            if (ph == PH_GRAD) {
                const int ops[5] = {OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM};
                member_sums<5>(Q, ops, sums);
            } else if (ph == PH_CAUCHY || ph == PH_SEARCH) {
                const int ops[3] = {OP_SUM, OP_SUM, OP_SUM};
                member_sums<3>(Q, ops, sums);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if constexpr (SECOND) transition2(S, sums);
        else transition1(S, sums);
    }
    __syncthreads();
    if (K.first && threadIdx.x < kWords)
        reinterpret_cast<int *>(out + K.p)[threadIdx.x] = reinterpret_cast<const int *>(&S)[threadIdx.x];
    if (fast) return r;
    if constexpr (SECOND) {
        r.what = S.phase == PH_CG && S.cgdone != 0 ? (int)PH_DONE : S.phase;
        r.buf = S.ksbuf;
        r.a = S.phase == PH_CAUCHY ? S.ttrial : (S.phase == PH_SEARCH ? S.ts : S.beta);
    } else {
        r.what = S.vop;
        r.buf = S.cur;
        r.b = S.vop == VO_SETUP ? S.t : (S.vop == VO_APPLYW ? S.ts : S.alpha);
    }
    return r;
}

// Row pass: the second transition of the step before, then per slice the
// matrix pass of the member's phase.
//   GRAD    g = K c - f (float64 values); |pg|^2, #non-finite, ||min(c,g)||_inf,
//           min c, #(c == 0)
//   CAUCHY  s = P(c + ttrial g) - c gathered, ks = K s into buffer ksbuf;
//           g.s, s.Ks, s.s
//   CG      p <- z + beta p, q <- K z + beta q on the free rows; p.q
//   SEARCH  s = P(c + ts w) - c on the free rows, K s; g.s, s.Ks, s.s
template <int WMAX, int CM, class VT, class VV>
__global__ __launch_bounds__(kFinBlock) void kb_rows(BDev B, const VT *__restrict__ gvals,
                                                     BVec<VV> V)
{
    if ((int)blockIdx.x >= B.cnt[0]) return;
    const BBlk K = B.blk[near_block(B.cnt[0])];
    const BTab &T = B.tab[K.p];
    __shared__ BState S;
    __shared__ double sums[kBNV];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nw = kBWaves;
    int s = K.s + wid;
    uint8_t m1 = 0;   // the next slice's flags, read ahead
    auto ahead = [&] {
        if (s < K.s + K.n) m1 = V.mask[s * kSlice + lane];
    };
    const BAct A = block_transition<true>(B, K, T, B.st, B.st2, S, sums, ahead);
    const int ph = __builtin_amdgcn_readfirstlane(A.what);
    // (no row work: the transition does not read these partials)
    if (ph != PH_GRAD && ph != PH_CAUCHY && ph != PH_CG && ph != PH_SEARCH) return;
    const double *__restrict__ c = B.cg;
    for (; s < K.s + K.n; s += nw) {
        const bool free_row = m1 != 0;
        if (s + nw < K.s + K.n) m1 = V.mask[(s + nw) * kSlice + lane];
        const int i = s * kSlice + lane;
        const bool row = (s - T.s0) * kSlice + lane < T.nrow;
        double a[kBNV] = {0.0, 0.0, 0.0, 0.0, 0.0};
        if (ph == PH_GRAD) {
            a[2] = -INFINITY;
            a[3] = INFINITY;
            const double kc = gsell_row<WMAX, CM, 4>(B, T, B.gv64, s, i,
                                                  [&](int ub, int l) { return (c + ub)[l]; });
            if (row) {
                const double gi = kc - B.fg[i];
                const double cv = c[i];
                V.g[i] = gi;
                const double pg = cv > B.lo ? (cv < B.hi ? gi : fmax(gi, 0.0)) : fmin(gi, 0.0);
                a[0] = pg * pg;
                a[1] = (isfinite(gi) && isfinite(cv)) ? 0.0 : 1.0;
                a[2] = fabs(fmax(cv - B.hi, fmin(gi, cv - B.lo)));
                a[3] = cv;
                a[4] = (cv == B.lo || cv == B.hi) ? 1.0 : 0.0;
            }
        } else if (ph == PH_CAUCHY) {
            const double t = A.a;
            const double *__restrict__ g = V.g;
            auto sv = [&](int ub, int l) {
                const double cj = (c + ub)[l];
                return projb(B, cj + t * (g + ub)[l]) - cj;
            };
            const double ksv = gsell_row<WMAX, CM, 4>(B, T, gvals, s, i, sv);
            if (row) {
                (A.buf ? V.ks1 : V.ks0)[i] = ksv;
                const double si = sv(0, i);
                a[0] = g[i] * si;
                a[1] = si * ksv;
                a[2] = si * si;
            }
        } else if (ph == PH_CG) {
            const bool live = row && free_row;
            if (__ballot(live) != 0) {
                const VV *__restrict__ z = V.z;
                // the own-row values load before the gathers
                VV pold = VV(0), qold = VV(0), zi = VV(0);
                if (live) {
                    pold = V.p[i];
                    qold = V.q[i];
                    zi = z[i];
                }
                const double kz = gsell_row<WMAX, CM, 8>(B, T, gvals, s, i,
                                                         [&](int ub, int l) { return (z + ub)[l]; });
                if (live) {
                    const double beta = A.a;
                    const VV pi = (VV)fma(beta, (double)pold, (double)zi);
                    const VV qi = (VV)fma(beta, (double)qold, kz);
                    V.p[i] = pi;
                    V.q[i] = qi;
                    a[0] = (double)pi * (double)qi;
                }
            }
        } else {   // PH_SEARCH
            const bool live = row && free_row;
            if (__ballot(live) != 0) {
                const double t = A.a;
                const VV *__restrict__ w = V.w;
                auto sv = [&](int ub, int l) {
                    const double cj = (c + ub)[l];
                    return projb(B, cj + t * (double)(w + ub)[l]) - cj;
                };
                const double ksv = gsell_row<WMAX, CM, 4>(B, T, gvals, s, i, sv);
                if (live) {
                    const double si = sv(0, i);
                    a[0] = V.g[i] * si;
                    a[1] = si * ksv;
                    a[2] = si * si;
                }
            }
        }
        // wave combination (the phase is uniform in the wave): only the
        // values the phase reports
        const int nv = ph == PH_GRAD ? 5 : (ph == PH_CG ? 1 : 3);
        a[0] = wave_sum(a[0]);
        if (nv >= 3) {
            a[1] = wave_sum(a[1]);
            if (nv == 3) {
                a[2] = wave_sum(a[2]);
            } else {
                a[2] = wave_max(a[2]);
                a[3] = wave_min(a[3]);
                a[4] = wave_sum(a[4]);
            }
        }
        if (lane == 0)
            for (int v = 0; v < nv; v++) B.part[(size_t)v * B.nslices + s] = a[v];
    }
}

// Vector pass: the first transition, then per slice the operation it chose.
//   SETUP   c = P(c - t g), g += K s (accepted Cauchy trial); free = not
//           (c == 0 and g >= 0); dm = 1/diag, r = -g on free rows; z = dm r;
//           p = q = w = 0; r.z, r.r, #free, nnz of the free rows
//   UPDATE  w += alpha p, r -= alpha q, z = dm r on free rows; r.z, r.r
//   BREAK   min over w < 0 of c/(-w), g.w, w.w
//   APPLYW  c = P(c + ts w)
template <class VV>
__global__ __launch_bounds__(kFinBlock) void kb_vec(BDev B, BVec<VV> V)
{
    if ((int)blockIdx.x >= B.cnt[0]) return;
    const BBlk K = B.blk[near_block(B.cnt[0])];
    const BTab &T = B.tab[K.p];
    __shared__ BState S;
    __shared__ double sums[kBNV];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int s = K.s + wid;
    // the mask of the next slice is read ahead (only a set-up writes a mask,
    // and only its own slice's, which it does not read)
    uint8_t m1 = 0;
    auto ahead = [&] {
        if (s < K.s + K.n) m1 = V.mask[s * kSlice + lane];
    };
    const BAct A = block_transition<false>(B, K, T, B.st2, B.st, S, sums, ahead);
    const int vop = __builtin_amdgcn_readfirstlane(A.what);
    if (vop == VO_NONE) return;
    for (; s < K.s + K.n; s += kBWaves) {
        const bool free_row = m1 != 0;
        if (s + kBWaves < K.s + K.n) m1 = V.mask[(s + kBWaves) * kSlice + lane];
        const int i = s * kSlice + lane;
        const bool row = (s - T.s0) * kSlice + lane < T.nrow;
        double *__restrict__ c = B.cg;
        double a[4] = {0.0, 0.0, 0.0, 0.0};
        if (vop == VO_SETUP) {
            if (!row) {
                V.mask[i] = 0;
                V.dm[i] = V.r[i] = V.z[i] = V.p[i] = V.q[i] = V.w[i] = VV(0);
            } else {
                const double gi0 = V.g[i];
                const double cv = projb(B, c[i] - A.b * gi0);
                const double gi = gi0 + (A.buf ? V.ks1 : V.ks0)[i];
                c[i] = cv;
                V.g[i] = gi;
                const bool fr = !((cv == B.lo && gi >= 0.0) || (cv == B.hi && gi <= 0.0));
                const VV dmi = fr ? (VV)(1.0 / B.dg[i]) : VV(0);
                const VV ri = fr ? (VV)(-gi) : VV(0);
                const VV zi = dmi * ri;
                V.mask[i] = fr ? 1 : 0;
                V.dm[i] = dmi;
                V.r[i] = ri;
                V.z[i] = zi;
                V.p[i] = VV(0);
                V.q[i] = VV(0);
                V.w[i] = VV(0);
                a[0] = (double)ri * (double)zi;
                a[1] = (double)ri * (double)ri;
                a[2] = fr ? 1.0 : 0.0;
                a[3] = fr ? (double)B.rlen[i] : 0.0;
            }
        } else if (vop == VO_UPDATE) {
            if (row && free_row) {
                const double alpha = A.b;
                const VV ri = (VV)((double)V.r[i] - alpha * (double)V.q[i]);
                const VV zi = V.dm[i] * ri;
                V.w[i] = (VV)((double)V.w[i] + alpha * (double)V.p[i]);
                V.r[i] = ri;
                V.z[i] = zi;
                a[0] = (double)ri * (double)zi;
                a[1] = (double)ri * (double)ri;
            }
        } else if (vop == VO_BREAK) {
            a[0] = INFINITY;
            if (row) {
                const double wi = (double)V.w[i];
                if (wi < 0.0) a[0] = (c[i] - B.lo) / (-wi);
                else if (wi > 0.0) a[0] = (B.hi - c[i]) / wi;
                a[1] = V.g[i] * wi;
                a[2] = wi * wi;
            }
        } else {   // VO_APPLYW
            if (row) c[i] = projb(B, c[i] + A.b * (double)V.w[i]);
            continue;
        }
        // (an update reports two values, a breakpoint three)
        a[0] = vop == VO_BREAK ? wave_min(a[0]) : wave_sum(a[0]);
        a[1] = wave_sum(a[1]);
        if (vop != VO_UPDATE) {
            a[2] = wave_sum(a[2]);
            a[3] = wave_sum(a[3]);
        }
        if (lane == 0) {
            const int nv = vop == VO_UPDATE ? 2 : (vop == VO_BREAK ? 3 : 4);
            for (int v = 0; v < nv; v++) B.part2[(size_t)v * B.nslices + s] = a[v];
        }
    }
}

// The shares of the large members: what thread t of a transition's block would
// add up of the member's partials, places t, t + 256, ... in order, so that a
// block of the member reads 256 numbers per value instead of one per slice.
// Block: one value of one member, 64 of its 256 shares.
template <bool SECOND>
__global__ __launch_bounds__(64) void kb_share(BDev B)
{
    const int m = blockIdx.x / (kBNV * kBWaves), k = blockIdx.x / kBWaves % kBNV;
    const int p = B.large[m], t = (blockIdx.x % kBWaves) * 64 + threadIdx.x;
    const BState &S = (SECOND ? B.st : B.st2)[p];
    // values and operation of the pass behind it (as the transitions read them)
    int nv = 0, op = OP_SUM;
    if constexpr (SECOND) {
        const int vop = S.vop;
        nv = vop == VO_SETUP ? 4 : vop == VO_UPDATE ? 2 : vop == VO_BREAK ? 3 : 0;
        if (vop == VO_BREAK && k == 0) op = OP_MIN;
    } else {
        const int ph = S.phase;
        nv = ph == PH_GRAD ? 5 : ph == PH_CAUCHY || ph == PH_SEARCH ? 3 : ph == PH_CG && S.cgdone == 0 ? 1 : 0;
        if (ph == PH_GRAD && k == 2) op = OP_MAX;
        if (ph == PH_GRAD && k == 3) op = OP_MIN;
    }
    if (k >= nv) return;
    const BTab &T = B.tab[p];
    const double *v = (SECOND ? B.part2 : B.part) + (size_t)k * B.nslices + T.s0;
    double a = bident(op);
    constexpr int U = 16;   // loads in flight
    int s = t;
    for (; s + (U - 1) * kFinBlock < T.nsl; s += U * kFinBlock) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; u++) x[u] = v[s + u * kFinBlock];
#pragma unroll
        for (int u = 0; u < U; u++) a = bcomb(op, a, x[u]);
    }
    for (; s < T.nsl; s += kFinBlock) a = bcomb(op, a, v[s]);
    B.shares[((size_t)m * kBNV + k) * kFinBlock + t] = a;
}

// Second transition on its own, in place: the states the host reads (and the
// next chunk's first row pass, which finds no vector operation to decide on).
__global__ __launch_bounds__(kFinBlock) void kb_step2(BDev B)
{
    if ((int)blockIdx.x >= B.cnt[1]) return;
    const int p = B.plist[blockIdx.x];
    __shared__ BState S;
    __shared__ double sums[kBNV];
    block_transition<true>(B, BBlk{p, 0, 0, 1}, B.tab[p], B.st, B.st, S, sums, [] {});
}

// ---------------------------------------------------------------- host side
// The same with the kernel's own begin and end recorded into e0, e1 when
// they are not null (hipExtLaunchKernelGGL).
#ifndef NNQP_BATCH_PAIRS
#define NNQP_BATCH_PAIRS 1   // float64 batches read the concatenated matrix in pairs
#endif

#define NN_BLAUNCH_EV(KERNEL, grid, block, stream, e0, e1, ...)                                 \
    do {                                                                                        \
        if (e0)                                                                                 \
            hipExtLaunchKernelGGL(KERNEL, dim3(grid), dim3(block), 0, stream, e0, e1, 0,         \
                                  __VA_ARGS__);                                                 \
        else                                                                                    \
            hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(block), 0, stream, __VA_ARGS__);        \
    } while (0)
#define NN_BDISPATCH_EV(wmax, KERNEL, grid, block, stream, e0, e1, ...)                         \
    do {                                                                                        \
        if ((wmax) <= 8) {                                                                      \
            constexpr int WM = 8;                                                               \
            NN_BLAUNCH_EV(KERNEL, grid, block, stream, e0, e1, __VA_ARGS__);                    \
        } else if ((wmax) <= 16) {                                                              \
            constexpr int WM = 16;                                                              \
            NN_BLAUNCH_EV(KERNEL, grid, block, stream, e0, e1, __VA_ARGS__);                    \
        } else {                                                                                \
            constexpr int WM = 32;                                                              \
            NN_BLAUNCH_EV(KERNEL, grid, block, stream, e0, e1, __VA_ARGS__);                    \
        }                                                                                       \
    } while (0)

#define NN_BDISPATCH(wmax, KERNEL, grid, block, stream, ...)                                    \
    do {                                                                                        \
        if ((wmax) <= 8) {                                                                      \
            constexpr int WM = 8;                                                               \
            hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(block), 0, stream, __VA_ARGS__);        \
        } else if ((wmax) <= 16) {                                                              \
            constexpr int WM = 16;                                                              \
            hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(block), 0, stream, __VA_ARGS__);        \
        } else {                                                                                \
            constexpr int WM = 32;                                                              \
            hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(block), 0, stream, __VA_ARGS__);        \
        }                                                                                       \
    } while (0)

// Device and pinned host memory of one batched call, released on every exit.
struct Arena {
    const DevAlloc &al;   // the context's device memory hooks
    std::vector<void *> dev, host;
    bool ok = true;
    explicit Arena(const DevAlloc &a) : al(a) {}
    template <class T>
    T *d(size_t n)
    {
        void *p = nullptr;
        if (dev_malloc(al, &p, sizeof(T) * std::max<size_t>(n, 1)) != hipSuccess) {
            ok = false;
            return nullptr;
        }
        dev.push_back(p);
        return (T *)p;
    }
    template <class T>
    T *h(size_t n)
    {
        void *p = nullptr;
        if (hipHostMalloc(&p, sizeof(T) * std::max<size_t>(n, 1), hipHostMallocDefault) !=
            hipSuccess) {
            ok = false;
            return nullptr;
        }
        host.push_back(p);
        return (T *)p;
    }
    ~Arena()
    {
        for (void *p : dev) dev_free(al, p);
        for (void *p : host) (void)hipHostFree(p);
    }
};

// Captured chunks of global steps, one per launch-size class (the grid of a
// captured launch is fixed; the lists it walks are read from device memory).
struct GraphCache {
    struct G {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
    };
    std::map<int, G> by_class;
    ~GraphCache()
    {
        for (auto &kv : by_class) {
            if (kv.second.exec) (void)hipGraphExecDestroy(kv.second.exec);
            if (kv.second.graph) (void)hipGraphDestroy(kv.second.graph);
        }
    }
};

struct Events {
    std::vector<hipEvent_t> ev;
    ~Events()
    {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
    }
    bool create(size_t n, unsigned flags)
    {
        ev.assign(n, nullptr);
        for (hipEvent_t &e : ev)
            if (hipEventCreateWithFlags(&e, flags) != hipSuccess) return false;
        return true;
    }
};

// Algorithmic bytes of the row pass of one member in its current state (the
// same byte model as the member's own transitions).
double row_bytes(const BState &S)
{
    const double n = S.n, nnz = S.nnz;
    switch (S.phase) {
    case PH_GRAD:
        return 4.0 * (n + 1) + S.eg * nnz + 32.0 * n;
    case PH_CAUCHY:
    case PH_SEARCH:
        return 4.0 * (n + 1) + S.eb * nnz + 32.0 * n;
    case PH_CG:
        return S.cgdone ? 0.0
                        : n + 4.0 * S.n_free + S.eb * S.nnz_free + 5.0 * S.vb * S.n_free;
    default:
        return 0.0;
    }
}

// The same under the paper's CSR model (4-byte column indices; the CG
// matrix pass as a masked SpMV plus a separate direction update).
double row_bytes_csr(const BState &S)
{
    const double n = S.n, nnz = S.nnz;
    switch (S.phase) {
    case PH_GRAD:
        return 4.0 * (n + 1) + 12.0 * nnz + 32.0 * n;
    case PH_CAUCHY:
    case PH_SEARCH:
        return 4.0 * (n + 1) + (4.0 + S.vb) * nnz + 32.0 * n;
    case PH_CG:
        return S.cgdone ? 0.0
                        : (4.0 + S.vb) * S.nnz_free + (4.0 + 6.0 * S.vb) * S.n_free;
    default:
        return 0.0;
    }
}

}  // namespace

nn_status solve_batch_impl(nn_ctx *ctx, int P, nn_matrix *const *K, const double *const *f,
                           const nn_opts *o, double *const *c, uint8_t *const *active,
                           nn_stats *stats, double dt)
{
    hipStream_t st = ctx->stream;
    const bool mixed = o->precision == NN_MIXED;
    const bool transient = dt > 0.0;
    std::vector<nn_stats> SP(P);
    for (nn_stats &x : SP) std::memset(&x, 0, sizeof(x));

    // ---- slice numbering
    std::vector<int> s0(P), nrow(P), nsl(P), sprob;
    int wmax = 1;
    int64_t S = 0;
    for (int p = 0; p < P; p++) {
        const int64_t n = K[p]->n;
        nrow[p] = (int)n;
        s0[p] = (int)S;
        nsl[p] = (int)((n + kSlice - 1) / kSlice);
        S += nsl[p];
        if (S * kSlice >= (int64_t)1 << 31)
            return fail(ctx, NN_EINVAL, "batch too large: total rows must stay below 2^31");
        for (int t = 0; t < nsl[p]; t++) sprob.push_back(p);
        if (n > 0) wmax = std::max(wmax, K[p]->wmax);
        const float *v32 = nullptr;
        if (mixed && n > 0 && !transient) {
            const nn_status rc = ensure_val32(ctx, K[p], &v32);
            if (rc != NN_OK) return rc;
        }
    }
    if (S == 0) {
        if (stats)
            for (int p = 0; p < P; p++) stats[p] = SP[p];
        ctx->err.clear();
        return NN_OK;
    }
    const int64_t R = S * kSlice;
    std::vector<int> large;   // members whose shares are formed by a launch of their own
    for (int p = 0; p < P; p++)
        if (nsl[p] > kBLarge) large.push_back(p);
    bool all_d16 = true;
    for (int p = 0; p < P; p++)
        if (K[p]->n > 0 && !K[p]->sl_d16) all_d16 = false;
    const double vb = mixed ? 4.0 : 8.0;                // bytes per CG vector entry and per value
    // Mixed precision reads the concatenated matrix in the quad layout (int16
    // offsets, four float32 values per load): on the 512-member batch the row
    // pass takes 67 instead of 107 us.  Float64 reads it in pairs (int16
    // offset pairs, one 16-byte load per value pair): 95-97 instead of
    // 90-106 us (its quad layout was no faster, column-major int16 offsets
    // slower).
    // diagonal arrays when every member has them in one regular run
    bool all_diag = true;
    std::vector<DiagReg> dreg(P);
    {
        // (locked in the order of their addresses, each once)
        std::vector<nn_matrix *> all, fresh;
        for (int p = 0; p < P; p++)
            if (K[p]->n > 0) all.push_back(K[p]);
        std::sort(all.begin(), all.end());
        all.erase(std::unique(all.begin(), all.end()), all.end());
        std::vector<std::unique_lock<std::recursive_mutex>> locks;
        locks.reserve(all.size());
        for (nn_matrix *A : all) {
            locks.emplace_back(A->copies);
            DiagReg reg;
            if (!A->diag_tried) fresh.push_back(A);
            else if (!diag_one_run(A, &reg)) all_diag = false;
        }
        nn_status rc = NN_OK;
        if (all_diag && !fresh.empty()) {
            // The members that are new are looked over together: one at a time
            // the first solve of 512 new members of 39^2 rows took 71 ms, 22 of
            // them later.  (The layout is read for speed only: without room to
            // look for it the batch takes another.)
            void *tmp = nullptr;
            const int m = (int)fresh.size();
            if (dev_malloc(ctx->al, &tmp, diag_find_bytes(fresh.data(), m)) != hipSuccess) rc = NN_EOOM;
            else rc = diag_find_many(ctx, fresh.data(), m, tmp);
            dev_free(ctx->al, tmp);
        }
        for (int p = 0; p < P && all_diag; p++)
            if (K[p]->n > 0) all_diag = diag_one_run(K[p], &dreg[p]);
        if ((rc = without_copy(ctx, rc)) != NN_OK) return rc;
    }
    const bool quad = !all_diag && mixed && all_d16;
    const bool pair = !all_diag && !mixed && all_d16 && NNQP_BATCH_PAIRS;
    const int layout = all_diag ? CM_DIAG : quad ? CM_Q4 : (pair ? CM_P2 : CM_I32);

    // ---- tables, work vectors, lists, pinned state mirrors
    Arena A(ctx->al);
    int *d_sprob = A.d<int>(S), *d_s0 = A.d<int>(P), *d_nrow = A.d<int>(P);
    int *d_list = A.d<int>((size_t)2 + P);
    BBlk *d_blk = A.d<BBlk>(S);
    BTab *d_tab = A.d<BTab>(P);
    const int **d_so = A.d<const int *>(P), **d_sc = A.d<const int *>(P),
              **d_rp = A.d<const int *>(P);
    const short **d_sd = A.d<const short *>(P);
    const double **d_v64 = A.d<const double *>(P), **d_diag = A.d<const double *>(P),
                 **d_f = A.d<const double *>(P), **d_f0 = A.d<const double *>(P),
                 **d_mv = A.d<const double *>(P);
    const float **d_v32 = A.d<const float *>(P);
    double **d_c = A.d<double *>(P);
    uint8_t **d_act = A.d<uint8_t *>(P);
    BState *d_st = A.d<BState>(P), *d_st2 = A.d<BState>(P);
    double *d_part = A.d<double>((size_t)S * kBNV), *d_part2 = A.d<double>((size_t)S * kBNV),
           *d_pres = A.d<double>((size_t)P * kBNV);
    int *d_large = large.empty() ? nullptr : A.d<int>(large.size());
    double *d_shares = large.empty() ? nullptr : A.d<double>(large.size() * kBNV * kFinBlock);
    double *g = A.d<double>(R), *ks0 = A.d<double>(R), *ks1 = A.d<double>(R);
    uint8_t *mask = A.d<uint8_t>(R);
    // concatenated layout: vectors and the block-diagonal matrix
    std::vector<int64_t> ebase(P);
    int64_t E = 0;
    for (int p = 0; p < P; p++) {
        ebase[p] = E;
        E += K[p]->n > 0 ? K[p]->nsell : 0;
    }
    if (E >= (int64_t)1 << 31) return fail(ctx, NN_EINVAL, "batch too large: sliced-ELL entries must stay below 2^31");
    double *cg = A.d<double>(R), *fg = A.d<double>(R), *dg = A.d<double>(R);
    int *rlen = A.d<int>(R);
    double *ft = fg;   // a transient step's loads f + M c/dt are formed in place
    int *gso = A.d<int>(S + 1), *gcol = all_diag ? nullptr : A.d<int>(E);
    int64_t *d_ebase = A.d<int64_t>(P);
    double *gv64 = A.d<double>(E);
    float *gv32 = mixed ? A.d<float>(E) : nullptr;
    short *gd16 = quad || pair ? A.d<short>(E) : nullptr;
    BVec<double> V64{g, ks0, ks1, mask, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    BVec<float> V32{g, ks0, ks1, mask, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    if (mixed) {
        V32.w = A.d<float>(R), V32.r = A.d<float>(R), V32.z = A.d<float>(R);
        V32.p = A.d<float>(R), V32.q = A.d<float>(R), V32.dm = A.d<float>(R);
    } else {
        V64.w = A.d<double>(R), V64.r = A.d<double>(R), V64.z = A.d<double>(R);
        V64.p = A.d<double>(R), V64.q = A.d<double>(R), V64.dm = A.d<double>(R);
    }
    // Pinned host memory, in one allocation: a pair of hipHostMalloc and
    // hipHostFree takes 25 to 55 us, and a call has eighteen such arrays
    // (a backward-Euler step of three members of 59^2 rows 2.3 -> 1.6 ms, of four of
    // 55^3 10.4 -> 7.0).
    // Uploads from pinned memory read their source when they execute, so
    // the host writes each upload into a staging copy that it does not touch
    // again until the copy's event has completed.
    constexpr int kStage = 4;
    BState *hs, *land[2], *st_stage[kStage];
    double *pres;
    const void **tab;
    int *lst_stage[kStage];
    BBlk *blk_stage[kStage];
    BTab *tabs;
    {
        char *base = nullptr;
        for (int pass = 0; pass < 2 && A.ok; pass++) {   // sizes, then addresses
            size_t at = 0;
            auto take = [&](auto *&p, size_t n) {
                p = pass ? reinterpret_cast<std::decay_t<decltype(p)>>(base + at) : nullptr;
                at += (sizeof(*p) * n + 63) / 64 * 64;
            };
            take(hs, P);
            for (BState *&l : land) take(l, P);
            take(pres, (size_t)P * kBNV);
            take(tab, (size_t)P * 12);
            take(tabs, P);
            for (int k = 0; k < kStage; k++) {
                take(st_stage[k], P);
                take(lst_stage[k], (size_t)2 + P);
                take(blk_stage[k], S);
            }
            if (!pass) base = A.h<char>(at);
        }
    }
    if (!A.ok) return fail(ctx, NN_EOOM, "batch workspace allocation failed");
    Events ev_st, ev_lst, ev_land, ev_t;
    if (!ev_st.create(kStage, hipEventDisableTiming) ||
        !ev_land.create(2, hipEventDisableTiming) ||
        !ev_lst.create(kStage, hipEventDisableTiming) || !ev_t.create(2, hipEventDefault))
        return fail(ctx, NN_EHIP, "event creation");
    hipEvent_t t0 = ev_t.ev[0], t1 = ev_t.ev[1];

    // a transient step solves with the M/dt + K values, loads f + M c/dt
    for (int p = 0; p < P; p++) {
        tab[0 * P + p] = K[p]->sl_off;
        tab[1 * P + p] = K[p]->sl_col;
        tab[2 * P + p] = K[p]->rowptr;
        tab[3 * P + p] = transient ? K[p]->kt : K[p]->val;
        tab[4 * P + p] = transient ? K[p]->kt_diag : K[p]->diag;
        tab[5 * P + p] = transient ? (const void *)(ft + (size_t)s0[p] * kSlice) : f[p];
        tab[6 * P + p] = transient ? K[p]->kt32 : K[p]->val32;
        tab[7 * P + p] = c[p];
        tab[8 * P + p] = active ? active[p] : nullptr;
        tab[9 * P + p] = f[p];
        tab[10 * P + p] = K[p]->mval;
        tab[11 * P + p] = K[p]->sl_d16;
    }
    {
        void *dsts[12] = {d_so, d_sc, d_rp, d_v64, d_diag, d_f, d_v32, d_c, d_act, d_f0, d_mv, d_sd};
        for (int k = 0; k < 12; k++)
            NN_HIP_TRY(ctx, hipMemcpyAsync(dsts[k], tab + (size_t)k * P, sizeof(void *) * P,
                                           hipMemcpyHostToDevice, st));
        NN_HIP_TRY(ctx, hipMemcpyAsync(d_sprob, sprob.data(), sizeof(int) * S,
                                       hipMemcpyHostToDevice, st));
        NN_HIP_TRY(ctx, hipMemcpyAsync(d_s0, s0.data(), sizeof(int) * P, hipMemcpyHostToDevice, st));
        NN_HIP_TRY(ctx,
                   hipMemcpyAsync(d_nrow, nrow.data(), sizeof(int) * P, hipMemcpyHostToDevice, st));
        for (int p = 0, l = 0; p < P; p++) {
            BTab t{};
            t.share = nsl[p] > kBLarge ? l++ : -1;
            t.s0 = s0[p];
            t.nsl = nsl[p];
            t.nrow = nrow[p];
            if (all_diag && nrow[p] > 0) {
                t.W = K[p]->wmax <= 8 ? 7 : 15;
                t.reg = dreg[p];
                t.reg.b0 = (int)(ebase[p] + dreg[p].b0 - (int64_t)s0[p] * kSlice);
            }
            tabs[p] = t;
        }
        if (d_large)
            NN_HIP_TRY(ctx, hipMemcpyAsync(d_large, large.data(), sizeof(int) * large.size(),
                                           hipMemcpyHostToDevice, st));
        NN_HIP_TRY(ctx, hipMemcpyAsync(d_tab, tabs, sizeof(BTab) * P, hipMemcpyHostToDevice, st));
        NN_HIP_TRY(ctx, hipMemcpyAsync(d_ebase, ebase.data(), sizeof(int64_t) * P,
                                       hipMemcpyHostToDevice, st));
        const int e_total = (int)E;
        NN_HIP_TRY(ctx, hipMemcpyAsync(gso + S, &e_total, sizeof(int), hipMemcpyHostToDevice, st));
        // the pageable sources above must stay alive until the copies finish
        NN_HIP_TRY(ctx, hipStreamSynchronize(st));
    }
    BDev B;
    B.P = P;
    B.nslices = (int)S;
    B.cnt = d_list;
    B.plist = d_list + 2;
    B.blk = d_blk;
    B.tab = d_tab;
    B.sprob = d_sprob;
    B.s0 = d_s0;
    B.nrow = d_nrow;
    B.so = d_so;
    B.sc = d_sc;
    B.sd = d_sd;
    B.v64 = d_v64;
    B.v32 = d_v32;
    B.diag = d_diag;
    B.rowptr = d_rp;
    B.c = d_c;
    B.f = d_f;
    B.f0 = d_f0;
    B.mv = d_mv;
    B.act_out = d_act;
    B.st = d_st;
    B.st2 = d_st2;
    B.part = d_part;
    B.part2 = d_part2;
    B.pres = d_pres;
    B.large = d_large;
    B.shares = d_shares;
    B.gso = gso;
    B.gcol = gcol;
    B.gd16 = gd16;
    B.gv64 = gv64;
    B.gv32 = gv32;
    B.cg = cg;
    B.fg = fg;
    B.dg = dg;
    B.rlen = rlen;
    B.lo = o->lower;
    B.hi = o->upper;

    // ---- member states
    std::memset(hs, 0, sizeof(BState) * P);
    for (int p = 0; p < P; p++) {
        BState &M = hs[p];
        M.phase = nrow[p] > 0 ? PH_GRAD : PH_DONE;
        M.status = NN_OK;
        M.max_outer = o->max_outer;
        M.max_cg = o->max_cg;
        M.tcau = 1.0;
        M.delta = o->delta0 > 0.0 ? o->delta0 : INFINITY;
        M.tol = o->tol;
        M.rtol2 = o->inner_rtol * o->inner_rtol;
        M.n = (double)nrow[p];
        M.nnz = (double)K[p]->nnz;
        M.eb = entry_bytes(K[p], vb, all_diag, quad || pair);
        M.eg = entry_bytes(K[p], 8.0, all_diag, quad || pair);
        M.vb = vb;
        M.mixed = mixed ? 1 : 0;
    }
    int st_next = 0, lst_next = 0;
    auto push = [&]() {
        const int k = st_next;
        st_next = (st_next + 1) % kStage;
        if (hipEventSynchronize(ev_st.ev[k]) != hipSuccess) return false;
        std::memcpy(st_stage[k], hs, sizeof(BState) * P);
        return hipMemcpyAsync(d_st, st_stage[k], sizeof(BState) * P, hipMemcpyHostToDevice, st) ==
                   hipSuccess &&
               hipEventRecord(ev_st.ev[k], st) == hipSuccess;
    };
    // The states as the chunk enqueued last leaves them: pull(k) into landing
    // buffer k; look(k) waits for it and makes them the states in hs.
    auto pull = [&](int k) {
        return hipMemcpyAsync(land[k], d_st, sizeof(BState) * P, hipMemcpyDeviceToHost, st) ==
                   hipSuccess &&
               hipEventRecord(ev_land.ev[k], st) == hipSuccess;
    };
    auto look = [&](int k) {
        if (hipEventSynchronize(ev_land.ev[k]) != hipSuccess) return false;
        std::memcpy(hs, land[k], sizeof(BState) * P);
        return true;
    };
    // The members still running and their blocks, as device lists: rebuilt
    // and uploaded only when the set changes.  A block takes `per` slices of
    // one member, four at a time (one per wavefront): as many as spread the
    // running slices over kBGrid blocks, at most kBMost (results do not depend
    // on it).
    std::vector<char> sel(P, 0), sel_cur(P, 2);
    int n_bl = 0, n_pr = 0;
    auto select = [&]() -> bool {
        bool same = true;
        for (int p = 0; p < P; p++) {
            sel[p] = hs[p].phase != PH_DONE ? 1 : 0;
            same = same && sel[p] == sel_cur[p];
        }
        if (same) return true;
        const int k = lst_next;
        lst_next = (lst_next + 1) % kStage;
        if (hipEventSynchronize(ev_lst.ev[k]) != hipSuccess) return false;
        int *h = lst_stage[k];
        BBlk *bl = blk_stage[k];
        int np = 0, nb = 0;
        int64_t ns = 0;
        for (int p = 0; p < P; p++)
            if (sel[p]) ns += nsl[p];
        const int per = (int)std::min<int64_t>(
            kBMost, std::max<int64_t>(1, (ns + (int64_t)kBGrid * kBWaves - 1) / ((int64_t)kBGrid * kBWaves)) * kBWaves);
        for (int p = 0; p < P; p++) {
            sel_cur[p] = sel[p];
            if (!sel[p]) continue;
            h[2 + np++] = p;
            for (int t = 0; t < nsl[p]; t += per)
                bl[nb++] = BBlk{p, s0[p] + t, std::min(per, nsl[p] - t), t == 0 ? 1 : 0};
        }
        h[0] = nb;
        h[1] = np;
        n_bl = nb;
        n_pr = np;
        return hipMemcpyAsync(d_list, h, sizeof(int) * ((size_t)2 + np), hipMemcpyHostToDevice, st) ==
                   hipSuccess &&
               (nb == 0 || hipMemcpyAsync(d_blk, bl, sizeof(BBlk) * nb, hipMemcpyHostToDevice, st) ==
                               hipSuccess) &&
               hipEventRecord(ev_lst.ev[k], st) == hipSuccess;
    };

    int num_cu = 256;
    {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, ctx->device) == hipSuccess && prop.multiProcessorCount > 0)
            num_cu = prop.multiProcessorCount;
    }
    auto grid_for = [&](int blocks) { return (unsigned)std::max(1, blocks); };

    NN_HIP_TRY(ctx, push() ? hipSuccess : hipErrorUnknown);
    NN_HIP_TRY(ctx, select() ? hipSuccess : hipErrorUnknown);
    NN_HIP_TRY(ctx, hipEventRecord(t0, st));

    // ---- transient right-hand sides (from c^n, before the start point is set)
    if (transient)
        NN_BDISPATCH(wmax, (kb_transient_rhs<WM>), grid_for(n_bl), kFinBlock, st, B, dt, ft);
    // ---- the members into the concatenated layout
    {
        const int64_t blocks = std::min<int64_t>((S + 3) / 4, (int64_t)num_cu * 8);
        hipLaunchKernelGGL(kb_gather, dim3((int)std::max<int64_t>(blocks, 1)), dim3(256), 0, st, B,
                           (const int64_t *)d_ebase, gso, gcol, gd16, gv64, gv32, dg, rlen,
                           transient ? 0 : 1, layout);
    }
    // ---- start point and load statistics
    hipLaunchKernelGGL(kb_init, dim3(grid_for(n_bl)), dim3(kFinBlock), 0, st, B,
                       o->c0_mode == 1 ? 1 : 0, std::min(std::max(o->c0_value, o->lower), o->upper));
    hipLaunchKernelGGL(kb_reduce_init, dim3(std::max(n_pr, 1)), dim3(kFinBlock), 0, st, B);
    NN_HIP_TRY(ctx, hipMemcpyAsync(pres, d_pres, sizeof(double) * P * kBNV, hipMemcpyDeviceToHost,
                                   st));
    NN_HIP_TRY(ctx, hipStreamSynchronize(st));
    for (int p = 0; p < P; p++) {
        BState &M = hs[p];
        if (M.phase == PH_DONE) continue;
        const double *r = &pres[(size_t)p * kBNV];
        M.normf = std::sqrt(r[0]);
        M.bytes += 16.0 * nrow[p];
        if (r[2] != 0.0 || r[3] != 0.0) {
            M.status = NN_ENONFINITE;
            M.phase = PH_DONE;
        } else if (o->lower == 0.0 && !(r[1] > 0.0)) {
            // f <= 0 with lower bound 0: c = 0 satisfies c >= 0, g = -f >= 0, c.g = 0
            NN_HIP_TRY(ctx, hipMemsetAsync(cg + (size_t)s0[p] * kSlice, 0,
                                           sizeof(double) * nrow[p], st));
            M.n_active = nrow[p];
            M.phase = PH_DONE;
        }
    }
    NN_HIP_TRY(ctx, push() ? hipSuccess : hipErrorUnknown);
    NN_HIP_TRY(ctx, select() ? hipSuccess : hipErrorUnknown);

    // ---- one global step on stream s with gr blocks, the row and vector passes
    // optionally recording their own begin and end into ev[0..1] and ev[2..3]
    auto step = [&](hipStream_t s, unsigned gr, hipEvent_t *ev) {
        hipEvent_t e0 = ev ? ev[0] : nullptr, e1 = ev ? ev[1] : nullptr;
        if (all_diag && mixed)
            NN_BDISPATCH_EV(wmax, (kb_rows<WM, CM_DIAG, float, float>), gr, kFinBlock, s, e0, e1, B,
                            (const float *)gv32, V32);
        else if (all_diag)
            NN_BDISPATCH_EV(wmax, (kb_rows<WM, CM_DIAG, double, double>), gr, kFinBlock, s, e0, e1, B,
                            (const double *)gv64, V64);
        else if (quad)
            NN_BDISPATCH_EV(wmax, (kb_rows<WM, CM_Q4, float, float>), gr, kFinBlock, s, e0, e1, B,
                            (const float *)gv32, V32);
        else if (mixed)
            NN_BDISPATCH_EV(wmax, (kb_rows<WM, CM_I32, float, float>), gr, kFinBlock, s, e0, e1, B,
                            (const float *)gv32, V32);
        else if (pair)
            NN_BDISPATCH_EV(wmax, (kb_rows<WM, CM_P2, double, double>), gr, kFinBlock, s, e0, e1, B,
                            (const double *)gv64, V64);
        else
            NN_BDISPATCH_EV(wmax, (kb_rows<WM, CM_I32, double, double>), gr, kFinBlock, s, e0, e1, B,
                            (const double *)gv64, V64);
        const unsigned ns = (unsigned)(large.size() * kBNV * kBWaves);
        if (ns) hipLaunchKernelGGL(kb_share<false>, dim3(ns), dim3(64), 0, s, B);
        e0 = ev ? ev[2] : nullptr, e1 = ev ? ev[3] : nullptr;
        if (mixed) NN_BLAUNCH_EV((kb_vec<float>), gr, kFinBlock, s, e0, e1, B, V32);
        else NN_BLAUNCH_EV((kb_vec<double>), gr, kFinBlock, s, e0, e1, B, V64);
        if (ns) hipLaunchKernelGGL(kb_share<true>, dim3(ns), dim3(64), 0, s, B);
    };
    // the last transition of a chunk
    auto settle = [&](hipStream_t s, int members) {
        hipLaunchKernelGGL(kb_step2, dim3(std::max(members, 1)), dim3(kFinBlock), 0, s, B);
    };

    // ---- chunks of global steps.  Without profiling a chunk is captured
    // into a graph on the context's private capture stream (the caller's
    // stream may be the legacy default stream, which cannot be captured) and
    // replayed on the caller's stream, one graph per size class of the
    // running list.  With profiling on, or if capture fails, steps are
    // launched one by one (with profiling, one step per chunk, each pass
    // bracketed by events).
    const int chunk = o->cg_chunk > 0 ? o->cg_chunk : 16;
    GraphCache graphs;
    bool use_graph = NNQP_BATCH_GRAPH && !ctx->prof;
    if (use_graph && !ctx->cap_stream &&
        hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking) != hipSuccess) {
        ctx->cap_stream = nullptr;
        use_graph = false;
    }
    auto graph_for = [&](int blocks) -> hipGraphExec_t {
        int cls = 0;
        while ((1 << cls) < blocks) cls++;
        auto it = graphs.by_class.find(cls);
        if (it != graphs.by_class.end()) return it->second.exec;
        const unsigned gr = 1u << cls;
        const int fg = std::min(P, 1 << cls);   // a listed member owns at least one block
        if (hipStreamBeginCapture(ctx->cap_stream, hipStreamCaptureModeRelaxed) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        for (int k = 0; k < chunk; k++) step(ctx->cap_stream, gr, nullptr);
        settle(ctx->cap_stream, fg);
        hipGraph_t gph = nullptr;
        const bool ended = hipStreamEndCapture(ctx->cap_stream, &gph) == hipSuccess && gph;
        (void)hipGetLastError();
        if (!ended) {
            if (gph) (void)hipGraphDestroy(gph);
            return nullptr;
        }
        hipGraphExec_t ex = nullptr;
        if (hipGraphInstantiate(&ex, gph, nullptr, nullptr, 0) != hipSuccess || !ex) {
            (void)hipGraphDestroy(gph);
            (void)hipGetLastError();
            return nullptr;
        }
        graphs.by_class[cls] = GraphCache::G{gph, ex};
        return ex;
    };
    Events ev_step;
    if (ctx->prof && !ev_step.create(4, hipEventDefault))
        return fail(ctx, NN_EHIP, "event creation");

    // Every member's step count is bounded by its caps (outer iterations,
    // trials per search, CG iterations); the guard only stops a runaway loop.
    const int64_t max_steps =
        (int64_t)(o->max_outer + 1) * (4 + 2 * kMaxTrials + 21 + o->max_cg) + 16;
    nn_status err = NN_OK;
    int64_t steps = 0, chunks = 0;
    while (steps < max_steps) {
        if (!select()) {
            err = fail(ctx, NN_EHIP, "batch list upload");
            break;
        }
        if (n_pr == 0) break;
        const unsigned gr = grid_for(n_bl);
        if (ctx->prof) {
            // one step; algorithmic bytes of the row pass from the states
            double brow = 0.0, brow_csr = 0.0;
            for (int p = 0; p < P; p++)
                if (hs[p].phase != PH_DONE) {
                    brow += row_bytes(hs[p]);
                    brow_csr += row_bytes_csr(hs[p]);
                }
            step(st, gr, ev_step.ev.data());
            settle(st, n_pr);
            steps++;
            if (!pull(0) || !look(0)) {
                err = fail(ctx, NN_EHIP, "batch read-back");
                break;
            }
            float m1 = 0.f, m2 = 0.f;
            if (brow > 0.0 && ((ctx->prof_mask >> KC_CG_SPMV) & 1) &&
                hipEventElapsedTime(&m1, ev_step.ev[0], ev_step.ev[1]) == hipSuccess)
                prof_add(ctx, KC_CG_SPMV, m1, brow, brow_csr);
            if (((ctx->prof_mask >> KC_CG_UPDATE) & 1) &&
                hipEventElapsedTime(&m2, ev_step.ev[2], ev_step.ev[3]) == hipSuccess)
                prof_add(ctx, KC_CG_UPDATE, m2, 0.0);
            (void)hipGetLastError();
            continue;
        }
        hipGraphExec_t ex = use_graph ? graph_for(n_bl) : nullptr;
        if (ex) {
            if (hipGraphLaunch(ex, st) != hipSuccess) {
                err = fail(ctx, NN_EHIP, "graph launch");
                break;
            }
        } else {
            for (int k = 0; k < chunk; k++) step(st, gr, nullptr);
            settle(st, n_pr);
        }
        steps += chunk;
        // One chunk stays enqueued behind the one whose states are looked at,
        // so the device does not wait for the read-back, the list and the
        // launch (85 us a chunk, where its 16 steps take 360 on 64 members of
        // 32^2 to 256^2 cells).  The lists lag by a chunk: a member that has
        // finished returns from its launches at once.
        const int k = chunks++ & 1;
        if (!pull(k) || (chunks > 1 && !look(k ^ 1))) {
            err = fail(ctx, NN_EHIP, "batch read-back");
            break;
        }
        if (o->verbose) {
            int nr = 0, ncg = 0;
            for (int p = 0; p < P; p++) {
                nr += hs[p].phase != PH_DONE ? 1 : 0;
                ncg += hs[p].phase == PH_CG ? 1 : 0;
            }
            std::fprintf(stderr,
                         "nnqp batch step %lld: %d of %d members running (%d in CG); member 0: "
                         "outer %d kkt %.3e\n",
                         (long long)steps, nr, P, ncg, hs[0].outer, hs[0].kkt_rel);
        }
    }
    // (after the last look every member had finished, or the guard has hit)
    if (err == NN_OK && chunks > 0 && !look((int)((chunks - 1) & 1)))
        err = fail(ctx, NN_EHIP, "batch read-back");
    if (err == NN_OK && steps >= max_steps) {
        for (int p = 0; p < P; p++)
            if (hs[p].phase != PH_DONE) {
                hs[p].status = NN_EMAXIT;
                hs[p].phase = PH_DONE;
            }
    }
    // ---- outputs: the solutions back into the members' vectors, active sets
    {
        const int64_t blocks = std::min<int64_t>((S + 3) / 4, (int64_t)num_cu * 8);
        hipLaunchKernelGGL(kb_scatter, dim3((int)std::max<int64_t>(blocks, 1)), dim3(256), 0, st, B);
    }
    (void)hipEventRecord(t1, st);
    const hipError_t e = hipEventSynchronize(t1);
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, t0, t1);
    prof_collect(ctx);
    if (err != NN_OK) return err;
    if (e != hipSuccess) return fail(ctx, NN_EHIP, hipGetErrorString(e));
    int first_bad = -1;
    for (int p = 0; p < P; p++) {
        const BState &M = hs[p];
        nn_stats &Q = SP[p];
        Q.kkt_rel = M.kkt_rel;
        Q.kkt_nat_inf = M.kkt_nat;
        Q.min_c = M.min_c;
        Q.norm_f = M.normf;
        Q.outer_its = M.outer;
        Q.cg_its = M.cg_its;
        Q.spmvs = M.spmvs;
        Q.n_active = M.n_active;
        Q.cauchy_trials = M.cauchy_trials;
        Q.search_trials = M.search_trials;
        Q.refinements = M.refinements;
        Q.status = M.status;
        Q.bytes_moved = M.bytes;
        Q.seconds = ms * 1e-3;   // the whole batched call
        if (M.status != NN_OK && first_bad < 0) first_bad = p;
    }
    if (stats)
        for (int p = 0; p < P; p++) stats[p] = SP[p];
    if (first_bad >= 0) {
        char msg[160];
        std::snprintf(msg, sizeof(msg),
                      "batch member %d (the first affected) ended with status %d; every member's "
                      "status is in its stats",
                      first_bad, hs[first_bad].status);
        return fail(ctx, (nn_status)hs[first_bad].status, msg);
    }
    ctx->err.clear();
    return NN_OK;
}

}  // namespace nnqp
