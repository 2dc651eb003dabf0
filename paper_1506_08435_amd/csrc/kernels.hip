// Row-parallel kernels of the non-negative QP solver for gfx950.
//
// Every kernel here is bound by HBM bandwidth (sparse matrix-vector products
// at ~0.14 flop/byte and vector streams), so the design goal is bytes and
// latency, not flops:
//  - K is held in sliced-ELL form (64-row slices, one lane per row, entries
//    column-major within a slice): a wavefront's index/value loads are single
//    contiguous segments, each lane issues all of its row's loads before the
//    first gather, and the row sum is a plain sequential chain (no cross-lane
//    shuffles, fixed order);
//  - vector updates and dot products are fused into the passes that already
//    touch the same rows;
//  - reductions leave one partial per block and are never combined with
//    atomics: what the host reads is combined by a launch that publishes it
//    (k_publish), and the CG scalars by every block of the next kernel, in the
//    same fixed order, so results are bitwise reproducible and no cross-XCD
//    synchronisation is needed inside a kernel.
#include <cmath>

#include "nnqp_internal.hpp"
#include "diag.hpp"

namespace nnqp {

// Neighbouring blocks share an XCD where that was measured faster: passes with
// one slice per wavefront at most (up to 524,288 rows: solves of 63^3, 71^3 and
// the holed cube of k = 9 12.0 -> 11.5, 21.4 -> 19.9, 26.1 -> 24.5 ms, 79^3 Galerkin
// 12.2 -> 10.7), and float32 passes of any size (100^3, 127^3: 26.4 -> 23.9,
// 79.8 -> 78.7 ms).  Larger float64 passes stream from HBM, where it costs some
// sizes more than the reuse gives others (81^3, 89^3, 99^3, 127^3 rows:
// 32.7 -> 31.4, 31.5 -> 32.7, 40.0 -> 38.9, 130.6 -> 138.9 ms); no rule in the
// size parts them, so they keep the order whose worst case is the smaller loss.
Part make_part(int64_t n, int max_blocks, bool f32)
{
    Part p;
    p.n = (int)n;
    int64_t nb = (p.nslices() + kWaves - 1) / kWaves;
    if (nb < 1) nb = 1;
    if (nb > max_blocks) nb = max_blocks;
    p.nb = (int)nb;
    if (f32 || p.nslices() <= nb * kWaves) {
        const int64_t last = (p.nslices() % (nb * kWaves) + kWaves - 1) / kWaves;
        p.heavy = (int)(last < nb ? last : 0);
    }
    return p;
}

// ---------------------------------------------------------------- kernels
template <int WMAX, class Cols>
__global__ __launch_bounds__(kBlock, walk_waves<Cols>()) void k_matvec(Part P, const int *__restrict__ so, Cols sc,
                                                   const double *__restrict__ v,
                                                   const double *__restrict__ x, double *__restrict__ y)
{
    walk_rows<WMAX>(P, so, sc, v, AllRows(), NoPre(), [&](int ub, int l) { return (x + ub)[l]; },
                    [&](int i, double s, int) { y[i] = s; });
}

// ft = f + (M c) / dt
template <int WMAX, class Cols>
__global__ __launch_bounds__(kBlock, walk_waves<Cols>()) void k_transient_rhs(Part P, const int *__restrict__ so, Cols sc,
                                                          const double *__restrict__ m,
                                                          const double *__restrict__ c,
                                                          const double *__restrict__ f, double dt,
                                                          double *__restrict__ ft)
{
    walk_rows<WMAX>(P, so, sc, m, AllRows(), [&](int i) { return f[i]; },
                    [&](int ub, int l) { return (c + ub)[l]; },
                    [&](int i, double s, double fi) { ft[i] = fi + s / dt; });
}

// g = K c - f with the projected-gradient report:
// |pg|^2, #non-finite, ||c - P(c - g)||_inf, min c, #(c at a bound)
// pg_i = g_i strictly inside [lo, hi], min(g_i, 0) at lo, max(g_i, 0) at hi;
// the natural residual c - P(c - g) = max(c - hi, min(g, c - lo)) (min(c, g)
// for [0, inf)).
constexpr uint32_t kOpsGrad = OPS5(OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM);

template <int WMAX, class Cols>
__global__ __launch_bounds__(kBlock, walk_waves<Cols>()) void k_grad(Part P, const int *__restrict__ so, Cols sc,
                                                 const double *__restrict__ v,
                                                 const double *__restrict__ c,
                                                 const double *__restrict__ f,
                                                 double *__restrict__ g, double *partials, Box B)
{
    double a[5];
    red_init<kOpsGrad, 5>(a);
    walk_rows<WMAX>(P, so, sc, v, AllRows(), [&](int i) { return Two{c[i], f[i]}; },
                    [&](int ub, int l) { return (c + ub)[l]; }, [&](int i, double s, Two cf) {
        const double gi = s - cf.b;
        const double cv = cf.a;
        g[i] = gi;
        const double pg = cv > B.lo ? (cv < B.hi ? gi : fmax(gi, 0.0)) : fmin(gi, 0.0);
        a[0] += pg * pg;
        a[1] += (isfinite(gi) && isfinite(cv)) ? 0.0 : 1.0;
        a[2] = fmax(a[2], fabs(fmax(cv - B.hi, fmin(gi, cv - B.lo))));
        a[3] = fmin(a[3], cv);
        a[4] += (cv == B.lo || cv == B.hi) ? 1.0 : 0.0;
    });
    block_partial<kOpsGrad, 5>(a, slot_ptr(partials, SLOT_HOST), block_id(P));
}

// Residual report of an unconstrained solve: r = K c - f (not stored);
// |r|^2, #non-finite, max c, min c, #(c < 0)
constexpr uint32_t kOpsResid = OPS5(OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM);

template <int WMAX, class Cols>
__global__ __launch_bounds__(kBlock, walk_waves<Cols>()) void k_resid(Part P, const int *__restrict__ so, Cols sc,
                                                  const double *__restrict__ v,
                                                  const double *__restrict__ c,
                                                  const double *__restrict__ f, double *partials)
{
    double a[5];
    red_init<kOpsResid, 5>(a);
    walk_rows<WMAX>(P, so, sc, v, AllRows(), [&](int i) { return Two{c[i], f[i]}; },
                    [&](int ub, int l) { return (c + ub)[l]; }, [&](int, double s, Two cf) {
                        const double ri = s - cf.b;
                        a[0] += ri * ri;
                        a[1] += (isfinite(ri) && isfinite(cf.a)) ? 0.0 : 1.0;
                        a[2] = fmax(a[2], cf.a);
                        a[3] = fmin(a[3], cf.a);
                        a[4] += cf.a < 0.0 ? 1.0 : 0.0;
                    });
    block_partial<kOpsResid, 5>(a, slot_ptr(partials, SLOT_HOST), block_id(P));
}

// c += w (no projection: the unconstrained solve)
template <class VV>
__global__ __launch_bounds__(kBlock) void k_add(Part P, double *__restrict__ c,
                                                const VV *__restrict__ w)
{
    for_rows(P, [&](int i, bool act) {
        if (act) c[i] += (double)w[i];
    });
}

// Trial point of a projected search: s = P(c + t d) - c, formed for every
// gathered column; ks = K s; report g.s, s.Ks, s.s.  Rows with mask == 0 are
// skipped when a mask is given (there d = 0, so s = 0 and they add nothing).
// BRK: the breakpoint pass (k_breakpoint) of the same direction in the same
// launch, its values into SLOT_Q; it reads nothing that the trial's rows have
// not loaded, so a launch of its own (3.8 us on 250 k rows, 18 us on 2 M)
// goes.
constexpr uint32_t kOpsTrial = OPS3(OP_SUM, OP_SUM, OP_SUM);
constexpr uint32_t kOpsBrk = OPS3(OP_MIN, OP_SUM, OP_SUM);

// Largest step along w before a free variable reaches a bound:
// min over w_i < 0 of (c_i - lo) / (-w_i) and over w_i > 0 of (hi - c_i) / w_i
// (+inf for hi = +inf), g.w, w.w
__device__ __forceinline__ void breakpoint(double ci, double wi, double gi, const Box &B, double (&a)[3])
{
    if (wi < 0.0) a[0] = fmin(a[0], (ci - B.lo) / (-wi));
    else if (wi > 0.0) a[0] = fmin(a[0], (B.hi - ci) / wi);
    a[1] += gi * wi;
    a[2] += wi * wi;
}

template <int WMAX, class VT, class VD, class Cols, bool BRK>
__global__ __launch_bounds__(kBlock, BRK ? 8 : walk_waves<Cols>()) void k_trial(Part P, const int *__restrict__ so, Cols sc,
                                                  const VT *__restrict__ v,
                                                  const double *__restrict__ c,
                                                  const VD *__restrict__ d, double t,
                                                  const double *__restrict__ g,
                                                  const uint8_t *__restrict__ mask,
                                                  double *__restrict__ ks, double *partials, Box B)
{
    auto sv = [&](int ub, int l) {
        const double cj = (c + ub)[l];
        return proj_box(cj + t * (double)(d + ub)[l], B) - cj;
    };
    double a[3], brk[3];
    red_init<kOpsTrial, 3>(a);
    red_init<kOpsBrk, 3>(brk);
    walk_rows<WMAX, 5>(P, so, sc, v, [&](int i) { return mask == nullptr || mask[i] != 0; },
                    [&](int i) { return Two{sv(0, i), g[i]}; }, sv, [&](int i, double s, Two sg) {
                        if (ks) ks[i] = s;
                        const double si = sg.a;
                        a[0] += sg.b * si;
                        a[1] += si * s;
                        a[2] += si * si;
                        if constexpr (BRK) breakpoint(c[i], (double)d[i], sg.b, B, brk);
                    });
    block_partial<kOpsTrial, 3>(a, slot_ptr(partials, SLOT_HOST), block_id(P));
    if constexpr (BRK) block_partial<kOpsBrk, 3>(brk, slot_ptr(partials, SLOT_Q), block_id(P));
}

// Cauchy ladder: the projected steepest-descent trial s_k = P(c - t_k g) - c
// for kLadder step lengths in one matrix pass (the entries are read once and
// each gathered column yields all kLadder trial values); ks_k = K s_k; per k
// the sums g.s_k, s_k.Ks_k, s_k.s_k as values 3k, 3k+1, 3k+2 of a
// 3 kLadder-value partial starting at SLOT_U0 (it may span SLOT_U1).
struct Ladder {
    double t[kLadder];
    double *ks[kLadder];
};

#ifndef NNQP_LADDER_PHASE
// entries per load phase of the Cauchy ladder pass (the diagonal layout's walk
// takes five)
#define NNQP_LADDER_PHASE 4
#endif

template <int WMAX, class VT, class Cols>
__global__ __launch_bounds__(kBlock) void k_ladder(Part P, const int *__restrict__ so, Cols sc,
                                                   const VT *__restrict__ v,
                                                   const double *__restrict__ c,
                                                   const double *__restrict__ g, Ladder L, Box B,
                                                   double *partials)
{
    double a[3 * kLadder];
#pragma unroll
    for (int k = 0; k < 3 * kLadder; k++) a[k] = 0.0;
    auto trials = [&](int ub, int l, double (&out)[kLadder]) {
        const double cj = (c + ub)[l], gj = (g + ub)[l];
#pragma unroll
        for (int k = 0; k < kLadder; k++) out[k] = proj_box(cj - L.t[k] * gj, B) - cj;
    };
    auto pre = [&](int i) { return Two{c[i], g[i]}; };
    auto epi = [&](int i, double (&kv)[kLadder], Two cg) {
        double si[kLadder];
        trials(0, i, si);
#pragma unroll
        for (int k = 0; k < kLadder; k++) {
            L.ks[k][i] = kv[k];
            a[3 * k] += cg.b * si[k];
            a[3 * k + 1] += si[k] * kv[k];
            a[3 * k + 2] += si[k] * si[k];
        }
    };
    // the nine running sums stay in registers for the whole pass, so the
    // entries load NNQP_LADDER_PHASE at a time
    walk_rows_n<WMAX, kLadder, NNQP_LADDER_PHASE>(P, so, sc, v, pre, trials, epi);
    block_partial<0u, 3 * kLadder>(a, slot_ptr(partials, SLOT_U0), block_id(P));
}

// c = P(c + t d)
template <class VD>
__global__ __launch_bounds__(kBlock) void k_apply(Part P, double *__restrict__ c,
                                                  const VD *__restrict__ d, double t, Box B)
{
    for_rows(P, [&](int i, bool act) {
        if (act) c[i] = proj_box(c[i] + t * (double)d[i], B);
    });
}

// c = c0v (mode 0) or c = P(c) (mode 1); report |f|^2, max f, #non-finite f,
// #non-finite c (before projection)
constexpr uint32_t kOpsInit = OPS4(OP_SUM, OP_MAX, OP_SUM, OP_SUM);

__global__ __launch_bounds__(kBlock) void k_init(Part P, double *__restrict__ c,
                                                 const double *__restrict__ f, int mode, double c0v,
                                                 double *partials, Box B)
{
    double a[4];
    red_init<kOpsInit, 4>(a);
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        const double fi = f[i];
        a[0] += fi * fi;
        a[1] = fmax(a[1], fi);
        a[2] += isfinite(fi) ? 0.0 : 1.0;
        if (mode == 0) {
            c[i] = c0v;
        } else {
            const double cv = c[i];
            a[3] += isfinite(cv) ? 0.0 : 1.0;
            c[i] = proj_box(cv, B);
        }
    });
    block_partial<kOpsInit, 4>(a, slot_ptr(partials, SLOT_HOST), block_id(P));
}

// Set-up of the inner CG on the face of (c, g + ks), behind the Cauchy step
// c <- P(c + t g) of length t (t != 0; a launch of its own before: 3.3 us on
// 250 k rows, and c and g twice):
//   g <- g + ks (gradient at the Cauchy point), free = not (c == 0 and g >= 0),
//   dm = 1/diag on free rows and 0 elsewhere (the mask folded into the
//   Jacobi preconditioner), r = -g on free rows, z = dm r, p = q = w = 0.
// Partials (SLOT_U0): r.z, r.r, #free, nnz of free rows.
constexpr uint32_t kOpsU = OPS4(OP_SUM, OP_SUM, OP_SUM, OP_SUM);

template <class VV>
__global__ __launch_bounds__(kBlock) void k_cg_setup(
    Part P, const int *__restrict__ rp, const double *__restrict__ diag,
    double *__restrict__ c, double *__restrict__ g, const double *__restrict__ ks, double t,
    uint8_t *__restrict__ mask, VV *__restrict__ dm, VV *__restrict__ r, VV *__restrict__ z,
    VV *__restrict__ p, VV *__restrict__ q, VV *__restrict__ w, double *partials, DevScalars *S,
    Box B, int face, VV *__restrict__ cres, VV *__restrict__ cdz0, VV *__restrict__ cdz1,
    double inv_theta)
{
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        double cv = c[i], gi = g[i];
        if (t != 0.0) {
            cv = proj_box(cv + t * gi, B);
            c[i] = cv;
        }
        if (ks) {
            gi = gi + ks[i];
            g[i] = gi;
        }
        const bool fr = face == FACE_ALL ? true
                      : face == FACE_INTERIOR ? (cv != B.lo && cv != B.hi)
                      : !((cv == B.lo && gi >= 0.0) || (cv == B.hi && gi <= 0.0));
        const VV dmi = fr ? (VV)(1.0 / diag[i]) : VV(0);
        const VV ri = fr ? (VV)(-gi) : VV(0);
        // Jacobi z = dm r, or the first Chebyshev term dm r / theta
        const VV zi = cres ? (VV)((double)dmi * (double)ri * inv_theta) : dmi * ri;
        mask[i] = fr ? 1 : 0;
        dm[i] = dmi;
        r[i] = ri;
        z[i] = zi;
        p[i] = VV(0);
        q[i] = VV(0);
        w[i] = VV(0);
        if (cres) {
            cres[i] = ri;
            cdz0[i] = zi;
            cdz1[i] = VV(0);
        }
        a[0] += (double)ri * (double)zi;
        a[1] += (double)ri * (double)ri;
        a[2] += fr ? 1.0 : 0.0;
        a[3] += fr ? (double)(rp[i + 1] - rp[i]) : 0.0;
    });
    block_partial<kOpsU, 4>(a, slot_ptr(partials, SLOT_U0), block_id(P));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        S->done = 0;
        S->it = 0;
        S->ww[0] = 0.0;   // w = 0
        S->tr_hit = 0;
    }
}

// CG iteration j, matrix pass.
// Prologue (identical in every block): r.z_j and r.r_j from the partials the
// previous kernel left in slot U[j%2]; stop if r.r_j <= rtol^2 r.r_0, at the
// iteration cap, or when the previous update stopped on the trust-region
// boundary; beta_j = r.z_j / r.z_{j-1} (0 for j = 0).
// Body: the direction update p <- z + beta p and its product q = K p are
// formed together, using K p = K z + beta (K p_old): only z is gathered, and
// p, q are updated in place on the free rows; partials of p.q into SLOT_Q
// (with TR, also p.p and w.p, which the update needs for |w + alpha p|).
// Columns outside the free set contribute 0 because z vanishes there.
// The CG solve has ended: its scalars to the host (one thread, behind its own
// stores to them).
__device__ inline void flow_end(const CgLink &L)
{
    L.F->scal = *L.S;
    __hip_atomic_store(&L.F->end, (unsigned long long)L.epoch, __ATOMIC_RELEASE,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// The prologue's scalars, read before anything else of the pass.
struct CgIn {
    double rr_stop, rz_old;
    int tr_hit;
};
__device__ __forceinline__ CgIn cg_in(const DevScalars *S, int j)
{
    return CgIn{S->rr_stop, S->rzh[(j - 1) & 1], S->tr_hit};
}

// u: this thread's partials of r.z and r.r.  Returns the iteration's beta and
// whether the CG ends here.
template <bool TR>
__device__ __forceinline__ bool cg_begin(const CgIn &in, const double *slot, int nb, double (&u)[2],
                                         const CgLink &L, int j, int max_it, double rtol2,
                                         double &beta)
{
    DevScalars *const S = L.S;
    combine_loaded<0u, 2>(u);
    double cnt[2] = {0.0, 0.0};   // #free rows and their nonzeros, from the set-up
    if (j == 0) {
        load_partials<0u, 2>(slot + 2 * kMaxBlocks, nb, cnt);
        __syncthreads();
        combine_loaded<0u, 2>(cnt);
    }
    const double rz = u[0], rr2 = u[1];
    const double rr_stop = j == 0 ? rtol2 * rr2 : in.rr_stop;
    int done = 0;
    if (TR && j > 0 && in.tr_hit) done = 2;
    else if (!isfinite(rz) || !isfinite(rr2)) done = 4;
    else if ((j == 0 && (rr2 == 0.0 || cnt[0] == 0.0)) || (j > 0 && rr2 <= rr_stop) ||
             j >= max_it || !(rz > 0.0))
        done = 1;
    beta = j == 0 ? 0.0 : rz / in.rz_old;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (j == 0) {
            S->rr_stop = rr_stop;
            S->n_free = cnt[0];
            S->nnz_free = cnt[1];
        }
        S->rzh[j & 1] = rz;
        if (done) {
            S->done = done;
            S->it = j;
            flow_end(L);
        } else {
            __hip_atomic_store(&L.F->cg, ((unsigned long long)L.epoch << 32) | (unsigned)(j + 1),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    return done != 0;
}

template <int WMAX, class VT, class VV, class Cols, bool TR>
__global__ __launch_bounds__(kBlock, walk_waves<Cols>()) void k_cg_spmv(Part P0, const int *__restrict__ so, Cols sc,
                                                    const VT *__restrict__ v,
                                                    const uint8_t *__restrict__ mask,
                                                    const VV *__restrict__ z,
                                                    VV *__restrict__ p, VV *__restrict__ q,
                                                    const VV *__restrict__ w,
                                                    double *partials, CgLink L, int j,
                                                    int max_it, double rtol2)
{
    // (what the launcher's choice of the kernel says about make_part's)
    Part P = P0;
    if constexpr (std::is_same_v<Cols, ColsDiag> && std::is_same_v<VV, double>) P.heavy = -1;
    const DevScalars *const S = L.S;
    if (S->done) return;
    const CgIn in = cg_in(S, j);
    const double *slot = slot_ptr(partials, (j & 1) ? SLOT_U1 : SLOT_U0);
    double u[2], beta;
    load_partials<0u, 2>(slot, P.nb, u);
    if (cg_begin<TR>(in, slot, P.nb, u, L, j, max_it, rtol2, beta)) return;
    constexpr int NQ = TR ? 3 : 1;
    double a[NQ];
#pragma unroll
    for (int k = 0; k < NQ; k++) a[k] = 0.0;
    walk_rows<WMAX>(P, so, sc, v, [&](int i) { return mask[i] != 0; },
                    [&](int i) { return Three{(double)p[i], (double)q[i], (double)z[i]}; },
                    [&](int ub, int l) { return (z + ub)[l]; },
                    [&](int i, double kz, Three pqz) {
                        const VV pi = (VV)fma(beta, pqz.a, pqz.c);
                        const VV qi = (VV)fma(beta, pqz.b, kz);
                        p[i] = pi;
                        q[i] = qi;
                        a[0] += (double)pi * (double)qi;
                        if constexpr (TR) {
                            a[1] += (double)pi * (double)pi;
                            a[2] += (double)w[i] * (double)pi;
                        }
                    });
    block_partial<0u, NQ>(a, slot_ptr(partials, SLOT_Q), block_id(P));
}

// The same pass on the diagonal layout when a wavefront has one slice at most
// (up to kMaxBlocks x kWaves slices, 524,288 rows).  Such a pass is bound by
// its chain of round trips, not by bytes: the partials, then every load of
// the slice are issued first (the layout's addresses depend on no index), and
// the combination of the partials runs while they are in flight.  A slice
// without free rows is loaded all the same.
// Two blocks share a CU above kMaxBlocks / 2 blocks, so PH, the entries loaded
// before the combination, is the whole row below that and eight above it
// (64 VGPRs; all values of the row but the vector in phases of 8, 5 or 4 took
// a solve of 493 k rows from 12.2 to 12.6, 12.8 and 12.9 ms).
template <int WMAX, class VT, class VV, bool TR, int PH>
__global__ __launch_bounds__(kBlock, PH < diag_width<WMAX>() ? 8 : 1) void k_cg_spmv_one(Part P0, ColsDiag sc,
                                                        const VT *__restrict__ v,
                                                        const uint8_t *__restrict__ mask,
                                                        const VV *__restrict__ z,
                                                        VV *__restrict__ p, VV *__restrict__ q,
                                                        const VV *__restrict__ w, double *partials,
                                                        CgLink L, int j, int max_it,
                                                        double rtol2)
{
    Part P = P0;
    P.heavy = 0;   // make_part's choice for a pass of one slice per wavefront
    constexpr int W = diag_width<WMAX>();
    const DevScalars *const S = L.S;
    const int stop = S->done;
    const CgIn in = cg_in(S, j);
    const double *slot = slot_ptr(partials, (j & 1) ? SLOT_U1 : SLOT_U0);
    double u[2], beta;
    load_partials<0u, 2>(slot, P.nb, u);
    const int lane = threadIdx.x & 63;
    const int blk = block_id(P);
    const int s0 = blk * kWaves + wave_id();
    const int s = min(s0, P.nslices() - 1);   // a wavefront past the last slice loads it and drops it
    const int row0 = s * kSlice, row = row0 + lane;
    const bool in_n = row < P.n;
    const int r = in_n ? row : P.n - 1;
    const DiagTab<W> t = diag_tab<W>(sc, s);
    const uint8_t m = mask[r];
    const VV po = p[r], qo = q[r], zo = z[r];
    const bool edge = t.kind == DR_EDGE;
    VT vv[PH];
    VV xv[PH];
    auto load = [&](int h) {
#pragma unroll
        for (int k = 0; k < PH; k++) {
            if (h + k >= W) continue;
            int d, b;
            diag_entry<W>(t, h + k, d, b);
            vv[k] = (v + (ptrdiff_t)(b + row0))[lane];
            if (edge) xv[k] = z[min(max(row + d, 0), P.n - 1)];
            else xv[k] = (z + (row0 + d))[lane];
        }
    };
    if (t.kind != DR_GENERAL) load(0);
    if (stop) return;
    if (cg_begin<TR>(in, slot, P.nb, u, L, j, max_it, rtol2, beta)) return;
    const bool act = in_n && m != 0 && s0 < P.nslices();
    double acc[1] = {0.0};
    if (t.kind != DR_GENERAL) {
#pragma unroll
        for (int h = 0; h < W; h += PH) {
            if (h > 0) load(h);
#pragma unroll
            for (int k = 0; k < PH; k++)
                if (h + k < W) acc[0] = __builtin_fma((double)vv[k], (double)xv[k], acc[0]);
        }
    } else {
        diag_row_gen<1, VV>(sc, v, P.n, s,
                            [&](int ub, int l, VV (&out)[1]) { out[0] = (z + ub)[l]; }, acc);
    }
    constexpr int NQ = TR ? 3 : 1;
    double a[NQ];
#pragma unroll
    for (int k = 0; k < NQ; k++) a[k] = 0.0;
    if (act) {
        const VV pi = (VV)fma(beta, (double)po, (double)zo);
        const VV qi = (VV)fma(beta, (double)qo, acc[0]);
        p[row] = pi;
        q[row] = qi;
        a[0] += (double)pi * (double)qi;
        if constexpr (TR) {
            a[1] += (double)pi * (double)pi;
            a[2] += (double)w[row] * (double)pi;
        }
    }
    block_partial<0u, NQ>(a, slot_ptr(partials, SLOT_Q), blk);
}

// CG iteration j, vector update on free rows.
// Prologue: p.q_j from SLOT_Q, alpha_j = r.z_j / p.q_j (r.z_j stored by the
// matrix pass).  Body: w += alpha p, r -= alpha q, z = dm r; partials of
// r.z_{j+1}, r.r_{j+1} into slot U[(j+1)%2].  With the Chebyshev
// preconditioner (cres set) z starts as dm r / theta, the Chebyshev residual
// and first increment are set, and the last Chebyshev pass replaces r.z.
// With a finite trust region (TR, radius^2 delta2) the step alpha that
// would take |w + alpha p| past the radius is cut to the tau >= 0 with
// |w + tau p| = radius (Steihaug's truncated CG, as TRON's inner solve),
// using |w|^2 kept on the device by the recurrence
// |w + t p|^2 = |w|^2 + 2 t w.p + t^2 p.p; the next matrix pass then ends
// the CG (done = 2).
// ONE: a wavefront has one slice at most, and issues its loads before the
// partials' combination (as k_cg_spmv_one).
template <class VV, bool TR, bool ONE>
__global__ __launch_bounds__(kBlock) void k_cg_update(Part P0, const uint8_t *__restrict__ mask,
                                                      const VV *__restrict__ p,
                                                      const VV *__restrict__ q,
                                                      const VV *__restrict__ dm,
                                                      VV *__restrict__ w, VV *__restrict__ r,
                                                      VV *__restrict__ z, double *partials,
                                                      CgLink L, int j, VV *__restrict__ cres,
                                                      VV *__restrict__ cdz0, double inv_theta,
                                                      double delta2)
{
    Part P = P0;
    if constexpr (ONE) P.heavy = 0;
    else if constexpr (std::is_same_v<VV, double>) P.heavy = -1;
    DevScalars *const S = L.S;
    const int stop = S->done;
    if constexpr (!ONE)
        if (stop) return;
    const double rz = S->rzh[j & 1];
    constexpr int NQ = TR ? 3 : 1;
    double pqa[NQ];
    load_partials<0u, NQ>(slot_ptr(partials, SLOT_Q), P.nb, pqa);
    struct Own {
        VV r, q, dm, w, p;
        uint8_t m;
    };
    auto own = [&](int i) { return Own{r[i], q[i], dm[i], w[i], p[i], mask[i]}; };
    Own o1{};
    const int blk = block_id(P);
    const int i1 = (blk * kWaves + wave_id()) * kSlice + (threadIdx.x & 63);
    if constexpr (ONE) {
        o1 = own(min(i1, P.n - 1));
        if (stop) return;
    }
    combine_loaded<0u, NQ>(pqa);
    const double pq = pqa[0];
    if (!(pq > 0.0 && isfinite(pq))) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            S->done = isfinite(pq) ? 3 : 4;
            S->it = j;
            flow_end(L);
        }
        return;
    }
    double alpha = rz / pq;
    if constexpr (TR) {
        const double pp = pqa[1], wp = pqa[2], ww = S->ww[j & 1];
        double wn = ww + alpha * (2.0 * wp + alpha * pp);
        int hit = 0;
        if (wn >= delta2) {
            // positive root of pp t^2 + 2 wp t + (ww - delta2) = 0 (ww <= delta2),
            // in the form without cancellation for either sign of wp
            const double room = fmax(delta2 - ww, 0.0);
            const double disc = sqrt(wp * wp + pp * room);
            alpha = wp >= 0.0 ? room / (wp + disc) : (disc - wp) / pp;
            wn = delta2;
            hit = 1;
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            S->ww[(j + 1) & 1] = wn;
            S->tr_hit = hit;
        }
    }
    double a[2] = {0.0, 0.0};
    auto step = [&](int i, const Own &o) {
        const VV ri = (VV)((double)o.r - alpha * (double)o.q);
        const VV zi = cres ? (VV)((double)o.dm * (double)ri * inv_theta) : o.dm * ri;
        w[i] = (VV)((double)o.w + alpha * (double)o.p);
        r[i] = ri;
        z[i] = zi;
        if (cres) {
            cres[i] = ri;
            cdz0[i] = zi;
        }
        a[0] += (double)ri * (double)zi;
        a[1] += (double)ri * (double)ri;
    };
    if constexpr (ONE) {
        if (i1 < P.n && o1.m) step(i1, o1);
    } else {
        for_rows(P, [&](int i, bool act) {
            if (act && mask[i]) step(i, own(i));
        });
    }
    block_partial<0u, 2>(a, slot_ptr(partials, ((j + 1) & 1) ? SLOT_U1 : SLOT_U0), blk);
    if (blockIdx.x == 0 && threadIdx.x == 0) S->it = j + 1;
}

// One step of the Chebyshev iteration for A_FF z = r from z = 0 with the
// Jacobi splitting (the polynomial preconditioner of the inner CG), on the
// free rows: res -= A dzp (dzp gathered; zero off the face), dzn = ca dzp +
// cb dm res, z += dzn.  The last step leaves r.z in value 0 of `slot` (the
// slot whose r.r the update or set-up kernel wrote).
template <int WMAX, class VT, class VV, class Cols>
__global__ __launch_bounds__(kBlock, walk_waves<Cols>()) void k_cheb(Part P, const int *__restrict__ so, Cols sc,
                                                 const VT *__restrict__ v,
                                                 const uint8_t *__restrict__ mask,
                                                 const VV *__restrict__ dm,
                                                 const VV *__restrict__ r, VV *__restrict__ res,
                                                 const VV *__restrict__ dzp, VV *__restrict__ dzn,
                                                 VV *__restrict__ z, double ca, double cb,
                                                 int last, int slot, double *partials,
                                                 DevScalars *S)
{
    if (S->done) return;
    double a[1] = {0.0};
    walk_rows<WMAX>(P, so, sc, v, [&](int i) { return mask[i] != 0; },
                    [&](int i) { return Three{(double)res[i], (double)dzp[i], (double)z[i]}; },
                    [&](int ub, int l) { return (dzp + ub)[l]; }, [&](int i, double kd, Three x) {
                        const double rn = x.a - kd;
                        const double dn = ca * x.b + cb * (double)dm[i] * rn;
                        const VV zn = (VV)(x.c + dn);
                        res[i] = (VV)rn;
                        dzn[i] = (VV)dn;
                        z[i] = zn;
                        a[0] += (double)r[i] * (double)zn;
                    });
    if (last) block_partial<OP_SUM, 1>(a, slot_ptr(partials, slot), block_id(P));
}

// Gershgorin bound of the spectrum of D^-1 A: max over rows of sum_j |a_ij| / a_ii
// (an upper bound for every principal submatrix too).
__global__ __launch_bounds__(kBlock) void k_gersh(Part P, const int *__restrict__ so,
                                                  const double *__restrict__ v,
                                                  const double *__restrict__ diag, double *partials)
{
    double a[1] = {0.0};
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        const int s = i / kSlice, lane = i % kSlice;
        const int off = so[s], w = (so[s + 1] - off) / kSlice;
        double sum = 0.0;
        for (int k = 0; k < w; k++) sum += fabs(v[off + k * kSlice + lane]);
        a[0] = fmax(a[0], sum / diag[i]);
    });
    block_partial<OP_MAX, 1>(a, slot_ptr(partials, SLOT_HOST), block_id(P));
}

// The breakpoint pass on its own (no trial beside it); partials into SLOT_Q.
template <class VV>
__global__ __launch_bounds__(kBlock) void k_breakpoint(Part P, const double *__restrict__ c,
                                                       const VV *__restrict__ w,
                                                       const double *__restrict__ g,
                                                       double *partials, Box B)
{
    double a[3];
    red_init<kOpsBrk, 3>(a);
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        breakpoint(c[i], (double)w[i], g[i], B, a);
    });
    block_partial<kOpsBrk, 3>(a, slot_ptr(partials, SLOT_Q), block_id(P));
}

__global__ __launch_bounds__(kBlock) void k_active(Part P, const double *__restrict__ c,
                                                   uint8_t *__restrict__ active, Box B)
{
    for_rows(P, [&](int i, bool act) {
        if (act) active[i] = c[i] == B.lo ? 1 : (c[i] == B.hi ? 2 : 0);
    });
}

__global__ __launch_bounds__(kBlock) void k_vals_mdt_plus_k(int64_t nnz, const double *__restrict__ m,
                                                            double dt, const double *__restrict__ k,
                                                            double *__restrict__ out)
{
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < nnz;
         t += (int64_t)gridDim.x * kBlock)
        out[t] = m[t] / dt + k[t];
}

// Paired copy of a sliced-ELL array (the layout of nn_matrix::d16p): within
// slice s of width w, entry k of lane l moves from off + 64 k + l to
// off + 128 (k / 2) + 2 l + k % 2 for k < 2 (w / 2); an odd last column stays.
template <class T>
__global__ __launch_bounds__(kBlock) void k_pair(Part P, const int *__restrict__ so,
                                                 const T *__restrict__ src, T *__restrict__ dst)
{
    const int lane = threadIdx.x & 63, wid = wave_id();
    for (int s = block_id(P) * kWaves + wid; s < P.nslices(); s += P.nb * kWaves) {
        const int off = so[s], w = (so[s + 1] - off) / kSlice, wp = 2 * (w / 2);
        for (int k = 0; k < w; k++) {
            const int from = off + k * kSlice + lane;
            const int to = k < wp ? off + (k / 2) * 2 * kSlice + 2 * lane + (k & 1) : from;
            dst[to] = src[from];
        }
    }
}

// Quad copy of a sliced-ELL array (the layout of nn_matrix::d16q): within
// slice s of width w, entry k of lane l moves to off + 256 (k / 4) + 4 l + k % 4
// for k < 4 (w / 4); the next two, if there are two left, to
// off + 256 (w / 4) + 2 l + (k - 4 (w / 4)); an odd last one stays.
template <class T>
__global__ __launch_bounds__(kBlock) void k_quad(Part P, const int *__restrict__ so,
                                                 const T *__restrict__ src, T *__restrict__ dst)
{
    const int lane = threadIdx.x & 63, wid = wave_id();
    for (int s = block_id(P) * kWaves + wid; s < P.nslices(); s += P.nb * kWaves) {
        const int off = so[s], w = (so[s + 1] - off) / kSlice;
        const int nq = w / 4, np = (w - 4 * nq) / 2;
        for (int k = 0; k < w; k++) {
            const int from = off + k * kSlice + lane;
            int to = from;
            if (k < 4 * nq) to = off + (k / 4) * 4 * kSlice + 4 * lane + (k & 3);
            else if (k < 4 * nq + 2 * np) to = off + nq * 4 * kSlice + 2 * lane + (k - 4 * nq);
            dst[to] = src[from];
        }
    }
}

// float32 copy of a value array (round to nearest)
__global__ __launch_bounds__(kBlock) void k_to_f32(int64_t m, const double *__restrict__ a,
                                                   float *__restrict__ b)
{
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < m;
         t += (int64_t)gridDim.x * kBlock)
        b[t] = (float)a[t];
}

// diag[i] = entry of row i in column i (sliced-ELL)
__global__ __launch_bounds__(kBlock) void k_diag(Part P, const int *__restrict__ so,
                                                 const int *__restrict__ sc,
                                                 const double *__restrict__ v,
                                                 double *__restrict__ diag)
{
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        const int s = i / kSlice, lane = i % kSlice;
        const int off = so[s], w = (so[s + 1] - off) / kSlice;
        double d = 0.0;
        bool found = false;
        for (int k = 0; k < w; k++) {
            const int e = off + k * kSlice + lane;
            if (!found && sc[e] == i) {   // the real entry precedes any padding
                d = v[e];
                found = true;
            }
        }
        diag[i] = d;
    });
}

// CSR (rowptr-ordered values) -> sliced-ELL: entry k of row i goes to
// so[i/64] + k*64 + i%64; padding entries get column i and value 0.
__global__ __launch_bounds__(kBlock) void k_csr_to_sell(Part P, const int *__restrict__ rp,
                                                        const int *__restrict__ ci,
                                                        const double *__restrict__ val,
                                                        const double *__restrict__ mval,
                                                        const int *__restrict__ so,
                                                        int *__restrict__ sc, double *__restrict__ sv,
                                                        double *__restrict__ smv)
{
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        const int s = i / kSlice, lane = i % kSlice;
        const int off = so[s], w = (so[s + 1] - off) / kSlice;
        const int k0 = rp[i], len = rp[i + 1] - rp[i];
        for (int k = 0; k < w; k++) {
            const int e = off + k * kSlice + lane;
            const bool real = k < len;
            sc[e] = real ? ci[k0 + k] : i;
            sv[e] = real ? val[k0 + k] : 0.0;
            if (smv) smv[e] = real ? mval[k0 + k] : 0.0;
        }
    });
}

// The rows of the last slice past n keep their padding: fill them so every
// entry of the sliced-ELL arrays is defined (column 0, value 0).
__global__ __launch_bounds__(kBlock) void k_sell_tail(int n, int nslices, const int *__restrict__ so,
                                                      int *__restrict__ sc, double *__restrict__ sv,
                                                      double *__restrict__ smv)
{
    const int s = nslices - 1;
    if (s < 0) return;
    const int off = so[s], w = (so[s + 1] - off) / kSlice;
    for (int t = threadIdx.x; t < w * kSlice; t += kBlock) {
        const int lane = t % kSlice;
        if (s * kSlice + lane < n) continue;
        sc[off + t] = 0;
        sv[off + t] = 0.0;
        if (smv) smv[off + t] = 0.0;
    }
}

// int16 offsets col - row of the sliced-ELL entries and the largest |col - row|
// over real rows (one partial per block, SLOT_HOST).  Lanes past the last row
// get offsets that point at the last row, so every decoded column is valid.
__global__ __launch_bounds__(kBlock) void k_sell_d16(Part P, const int *__restrict__ so,
                                                     const int *__restrict__ sc,
                                                     short *__restrict__ sd, double *partials)
{
    double a[1];
    red_init<OP_MAX, 1>(a);
    for_rows(P, [&](int i, bool act) {
        const int s = i / kSlice, lane = i % kSlice;
        const int off = so[s], w = (so[s + 1] - off) / kSlice;
        for (int k = 0; k < w; k++) {
            const int e = off + k * kSlice + lane;
            const int d = act ? sc[e] - i : (P.n - 1) - i;
            if (act) a[0] = fmax(a[0], (double)abs(d));
            sd[e] = (short)max(-32768, min(32767, d));
        }
    });
    block_partial<OP_MAX, 1>(a, slot_ptr(partials, SLOT_HOST), block_id(P));
}

// ---------------------------------------------------------------- launchers
// (NN_DISPATCH_W, in rows.hpp, instantiates a kernel for the matrix's slice
// width class.)

void launch_matvec(nn_ctx *ctx, const nn_matrix *A, const double *vals, const double *x, double *y)
{
    if (A->n == 0) return;
    Part P = make_part(A->n);
    NN_DISPATCH_W(A->wmax, (k_matvec<WM, ColsI32>), P.nb, P, A->sl_off, ColsI32{A->sl_col}, vals, x, y);
}

void launch_transient_rhs(nn_ctx *ctx, const nn_matrix *A, const double *c, const double *f,
                          double dt, double *ft)
{
    if (A->n == 0) return;
    Part P = make_part(A->n);
    NN_DISPATCH_W(A->wmax, (k_transient_rhs<WM, ColsI32>), P.nb, P, A->sl_off, ColsI32{A->sl_col}, A->mval,
                  c, f, dt, ft);
}

void launch_init(nn_ctx *ctx, int64_t n, double *c, const double *f, int mode, double c0v, Box B)
{
    Part P = make_part(n);
    k_init<<<P.nb, kBlock, 0, ctx->stream>>>(P, c, f, mode, c0v, ctx->partials, B);
}

void launch_grad(nn_ctx *ctx, const nn_matrix *A, const double *vals, const double *vals_p,
                 const double *c, const double *f, double *g, Box B)
{
    Part P = make_part(A->n);
    if (vals_p && A->diag_plan)
        NN_DISPATCH_W(A->wmax, (k_grad<WM, ColsDiag>), P.nb, P, A->sl_off, diag_cols(A, A->d16p),
                      vals_p, c, f, g, ctx->partials, B);
    else if (vals_p && A->d16p)
        NN_DISPATCH_W(A->wmax, (k_grad<WM, ColsD16P>), P.nb, P, A->sl_off, ColsD16P{A->d16p}, vals_p,
                      c, f, g, ctx->partials, B);
    else
        NN_DISPATCH_W(A->wmax, (k_grad<WM, ColsI32>), P.nb, P, A->sl_off, ColsI32{A->sl_col}, vals,
                      c, f, g, ctx->partials, B);
}

void launch_trial(nn_ctx *ctx, const nn_matrix *A, const Vals &V, const double *c, Dir d,
                  double t, const double *g, const uint8_t *mask, double *ks, Box B, bool brk)
{
    Part P = make_part(A->n, kMaxBlocks, V.v32 || V.v32q);
    auto go = [&](auto cols, const auto *v, const auto *dv) {
        using Cols = decltype(cols);
        using VT = std::remove_cv_t<std::remove_pointer_t<decltype(v)>>;
        using VD = std::remove_cv_t<std::remove_pointer_t<decltype(dv)>>;
        if constexpr (std::is_same_v<VT, VD>) {   // the CG step's type
            if (brk) {
                NN_DISPATCH_W(A->wmax, (k_trial<WM, VT, VD, Cols, true>), P.nb, P, A->sl_off, cols,
                              v, c, dv, t, g, mask, ks, ctx->partials, B);
                return;
            }
        }
        NN_DISPATCH_W(A->wmax, (k_trial<WM, VT, VD, Cols, false>), P.nb, P, A->sl_off, cols, v, c,
                      dv, t, g, mask, ks, ctx->partials, B);
    };
    // float32 values: the Cauchy direction is float64, the CG step float32
    auto go32 = [&](auto cols, const float *v) {
        if (d.f32) go(cols, v, d.f32);
        else go(cols, v, d.f64);
    };
    if (A->diag_plan && V.v32q) go32(diag_cols(A, A->d16q), V.v32q);
    else if (A->diag_plan && V.v64p) go(diag_cols(A, A->d16p), V.v64p, d.f64);
    else if (V.v32q && A->d16q) go32(ColsD16Q{A->d16q}, V.v32q);
    else if (V.v32 && A->sl_d16) go32(ColsD16{A->sl_d16}, V.v32);
    else if (V.v32) go32(ColsI32{A->sl_col}, V.v32);
    else if (V.v64p && A->d16p) go(ColsD16P{A->d16p}, V.v64p, d.f64);
    else go(ColsI32{A->sl_col}, V.v64, d.f64);
}

void launch_ladder(nn_ctx *ctx, const nn_matrix *A, const Vals &V, const double *c,
                   const double *g, const double *t, double *const *ks, Box B)
{
    // 3 kLadder accumulators per lane: one 1024-thread block per CU
    Part P = make_part(A->n, kLadderBlocks, V.v32 || V.v32q);
    Ladder L;
    for (int k = 0; k < kLadder; k++) {
        L.t[k] = t[k];
        L.ks[k] = ks[k];
    }
    if (A->diag_plan && V.v32q)
        NN_DISPATCH_W(A->wmax, (k_ladder<WM, float, ColsDiag>), P.nb, P, A->sl_off,
                      diag_cols(A, A->d16q), V.v32q, c, g, L, B, ctx->partials);
    else if (A->diag_plan && V.v64p)
        NN_DISPATCH_W(A->wmax, (k_ladder<WM, double, ColsDiag>), P.nb, P, A->sl_off,
                      diag_cols(A, A->d16p), V.v64p, c, g, L, B, ctx->partials);
    else if (V.v32q && A->d16q)
        NN_DISPATCH_W(A->wmax, (k_ladder<WM, float, ColsD16Q>), P.nb, P, A->sl_off,
                      ColsD16Q{A->d16q}, V.v32q, c, g, L, B, ctx->partials);
    else if (V.v32 && A->sl_d16)
        NN_DISPATCH_W(A->wmax, (k_ladder<WM, float, ColsD16>), P.nb, P, A->sl_off,
                      ColsD16{A->sl_d16}, V.v32, c, g, L, B, ctx->partials);
    else if (V.v32)
        NN_DISPATCH_W(A->wmax, (k_ladder<WM, float, ColsI32>), P.nb, P, A->sl_off,
                      ColsI32{A->sl_col}, V.v32, c, g, L, B, ctx->partials);
    else if (V.v64p && A->d16p)
        NN_DISPATCH_W(A->wmax, (k_ladder<WM, double, ColsD16P>), P.nb, P, A->sl_off,
                      ColsD16P{A->d16p}, V.v64p, c, g, L, B, ctx->partials);
    else
        NN_DISPATCH_W(A->wmax, (k_ladder<WM, double, ColsI32>), P.nb, P, A->sl_off,
                      ColsI32{A->sl_col}, V.v64, c, g, L, B, ctx->partials);
}

void launch_apply(nn_ctx *ctx, int64_t n, double *c, Dir d, double t, Box B)
{
    Part P = make_part(n, kMaxBlocks, d.f32);
    if (d.f32) k_apply<float><<<P.nb, kBlock, 0, ctx->stream>>>(P, c, d.f32, t, B);
    else k_apply<double><<<P.nb, kBlock, 0, ctx->stream>>>(P, c, d.f64, t, B);
}

void launch_resid(nn_ctx *ctx, const nn_matrix *A, const double *vals, const double *c,
                  const double *f)
{
    Part P = make_part(A->n);
    NN_DISPATCH_W(A->wmax, (k_resid<WM, ColsI32>), P.nb, P, A->sl_off, ColsI32{A->sl_col}, vals, c,
                  f, ctx->partials);
}

void launch_add(nn_ctx *ctx, int64_t n, double *c, const double *w)
{
    Part P = make_part(n);
    k_add<double><<<P.nb, kBlock, 0, ctx->stream>>>(P, c, w);
}

void launch_cg_setup(nn_ctx *ctx, const nn_matrix *A, const double *diag, double *c, double *g,
                     const double *ks, double t, bool f32, Box B, int face, const Cheb *ch)
{
    Part P = make_part(A->n, kMaxBlocks, f32);
    Workspace &W = ctx->ws;
    const double it = ch ? 1.0 / ch->theta : 0.0;
    if (f32)
        k_cg_setup<float><<<P.nb, kBlock, 0, ctx->stream>>>(
            P, A->rowptr, diag, c, g, ks, t, W.mask, W.dm32, W.r32, W.z32, W.p32, W.q32, W.w32,
            ctx->partials, ctx->scal, B, face, ch ? W.cres32 : nullptr,
            ch ? W.cdz32[0] : nullptr, ch ? W.cdz32[1] : nullptr, it);
    else
        k_cg_setup<double><<<P.nb, kBlock, 0, ctx->stream>>>(
            P, A->rowptr, diag, c, g, ks, t, W.mask, W.dm, W.r, W.z, W.p0, W.q, W.w, ctx->partials,
            ctx->scal, B, face, ch ? W.cres : nullptr, ch ? W.cdz[0] : nullptr,
            ch ? W.cdz[1] : nullptr, it);
}

void launch_cheb(nn_ctx *ctx, const nn_matrix *A, const Vals &V, const Cheb &ch, int step,
                 int slot)
{
    Part P = make_part(A->n, kMaxBlocks, V.v32 || V.v32q);
    Workspace &W = ctx->ws;
    const double ca = ch.ca[step], cb = ch.cb[step];
    const int last = step == ch.degree - 1 ? 1 : 0;
    const int ip = (step - 1) & 1, in = step & 1;
    if (A->diag_plan && V.v32q) {
        NN_DISPATCH_W(A->wmax, (k_cheb<WM, float, float, ColsDiag>), P.nb, P, A->sl_off,
                      diag_cols(A, A->d16q), V.v32q, W.mask, W.dm32, W.r32, W.cres32, W.cdz32[ip],
                      W.cdz32[in], W.z32, ca, cb, last, slot, ctx->partials, ctx->scal);
    } else if (A->diag_plan && V.v64p) {
        NN_DISPATCH_W(A->wmax, (k_cheb<WM, double, double, ColsDiag>), P.nb, P, A->sl_off,
                      diag_cols(A, A->d16p), V.v64p, W.mask, W.dm, W.r, W.cres, W.cdz[ip],
                      W.cdz[in], W.z, ca, cb, last, slot, ctx->partials, ctx->scal);
    } else if (V.v32 && A->sl_d16) {
        NN_DISPATCH_W(A->wmax, (k_cheb<WM, float, float, ColsD16>), P.nb, P, A->sl_off,
                      ColsD16{A->sl_d16}, V.v32, W.mask, W.dm32, W.r32, W.cres32, W.cdz32[ip],
                      W.cdz32[in], W.z32, ca, cb, last, slot, ctx->partials, ctx->scal);
    } else if (V.v32) {
        NN_DISPATCH_W(A->wmax, (k_cheb<WM, float, float, ColsI32>), P.nb, P, A->sl_off,
                      ColsI32{A->sl_col}, V.v32, W.mask, W.dm32, W.r32, W.cres32, W.cdz32[ip],
                      W.cdz32[in], W.z32, ca, cb, last, slot, ctx->partials, ctx->scal);
    } else {
        NN_DISPATCH_W(A->wmax, (k_cheb<WM, double, double, ColsI32>), P.nb, P, A->sl_off,
                      ColsI32{A->sl_col}, V.v64, W.mask, W.dm, W.r, W.cres, W.cdz[ip], W.cdz[in],
                      W.z, ca, cb, last, slot, ctx->partials, ctx->scal);
    }
}

void launch_gersh(nn_ctx *ctx, const nn_matrix *A, const double *vals, const double *diag)
{
    Part P = make_part(A->n);
    k_gersh<<<P.nb, kBlock, 0, ctx->stream>>>(P, A->sl_off, vals, diag, ctx->partials);
}

template <bool TR>
static void cg_spmv_tr(nn_ctx *ctx, const nn_matrix *A, const Vals &V, int j, int max_it,
                       double rtol)
{
    Part P = make_part(A->n, kMaxBlocks, V.v32 || V.v32q);
    Workspace &W = ctx->ws;
    const CgLink L{ctx->scal, ctx->flow, ctx->flow_cg};
    if (A->diag_plan && (V.v32q || V.v64p)) {
        // one slice per wavefront at most: every load before the prologue
        const bool one = P.nslices() <= P.nb * kWaves, lone = P.nb <= kMaxBlocks / 2;
        const ColsDiag cols = diag_cols(A, V.v32q ? A->d16q : A->d16p);
        if (V.v32q && one)
            NN_DISPATCH_W(A->wmax, (k_cg_spmv_one<WM, float, float, TR, diag_width<WM>()>), P.nb, P,
                          cols, V.v32q, W.mask, W.z32, W.p32, W.q32, W.w32, ctx->partials, L,
                          j, max_it, rtol * rtol);
        else if (V.v32q)
            NN_DISPATCH_W(A->wmax, (k_cg_spmv<WM, float, float, ColsDiag, TR>), P.nb, P, A->sl_off,
                          cols, V.v32q, W.mask, W.z32, W.p32, W.q32, W.w32, ctx->partials,
                          L, j, max_it, rtol * rtol);
        else if (one && lone)
            NN_DISPATCH_W(A->wmax, (k_cg_spmv_one<WM, double, double, TR, diag_width<WM>()>), P.nb, P,
                          cols, V.v64p, W.mask, W.z, W.p0, W.q, W.w, ctx->partials, L, j,
                          max_it, rtol * rtol);
        else if (one)
            NN_DISPATCH_W(A->wmax, (k_cg_spmv_one<WM, double, double, TR, 8>), P.nb, P, cols, V.v64p,
                          W.mask, W.z, W.p0, W.q, W.w, ctx->partials, L, j, max_it,
                          rtol * rtol);
        else
            NN_DISPATCH_W(A->wmax, (k_cg_spmv<WM, double, double, ColsDiag, TR>), P.nb, P,
                          A->sl_off, cols, V.v64p, W.mask, W.z, W.p0, W.q, W.w, ctx->partials,
                          L, j, max_it, rtol * rtol);
    } else if (V.v32q && A->d16q) {
        NN_DISPATCH_W(A->wmax, (k_cg_spmv<WM, float, float, ColsD16Q, TR>), P.nb, P, A->sl_off,
                      ColsD16Q{A->d16q}, V.v32q, W.mask, W.z32, W.p32, W.q32, W.w32,
                      ctx->partials, L, j, max_it, rtol * rtol);
    } else if (V.v32 && A->sl_d16) {
        NN_DISPATCH_W(A->wmax, (k_cg_spmv<WM, float, float, ColsD16, TR>), P.nb, P, A->sl_off,
                      ColsD16{A->sl_d16}, V.v32, W.mask, W.z32, W.p32, W.q32, W.w32,
                      ctx->partials, L, j, max_it, rtol * rtol);
    } else if (V.v32) {
        NN_DISPATCH_W(A->wmax, (k_cg_spmv<WM, float, float, ColsI32, TR>), P.nb, P, A->sl_off,
                      ColsI32{A->sl_col}, V.v32, W.mask, W.z32, W.p32, W.q32, W.w32,
                      ctx->partials, L, j, max_it, rtol * rtol);
    } else if (V.v64p && A->d16p) {
        NN_DISPATCH_W(A->wmax, (k_cg_spmv<WM, double, double, ColsD16P, TR>), P.nb, P, A->sl_off,
                      ColsD16P{A->d16p}, V.v64p, W.mask, W.z, W.p0, W.q, W.w, ctx->partials,
                      L, j, max_it, rtol * rtol);
    } else {
        NN_DISPATCH_W(A->wmax, (k_cg_spmv<WM, double, double, ColsI32, TR>), P.nb, P, A->sl_off,
                      ColsI32{A->sl_col}, V.v64, W.mask, W.z, W.p0, W.q, W.w, ctx->partials,
                      L, j, max_it, rtol * rtol);
    }
}

void launch_cg_spmv(nn_ctx *ctx, const nn_matrix *A, const Vals &V, int j, int max_it, double rtol,
                    bool tr)
{
    if (tr) cg_spmv_tr<true>(ctx, A, V, j, max_it, rtol);
    else cg_spmv_tr<false>(ctx, A, V, j, max_it, rtol);
}

template <bool TR>
static void cg_update_tr(nn_ctx *ctx, int64_t n, int j, bool f32, const Cheb *ch, double delta2)
{
    Part P = make_part(n, kMaxBlocks, f32);
    Workspace &W = ctx->ws;
    const CgLink L{ctx->scal, ctx->flow, ctx->flow_cg};
    const double it = ch ? 1.0 / ch->theta : 0.0;
    const bool one = P.nslices() <= P.nb * kWaves;
#define NN_UPD(VV, ONE, p_, q_, dm_, w_, r_, z_, cres_, cdz_)                                    \
    NN_LAUNCH_ROWS((k_cg_update<VV, TR, ONE>), P.nb, P, W.mask, p_, q_, dm_, w_, r_, z_,         \
                   ctx->partials, L, j, ch ? cres_ : nullptr, ch ? cdz_[0] : nullptr, it,        \
                   delta2)
    if (f32 && one) NN_UPD(float, true, W.p32, W.q32, W.dm32, W.w32, W.r32, W.z32, W.cres32, W.cdz32);
    else if (f32) NN_UPD(float, false, W.p32, W.q32, W.dm32, W.w32, W.r32, W.z32, W.cres32, W.cdz32);
    else if (one) NN_UPD(double, true, W.p0, W.q, W.dm, W.w, W.r, W.z, W.cres, W.cdz);
    else NN_UPD(double, false, W.p0, W.q, W.dm, W.w, W.r, W.z, W.cres, W.cdz);
#undef NN_UPD
}

void launch_cg_update(nn_ctx *ctx, int64_t n, int j, bool f32, const Cheb *ch, double delta2)
{
    if (std::isfinite(delta2)) cg_update_tr<true>(ctx, n, j, f32, ch, delta2);
    else cg_update_tr<false>(ctx, n, j, f32, ch, delta2);
}

void launch_breakpoint(nn_ctx *ctx, int64_t n, const double *c, Dir w, const double *g, Box B)
{
    Part P = make_part(n, kMaxBlocks, w.f32);
    if (w.f32)
        k_breakpoint<float><<<P.nb, kBlock, 0, ctx->stream>>>(P, c, w.f32, g, ctx->partials, B);
    else
        k_breakpoint<double><<<P.nb, kBlock, 0, ctx->stream>>>(P, c, w.f64, g, ctx->partials, B);
}

void launch_quad_f32(nn_ctx *ctx, const nn_matrix *A, const float *src, float *dst)
{
    Part P = make_part(A->n);
    k_quad<float><<<P.nb, kBlock, 0, ctx->stream>>>(P, A->sl_off, src, dst);
}

void launch_quad_d16(nn_ctx *ctx, const nn_matrix *A, const short *src, short *dst)
{
    Part P = make_part(A->n);
    k_quad<short><<<P.nb, kBlock, 0, ctx->stream>>>(P, A->sl_off, src, dst);
}

void launch_pair_f64(nn_ctx *ctx, const nn_matrix *A, const double *src, double *dst)
{
    Part P = make_part(A->n);
    k_pair<double><<<P.nb, kBlock, 0, ctx->stream>>>(P, A->sl_off, src, dst);
}

void launch_pair_d16(nn_ctx *ctx, const nn_matrix *A, const short *src, short *dst)
{
    Part P = make_part(A->n);
    k_pair<short><<<P.nb, kBlock, 0, ctx->stream>>>(P, A->sl_off, src, dst);
}

void launch_to_f32(nn_ctx *ctx, int64_t m, const double *a, float *b)
{
    int64_t nb = (m + kBlock - 1) / kBlock;
    if (nb > 2048) nb = 2048;
    if (nb < 1) nb = 1;
    k_to_f32<<<(int)nb, kBlock, 0, ctx->stream>>>(m, a, b);
}

void launch_active(nn_ctx *ctx, int64_t n, const double *c, uint8_t *active, Box B)
{
    Part P = make_part(n);
    k_active<<<P.nb, kBlock, 0, ctx->stream>>>(P, c, active, B);
}

void launch_axpby_vals(nn_ctx *ctx, int64_t nnz, const double *m, double dt, const double *k,
                       double *out)
{
    int64_t nb = (nnz + kBlock - 1) / kBlock;
    if (nb > 2048) nb = 2048;
    if (nb < 1) nb = 1;
    k_vals_mdt_plus_k<<<(int)nb, kBlock, 0, ctx->stream>>>(nnz, m, dt, k, out);
}

void launch_sell_d16(nn_ctx *ctx, const nn_matrix *A, short *sd)
{
    Part P = make_part(A->n);
    k_sell_d16<<<P.nb, kBlock, 0, ctx->stream>>>(P, A->sl_off, A->sl_col, sd, ctx->partials);
}

void launch_diag(nn_ctx *ctx, const nn_matrix *A, const double *vals, double *diag)
{
    Part P = make_part(A->n);
    k_diag<<<P.nb, kBlock, 0, ctx->stream>>>(P, A->sl_off, A->sl_col, vals, diag);
}

void launch_csr_to_sell(nn_ctx *ctx, nn_matrix *A, const double *csr_val, const double *csr_mval)
{
    Part P = make_part(A->n);
    k_csr_to_sell<<<P.nb, kBlock, 0, ctx->stream>>>(P, A->rowptr, A->col, csr_val, csr_mval,
                                                    A->sl_off, A->sl_col, A->val, A->mval);
    k_sell_tail<<<1, kBlock, 0, ctx->stream>>>((int)A->n, P.nslices(), A->sl_off, A->sl_col, A->val,
                                               A->mval);
}

}  // namespace nnqp
