// One-workgroup TRON solve for small problems.
//
// A solve of a few thousand rows is bound by launches and host round trips,
// not by bytes: each CG iteration of the multi-block path is two launches of
// a few microseconds, and every Cauchy or search decision waits for the host.
// Here one 512-thread workgroup runs the whole method of solver.hip (same
// steps, constants and tests) inside a single launch: every pass walks the
// problem's 64-row slices with the workgroup's eight wavefronts, every
// reduction is a fixed-order workgroup reduction, and every decision is
// taken by all threads from the same reduced values, so control flow stays
// uniform and the only synchronisation is the workgroup barrier.  The work
// vectors stay in the caches for the sizes this path serves.
//
// The Cauchy search takes its trials one by one in the sequential order of
// the multi-block solver's rule (start at the previous step length,
// extrapolate x10 while the sufficient-decrease test holds, else interpolate
// x0.1 until it holds); the multi-block solver evaluates the same trials three
// at a time, which changes nothing but the cost.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "nnqp_internal.hpp"
#include "diag.hpp"

namespace nnqp {

namespace {

constexpr double kMu0 = 0.01;       // sufficient-decrease constant
constexpr double kExtrap = 10.0;    // Cauchy extrapolation factor
constexpr double kInterp = 0.1;     // Cauchy interpolation factor
constexpr double kBack = 0.5;       // projected-search backtracking factor
constexpr int kMaxTrials = 60;

// report of one solve, written by thread 0 of the workgroup
struct SoloOut {
    double kkt_rel, kkt_nat_inf, min_c, norm_f, bytes;
    int outer_its, cg_its, spmvs, n_active, cauchy_trials, search_trials, status, pad;
};

struct SoloProb {
    int n, nsl;
    const int *so;          // [nsl + 1] slice offsets
    const int *sc;          // sliced-ELL columns
    const int *rp;          // CSR row pointers (row lengths for the byte model)
    const double *v;        // sliced-ELL values
    const double *diag;
    const double *f;
    double *c;              // in: start (c0_mode 1); out: solution
    uint8_t *active;        // out or null
    double *g, *w, *r, *z, *p, *q, *ks[2], *dm;
    uint8_t *mask;
    SoloOut *out;
};

struct SoloOpts {
    double tol, rtol2, c0v;
    int c0_mode, max_outer, max_cg;
};

// The workgroup: 512 threads, eight wavefronts (two per SIMD), so a
// wavefront may hold up to 256 registers and keep many slices in flight.
constexpr int kSoloBlock = 512;
constexpr int kSoloWaves = kSoloBlock / 64;
// Vectors in LDS: problems up to kSoloLdsRows rows keep c, g, z and w there
// (4 x 32 KiB); up to kSoloLdsRows5 rows also q (five vectors of 4,032 rows
// and the reduction buffer fill the 160 KiB of a CU; on the 64^2 square
// 6.31 -> 5.98 ms per solve).
constexpr int kSoloLdsRows = 4096;
constexpr int kSoloLdsRows5 = 4032;
// rows per LDS vector of the variant that keeps nv vectors there
__host__ __device__ constexpr int solo_lds_rows(int nv) { return nv == 5 ? kSoloLdsRows5 : kSoloLdsRows; }

// Reduced values of a pass, the same in every thread: wavefront shuffles,
// then the wavefronts' totals combined in wavefront order (a fixed order, so
// the result is reproducible).
// One barrier per reduction: the totals go to one of two halves of sh,
// alternating between calls (parity, the same in every thread since every
// thread makes the same calls), and every wavefront combines them itself, so a
// half is written again only two reductions later, after the next barrier.
// Up to DIRECT values read the totals as broadcast vector loads; more go lane by
// lane through scalar registers, as their totals would hold 16 registers each:
// the engine with the matrix in registers has none left for them (64^2 square
// 2.49 -> 1.93 ms), the other one has (5.98 -> 5.69).
constexpr int kDirectFew = 2, kDirectAll = kMaxRed;
template <uint32_t OPS, int DIRECT, int NV>
__device__ __forceinline__ void wg_reduce(double (&a)[NV], double *sh, int &parity)
{
    const int lane = threadIdx.x & 63, wid = wave_id();
    wave_red<OPS, NV>(a);
    double *buf = sh + parity * (kSoloWaves * (kMaxRed + 1));
    parity ^= 1;
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; k++) buf[k * kSoloWaves + wid] = a[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; k++) {
        if constexpr (NV <= DIRECT) {
            double v = buf[k * kSoloWaves];
#pragma unroll
            for (int w = 1; w < kSoloWaves; w++)
                v = red_comb(op_of<OPS>(k), v, buf[k * kSoloWaves + w]);
            a[k] = v;
        } else {
            a[k] = lanes_in_order<kSoloWaves>(op_of<OPS>(k),
                                              buf[k * kSoloWaves + (lane & (kSoloWaves - 1))]);
        }
    }
}

// Rows of the problem, slice by slice over the workgroup's wavefronts:
// body(i, act) for row i = 64 s + lane of every slice s of this wavefront.
template <class Body>
__device__ __forceinline__ void wg_rows(const SoloProb &P, Body body)
{
    const int lane = threadIdx.x & 63, wid = wave_id();
    for (int s = wid; s < P.nsl; s += kSoloWaves) {
        const int i = s * kSlice + lane;
        body(i, i < P.n);
    }
}

// Sliced-ELL product over the workgroup's slices: for each row i with
// mask[i] != 0 (every row without a mask), epi(i, sum over the row's entries
// of v * x(col), pre(i)).  The passes of a small problem are bound by memory
// round trips, not bytes (see wg_spmv).
template <int WMAX>
struct SliceEnt {
    int w;
    int cc[WMAX];
    double vv[WMAX];
};

// The entries of the slice whose first entry and width are off and w: raw
// words under wave-uniform guards (nothing here waits for them).
template <int WMAX>
__device__ __forceinline__ void load_slice(const SoloProb &P, int off, int w, SliceEnt<WMAX> &e)
{
    const int lane = threadIdx.x & 63;
    e.w = w;
#pragma unroll
    for (int k = 0; k < WMAX; k++) {
        if (k < w) {
            e.cc[k] = P.sc[off + k * kSlice + lane];
            e.vv[k] = P.v[off + k * kSlice + lane];
        } else {
            e.cc[k] = 0;
            e.vv[k] = 0.0;
        }
    }
}

// First entry and width of slice s (width 0 past the last slice), from two
// loads that need no guard.
__device__ __forceinline__ void slice_span(const SoloProb &P, int s, int &off, int &w)
{
    const int a = s < P.nsl ? s : P.nsl, b = s + 1 < P.nsl ? s + 1 : P.nsl;
    off = P.so[a];
    w = (P.so[b] - off) >> 6;
}

// Slices a wavefront loads ahead of the one it sums (slices up to 8 wide;
// wider ones one ahead, their entries take more registers).  On the 64^2
// square (3,969 rows, float64): one ahead 6.14 ms per solve, two 6.44 ms,
// three 6.66 ms.
#ifndef NNQP_SOLO_AHEAD
#define NNQP_SOLO_AHEAD 1
#endif

// mask: the free-row flags (null: every row).  A wavefront loads the slice
// offsets D + 1 slices ahead and the entries, own-row values and flags of the
// next D slices before it gathers and sums the current one; the own-row loads
// take a row every vector has (row 0 past the end) and keep the raw flag, so
// no load of a later slice is waited for before the current slice's sum.
template <int WMAX, class Pre, class X, class Epi>
__device__ __forceinline__ void wg_spmv(const SoloProb &P, const uint8_t *__restrict__ mask,
                                        Pre pre, X x, Epi epi)
{
    using PV = decltype(pre(0));
    constexpr int D = WMAX <= 8 ? NNQP_SOLO_AHEAD : 1;
    static_assert(D >= 1, "at least the next slice is loaded ahead");
    const int lane = threadIdx.x & 63, wid = wave_id();
    struct Own {
        bool in;
        uint8_t flag;
        PV pv;
    };
    auto own = [&](int s) {
        const int row = s * kSlice + lane;
        const bool in = s < P.nsl && row < P.n;
        const int r = in ? row : 0;
        return Own{in, mask ? mask[r] : (uint8_t)1, pre(r)};
    };
    SliceEnt<WMAX> ent[D + 1];
    Own ow[D + 1];
    int off, w;
#pragma unroll
    for (int t = 0; t < D; t++) {
        slice_span(P, wid + t * kSoloWaves, off, w);
        load_slice<WMAX>(P, off, w, ent[t]);
        ow[t] = own(wid + t * kSoloWaves);
    }
    slice_span(P, wid + D * kSoloWaves, off, w);   // the span of the next slice to load
    for (int s = wid; s < P.nsl; s += kSoloWaves) {
        int off2, w2;
        slice_span(P, s + (D + 1) * kSoloWaves, off2, w2);
        load_slice<WMAX>(P, off, w, ent[D]);
        ow[D] = own(s + D * kSoloWaves);
        const SliceEnt<WMAX> &cur = ent[0];
        const bool act_c = ow[0].in && ow[0].flag != 0;
        if (__ballot(act_c) != 0) {
            // every gather issued before the first product is added: a slot
            // past the slice's width has column 0 (a valid row) and its
            // product is not added (a select, the same fused multiply-adds in
            // the same order as a guarded sum)
            double xv[WMAX];
#pragma unroll
            for (int k = 0; k < WMAX; k++) xv[k] = x(cur.cc[k]);
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < WMAX; k++) {
                const double y = __builtin_fma(cur.vv[k], xv[k], acc);
                acc = k < cur.w ? y : acc;
            }
            if (cur.w > WMAX) {   // slices wider than the unrolled part
                int o, ww;
                slice_span(P, s, o, ww);
                for (int k = WMAX; k < ww; k++) {
                    const int e = o + k * kSlice + lane;
                    acc += P.v[e] * x(P.sc[e]);
                }
            }
            if (act_c) epi(s * kSlice + lane, acc, ow[0].pv);
        }
#pragma unroll
        for (int t = 0; t < D; t++) {
            ent[t] = ent[t + 1];
            ow[t] = ow[t + 1];
        }
        off = off2;
        w = w2;
    }
}

// Rows of the workgroup's slices in two phases, NR slices of a wavefront at a
// time: ld(i) loads a row's operands (i < n), then st(i, vals) computes and
// stores, so the loads of NR slices are in flight together.
template <int NR, class Ld, class St>
__device__ __forceinline__ void wg_rows2(const SoloProb &P, Ld ld, St st)
{
    using LV = decltype(ld(0));
    const int lane = threadIdx.x & 63, wid = wave_id();
    for (int s0 = wid; s0 < P.nsl; s0 += NR * kSoloWaves) {
        LV v[NR];
        bool in[NR];
#pragma unroll
        for (int t = 0; t < NR; t++) {
            const int i = (s0 + t * kSoloWaves) * kSlice + lane;
            in[t] = s0 + t * kSoloWaves < P.nsl && i < P.n;
            v[t] = in[t] ? ld(i) : LV();
        }
#pragma unroll
        for (int t = 0; t < NR; t++)
            if (in[t]) st((s0 + t * kSoloWaves) * kSlice + lane, v[t]);
    }
}

__device__ __forceinline__ bool ok_decrease(double gs, double sks)
{
    return gs < 0.0 && gs + 0.5 * sks <= kMu0 * gs;
}

// The whole solve of one problem by the calling workgroup.  LDSV = 4: the
// four vectors the passes gather (c, g, the CG vector z and the CG step w)
// live in the workgroup's LDS `lv` ([4][kSoloLdsRows]) for the whole solve,
// so a gather costs an LDS access instead of a cache round trip; c is read
// from and written back to global memory at the start and the end.  LDSV =
// 5: q as well ([5][kSoloLdsRows5]).  LDSV = 0: every vector in global memory.
template <int WMAX, int LDSV>
__device__ void solo_solve(const SoloProb &P, const SoloOpts &O, Box B, double *shbuf, double *lv)
{
    int par = 0;   // the half of shbuf the next reduction writes
    const int n = P.n;
    const double dn = n;
    SoloOut S = {};
    int status = NN_EMAXIT;
    double bytes = 0.0;
    const double spmv_b = 4.0 * (dn + 1) + 12.0 * (P.rp[n] - P.rp[0]) + 16.0 * dn;
    constexpr int LR = solo_lds_rows(LDSV);
    double *const C = LDSV ? lv : P.c;
    double *const G = LDSV ? lv + LR : P.g;
    double *const Z = LDSV ? lv + 2 * LR : P.z;
    double *const Wv = LDSV ? lv + 3 * LR : P.w;
    double *const Q = LDSV == 5 ? lv + 4 * LR : P.q;

    // ---- start point and load statistics
    {
        double a[4];
        red_init<OPS4(OP_SUM, OP_MAX, OP_SUM, OP_SUM), 4>(a);
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const double fi = P.f[i];
            a[0] += fi * fi;
            a[1] = fmax(a[1], fi);
            a[2] += isfinite(fi) ? 0.0 : 1.0;
            if (O.c0_mode == 0) {
                C[i] = O.c0v;
            } else {
                const double cv = P.c[i];
                a[3] += isfinite(cv) ? 0.0 : 1.0;
                C[i] = proj_box(cv, B);
            }
        }
        wg_reduce<OPS4(OP_SUM, OP_MAX, OP_SUM, OP_SUM), kDirectAll>(a, shbuf, par);
        bytes += 16.0 * dn;
        S.norm_f = sqrt(a[0]);
        if (a[2] != 0.0 || a[3] != 0.0) {
            status = NN_ENONFINITE;
            goto finish;
        }
        if (B.lo == 0.0 && !(a[1] > 0.0)) {
            // f <= 0 with lower bound 0: c = 0 is the minimiser
            for (int i = threadIdx.x; i < n; i += blockDim.x) C[i] = 0.0;
            S.n_active = n;
            status = NN_OK;
            goto finish;
        }
    }
    {
        const double normf = S.norm_f;
        double t_cauchy = 1.0;
        for (int outer = 0;; outer++) {
            // ---- 1. gradient g = K c - f and the KKT report
            double a5[5];
            red_init<OPS5(OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM), 5>(a5);
            wg_spmv<WMAX>(P, nullptr, [&](int i) { return Two{C[i], P.f[i]}; },
                          [&](int j) { return C[j]; }, [&](int i, double s, Two cf) {
                const double gi = s - cf.b, cv = cf.a;
                G[i] = gi;
                const double pg = cv > B.lo ? (cv < B.hi ? gi : fmax(gi, 0.0)) : fmin(gi, 0.0);
                a5[0] += pg * pg;
                a5[1] += (isfinite(gi) && isfinite(cv)) ? 0.0 : 1.0;
                a5[2] = fmax(a5[2], fabs(fmax(cv - B.hi, fmin(gi, cv - B.lo))));
                a5[3] = fmin(a5[3], cv);
                a5[4] += (cv == B.lo || cv == B.hi) ? 1.0 : 0.0;
            });
            wg_reduce<OPS5(OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM), kDirectAll>(a5, shbuf, par);
            S.spmvs++;
            bytes += spmv_b + 16.0 * dn;
            if (a5[1] != 0.0) {
                status = NN_ENONFINITE;
                break;
            }
            S.kkt_rel = sqrt(a5[0]) / normf;
            S.kkt_nat_inf = a5[2];
            S.min_c = a5[3];
            S.n_active = (int)a5[4];
            S.outer_its = outer;
            if (S.kkt_rel <= O.tol) {
                status = NN_OK;
                break;
            }
            if (outer >= O.max_outer) break;   // NN_EMAXIT

            // ---- 2. Cauchy point: trials s = P(c - t g) - c, K s into ks[buf]
            auto trial = [&](double t, int buf, double &gs, double &sks) {
                auto sv = [&](int j) {
                    const double cj = C[j];
                    return proj_box(cj - t * G[j], B) - cj;
                };
                double a3[2] = {0.0, 0.0};
                wg_spmv<WMAX>(P, nullptr, [&](int i) { return Two{sv(i), G[i]}; }, sv,
                              [&](int i, double s, Two sg) {
                                  P.ks[buf][i] = s;
                                  a3[0] += sg.b * sg.a;
                                  a3[1] += sg.a * s;
                              });
                wg_reduce<OPS2(OP_SUM, OP_SUM), kDirectAll>(a3, shbuf, par);
                gs = a3[0];
                sks = a3[1];
                S.spmvs++;
                S.cauchy_trials++;
                bytes += spmv_b + 16.0 * dn;
            };
            double t = t_cauchy, gs, sks;
            int best = 0;
            trial(t, best, gs, sks);
            if (ok_decrease(gs, sks)) {
                for (int k = 0; k < 20; k++) {
                    double gs2, sks2;
                    trial(t * kExtrap, 1 - best, gs2, sks2);
                    if (!ok_decrease(gs2, sks2)) break;
                    const bool same = gs2 == gs && sks2 == sks;
                    t *= kExtrap;
                    best = 1 - best;
                    gs = gs2;
                    sks = sks2;
                    if (same) break;   // every moving variable has reached its bound
                }
            } else {
                int k = 0;
                for (;;) {
                    t *= kInterp;
                    trial(t, best, gs, sks);
                    if (ok_decrease(gs, sks) || !(++k < kMaxTrials && gs < 0.0)) break;
                }
                if (!ok_decrease(gs, sks)) break;   // rounding floor: NN_EMAXIT
            }
            t_cauchy = t;
            // c = P(c - t g)
            wg_rows(P, [&](int i, bool act) {
                if (act) C[i] = proj_box(C[i] - t * G[i], B);
            });
            bytes += 24.0 * dn;
            __syncthreads();

            // ---- 3. Jacobi-PCG on the free face of the Cauchy point
            double u[4] = {0.0, 0.0, 0.0, 0.0};
            const double *ksb = P.ks[best];
            struct SV {
                double g, ks, c, d;
                int len;
            };
            wg_rows2<4>(P, [&](int i) { return SV{G[i], ksb[i], C[i], P.diag[i], P.rp[i + 1] - P.rp[i]}; },
                        [&](int i, const SV &v) {
                            const double gi = v.g + v.ks;
                            G[i] = gi;
                            const double cv = v.c;
                            const bool fr = !((cv == B.lo && gi >= 0.0) || (cv == B.hi && gi <= 0.0));
                            const double dmi = fr ? 1.0 / v.d : 0.0;
                            const double ri = fr ? -gi : 0.0;
                            const double zi = dmi * ri;
                            P.mask[i] = fr ? 1 : 0;
                            P.dm[i] = dmi;
                            P.r[i] = ri;
                            Z[i] = zi;
                            P.p[i] = 0.0;
                            Q[i] = 0.0;
                            Wv[i] = 0.0;
                            u[0] += ri * zi;
                            u[1] += ri * ri;
                            u[2] += fr ? 1.0 : 0.0;
                            u[3] += fr ? (double)v.len : 0.0;
                        });
            wg_reduce<0u, kDirectAll>(u, shbuf, par);
            bytes += 88.0 * dn;
            double rz = u[0], rr = u[1], rz_prev = 0.0;
            const double nf = u[2], nzf = u[3], rr_stop = O.rtol2 * u[1];
            int it = 0;
            bool cg_fail = false;
            for (int j = 0;; j++) {
                if (!isfinite(rz) || !isfinite(rr)) {
                    status = NN_ENONFINITE;
                    cg_fail = true;
                    break;
                }
                if ((j == 0 && (rr == 0.0 || nf == 0.0)) || (j > 0 && rr <= rr_stop) ||
                    j >= O.max_cg || !(rz > 0.0))
                    break;
                const double beta = j == 0 ? 0.0 : rz / rz_prev;
                // p <- z + beta p, q <- K z + beta q on the free rows (K p by linearity)
                double pq[1] = {0.0};
                wg_spmv<WMAX>(P, P.mask, [&](int i) { return Three{P.p[i], Q[i], Z[i]}; },
                              [&](int jj) { return Z[jj]; }, [&](int i, double kz, Three x) {
                                  const double pi = fma(beta, x.a, x.c);
                                  const double qi = fma(beta, x.b, kz);
                                  P.p[i] = pi;
                                  Q[i] = qi;
                                  pq[0] += pi * qi;
                              });
                wg_reduce<0u, kDirectAll>(pq, shbuf, par);
                if (!(pq[0] > 0.0 && isfinite(pq[0]))) {
                    status = isfinite(pq[0]) ? NN_ENOTSPD : NN_ENONFINITE;
                    cg_fail = true;
                    break;
                }
                const double alpha = rz / pq[0];
                double a2[2] = {0.0, 0.0};
                struct UV {
                    double r, q, dm, p;
                    int m;
                };
                wg_rows2<4>(P, [&](int i) { return UV{P.r[i], Q[i], P.dm[i], P.p[i], P.mask[i]}; },
                            [&](int i, const UV &v) {
                                if (!v.m) return;
                                const double ri = v.r - alpha * v.q;
                                const double zi = v.dm * ri;
                                Wv[i] += alpha * v.p;
                                P.r[i] = ri;
                                Z[i] = zi;
                                a2[0] += ri * zi;
                                a2[1] += ri * ri;
                            });
                wg_reduce<0u, kDirectAll>(a2, shbuf, par);
                rz_prev = rz;
                rz = a2[0];
                rr = a2[1];
                it++;
                S.spmvs++;
                bytes += (dn + 4.0 * nf + 12.0 * nzf + 40.0 * nf) + (dn + 64.0 * nf);
            }
            S.cg_its += it;
            if (cg_fail) break;

            // ---- 4. projected search along w
            double b3[3];
            red_init<OPS3(OP_MIN, OP_SUM, OP_SUM), 3>(b3);
            wg_rows(P, [&](int i, bool act) {
                if (!act) return;
                const double wi = Wv[i], ci = C[i];
                if (wi < 0.0) b3[0] = fmin(b3[0], (ci - B.lo) / (-wi));
                else if (wi > 0.0) b3[0] = fmin(b3[0], (B.hi - ci) / wi);
                b3[1] += G[i] * wi;
                b3[2] += wi * wi;
            });
            wg_reduce<OPS3(OP_MIN, OP_SUM, OP_SUM), kDirectAll>(b3, shbuf, par);
            bytes += 24.0 * dn;
            const double bmin = b3[0], gw = b3[1], wn = sqrt(b3[2]);
            if (it > 0 && gw < 0.0 && wn > 0.0) {
                double ts = 1.0;
                if (bmin < 1.0) {
                    for (int k = 0; k < kMaxTrials; k++) {
                        auto sv = [&](int j) {
                            const double cj = C[j];
                            return proj_box(cj + ts * Wv[j], B) - cj;
                        };
                        double a3[2] = {0.0, 0.0};
                        wg_spmv<WMAX>(P, P.mask, [&](int i) { return Two{sv(i), G[i]}; }, sv,
                                      [&](int, double s, Two sg) {
                                          a3[0] += sg.b * sg.a;
                                          a3[1] += sg.a * s;
                                      });
                        wg_reduce<OPS2(OP_SUM, OP_SUM), kDirectAll>(a3, shbuf, par);
                        S.spmvs++;
                        S.search_trials++;
                        bytes += spmv_b + 16.0 * dn;
                        if (ok_decrease(a3[0], a3[1])) break;
                        ts *= kBack;
                        if (ts <= bmin) {
                            ts = bmin;   // no bound is crossed: decrease is guaranteed
                            break;
                        }
                    }
                }
                if (ts > 0.0) {
                    wg_rows(P, [&](int i, bool act) {
                        if (act) C[i] = proj_box(C[i] + ts * Wv[i], B);
                    });
                    bytes += 24.0 * dn;
                    __syncthreads();
                }
            }
        }
    }
finish:
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const double ci = C[i];
        if (LDSV) P.c[i] = ci;
        if (P.active) P.active[i] = ci == B.lo ? 1 : (ci == B.hi ? 2 : 0);
    }
    if (threadIdx.x == 0) {
        S.status = status;
        S.bytes = bytes;
        *P.out = S;
    }
}

// ---------------------------------------------------------------- diagonal layout
// The same solve where the matrix has the diagonal layout in one regular run:
// the workgroup holds the matrix in registers.  Thread (wavefront w, lane l)
// owns the rows of lane l of the slices w, w + 8, ..., NS of them at most (the
// rows, and so every reduction's order, of the kernel above), with their
// entries (7 or 15; during a CG the last RK of them in registers, the others
// read from the caches each pass), p, q, r and w.  Only what
// neighbours gather lives in LDS, c and one vector y (z of the CG, or the
// trial step s, formed once per row instead of once per gather), with kSoloPad
// zeros on both sides so that no gather tests its index, next to g and
// 1 / diag, which have no room left in registers.  A CG iteration then reads
// 7 or 15 doubles of LDS per row and no memory.
//
// What bounds it: instruction issue of one CU (a 64^2 CG iteration is about 600
// instructions per wavefront, two wavefronts per SIMD) and its LDS reads (63
// slices x 7 x 512 B at 128 B per cycle, 1,770 cycles); passes outside the CG
// also fetch their entries (224 KB).  Measured: 2.45 us per CG iteration and
// 7 us per other pass on the 64^2 square, the solve 5.7 -> 1.9 ms against the
// kernel above; 13^3 rows 1.55 -> 0.86 ms.  The entries are loaded again at each
// CG: kept in registers for the whole solve they were spilled inside the CG
// loop (7.8 us per iteration).  The large variants still spill some of what
// lives across the passes: 16 VGPRs of <7, 8, 7>, 42 of <15, 5, 15> and 127 of
// <15, 8, 8> (none of <7, 2, 7>, <7, 4, 7> and <15, 2, 15>), and all of them
// scalar registers (94 to 395) into lanes of vector registers.
constexpr int kSoloPad = 512;                               // offsets reach at most this far
constexpr int kSoloSpan = kSoloLdsRows + 2 * kSoloPad;      // a gathered vector in LDS

struct SoloDiag {
    int n, nsl;
    DiagReg reg;
    const double *val;   // diagonal arrays
    const double *diag, *f;
    const int *rp;
    double *c;
    uint8_t *active;
    SoloOut *out;
    int64_t nnz;
};

// Global pointers that pass through an empty asm statement (which keeps loads
// from them out of loop-invariant code) keep their address space.
typedef const double __attribute__((address_space(1))) *GlobalD;
typedef const int __attribute__((address_space(1))) *GlobalI;

// Nothing below branches on a row's own state (present, free): a thread
// without a row holds zero entries, and sums take a zero by a select, so the
// register arrays see no divergent control flow.
template <int W, int NS, int RK>
__device__ __forceinline__ void solo_solve_diag(const SoloDiag &P, const SoloOpts &O, Box B,
                                                double *shbuf, double *lds)
{
    constexpr int H = W / 2, LK = W - RK;   // entries 0 .. LK - 1 are read from memory
    static_assert(LK <= H, "the diagonal entry and those after it stay in registers");
    constexpr int T = kSoloBlock;           // row stride between a thread's slices
    int par = 0;
    const int n = P.n;
    const double dn = n;
    int status = NN_EMAXIT, n_active = 0, outer = 0, cg_its = 0, spmvs = 0, ctr = 0, strl = 0;
    double bytes = 0.0, normf, kkt_rel = 0.0, kkt_nat = 0.0, min_c = 0.0;
    const double spmv_b = 4.0 * (dn + 1) + 12.0 * (double)P.nnz + 16.0 * dn;
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int i0 = wid * kSlice + lane;     // row of slice t: i0 + 512 t
    double *const C = lds + kSoloPad + i0;  // C[512 t]: own row
    double *const Y = lds + kSoloSpan + kSoloPad + i0;
    double *const G = lds + 2 * kSoloSpan + i0;
    double *const I = lds + 2 * kSoloSpan + kSoloLdsRows + i0;
    DiagTab<W> tab;
    tab.b0 = P.reg.b0;
    tab.stride = P.reg.stride;
#pragma unroll
    for (int u = 0; u < H; u++) tab.h[u] = P.reg.h[u];

    for (int k = threadIdx.x; k < 2 * kSoloSpan; k += T) lds[k] = 0.0;
    auto mine = [&](int t) { return i0 + t * T < n; };
#pragma unroll
    for (int t = 0; t < NS; t++) {
        const double dg = P.diag[mine(t) ? i0 + t * T : 0];
        I[t * T] = mine(t) ? 1.0 / dg : 0.0;
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();

    // The entries of slice t from entry k0 on (a slice past the last one reads
    // slice 0, a valid address).
    auto load = [&](GlobalD val, int t, int k0, auto &e) {
        const int s = wid + t * kSoloWaves;
        const int row0 = s < P.nsl ? s * kSlice : 0;
#pragma unroll
        for (int k = 0; k < (int)(sizeof(e) / sizeof(double)); k++) {
            int d, b;
            diag_entry<W>(tab, k0 + k, d, b);
            e[k] = (val + (ptrdiff_t)(b + row0))[lane];
        }
    };
    // Row sum of slice t with the gathered vector X (own-row pointer into
    // LDS): the first entries in a, the others in e; own: X of the row.
    auto row_sum = [&](const double *X, int t, const auto &a, const auto &e, double &own) {
        constexpr int NA = (int)(sizeof(a) / sizeof(double));
        double xv[W], acc = 0.0;
#pragma unroll
        for (int k = 0; k < W; k++) {
            int d, b;
            diag_entry<W>(tab, k, d, b);
            xv[k] = X[t * T + d];
        }
        own = xv[H];
#pragma unroll
        for (int k = 0; k < W; k++) acc = __builtin_fma(k < NA ? a[k < NA ? k : 0] : e[k < NA ? 0 : k - NA], xv[k], acc);
        return acc;
    };
    // A pass outside the CG, entries from the caches: epi(t, sum, own x) for
    // every slice t (a slice past the last one has x = 0).  No branch: the
    // loads of a slice summed under one would sink into it and wait there.
    auto product = [&](const double *X, auto epi) {
        GlobalD val = (GlobalD)P.val;
        asm volatile("" : "+s"(val));   // (loads of this pass, not loop-invariant ones)
        // the entries of DEP slices in flight (the CG's vectors are not live
        // here, so there is room for all of a 7-point thread's)
        constexpr int DEP = W == 7 ? NS : (NS < 5 ? NS : 5);
        double e[DEP][W];
#pragma unroll
        for (int t = 0; t < DEP; t++) load(val, t, 0, e[t]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NS; t++) {
            double own;
            const double acc = row_sum(X, t, e[t % DEP], e[t % DEP], own);
            if (t + DEP < NS) load(val, t + DEP, 0, e[t % DEP]);
            epi(t, acc, own);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // ---- start point and load statistics
    {
        double a[4];
        red_init<OPS4(OP_SUM, OP_MAX, OP_SUM, OP_SUM), 4>(a);
#pragma unroll
        for (int t = 0; t < NS; t++) {
            const bool m = mine(t);
            const int i = m ? i0 + t * T : 0;
            const double fi = P.f[i];
            a[0] = m ? a[0] + fi * fi : a[0];
            a[1] = m ? fmax(a[1], fi) : a[1];
            a[2] += m && !isfinite(fi) ? 1.0 : 0.0;
            double cv = O.c0v;
            if (O.c0_mode != 0) {
                cv = P.c[i];
                a[3] += m && !isfinite(cv) ? 1.0 : 0.0;
                cv = proj_box(cv, B);
            }
            C[t * T] = m ? cv : 0.0;
            __builtin_amdgcn_sched_barrier(0);
        }
        wg_reduce<OPS4(OP_SUM, OP_MAX, OP_SUM, OP_SUM), kDirectFew>(a, shbuf, par);
        bytes += 16.0 * dn;
        normf = sqrt(a[0]);
        if (a[2] != 0.0 || a[3] != 0.0) {
            status = NN_ENONFINITE;
            goto finish;
        }
        if (B.lo == 0.0 && !(a[1] > 0.0)) {
            // f <= 0 with lower bound 0: c = 0 is the minimiser
#pragma unroll
            for (int t = 0; t < NS; t++) C[t * T] = 0.0;
            n_active = n;
            status = NN_OK;
            goto finish;
        }
    }
    {
        double t_cauchy = 1.0;
#pragma nounroll
        for (int it_out = 0;; it_out++) {
            // what an iteration reads again (loads, row lengths) is kept out
            // of registers between iterations: the compiler may not take it
            // for loop-invariant
            GlobalD f_in = (GlobalD)P.f;
            GlobalI rp_in = (GlobalI)P.rp;
            int again = 0;
            asm volatile("" : "+s"(f_in), "+s"(rp_in), "+s"(again));
            // ---- 1. gradient g = K c - f and the KKT report
            double a5[5];
            red_init<OPS5(OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM), 5>(a5);
            {
                double fo[NS];
#pragma unroll
                for (int t = 0; t < NS; t++) fo[t] = f_in[mine(t) ? i0 + t * T : 0];
                product(C, [&](int t, double s, double cv) {
                    const bool m = mine(t);
                    const double gi = s - fo[t];
                    G[t * T] = m ? gi : 0.0;
                    double pg = cv > B.lo ? (cv < B.hi ? gi : fmax(gi, 0.0)) : fmin(gi, 0.0);
                    pg = m ? pg : 0.0;
                    a5[0] += pg * pg;
                    a5[1] += m && !(isfinite(gi) && isfinite(cv)) ? 1.0 : 0.0;
                    const double nat = fabs(fmax(cv - B.hi, fmin(gi, cv - B.lo)));
                    a5[2] = m ? fmax(a5[2], nat) : a5[2];
                    a5[3] = m ? fmin(a5[3], cv) : a5[3];
                    a5[4] += m && (cv == B.lo || cv == B.hi) ? 1.0 : 0.0;
                });
            }
            wg_reduce<OPS5(OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM), kDirectFew>(a5, shbuf, par);
            spmvs++;
            bytes += spmv_b + 16.0 * dn;
            if (a5[1] != 0.0) {
                status = NN_ENONFINITE;
                break;
            }
            kkt_rel = sqrt(a5[0]) / normf;
            kkt_nat = a5[2];
            min_c = a5[3];
            n_active = (int)a5[4];
            outer = it_out;
            if (kkt_rel <= O.tol) {
                status = NN_OK;
                break;
            }
            if (it_out >= O.max_outer) break;   // NN_EMAXIT

            // ---- 2. Cauchy point: trials s = P(c - t g) - c (s in Y), K s kept
            double ksb[NS], ksn[NS];
            auto trial = [&](double t_, double (&ks)[NS], double &gs, double &sks) {
#pragma unroll
                for (int t = 0; t < NS; t++) {
                    const double ci = C[t * T];
                    const double si = proj_box(ci - t_ * G[t * T], B) - ci;
                    Y[t * T] = mine(t) ? si : 0.0;
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
                double a3[2] = {0.0, 0.0};
                product(Y, [&](int t, double s, double si) {
                    ks[t] = s;
                    a3[0] += G[t * T] * si;
                    a3[1] += si * s;
                });
                wg_reduce<OPS2(OP_SUM, OP_SUM), kDirectFew>(a3, shbuf, par);
                gs = a3[0];
                sks = a3[1];
                spmvs++;
                ctr++;
                bytes += spmv_b + 16.0 * dn;
            };
            double t = t_cauchy, gs, sks;
#pragma unroll
            for (int q = 0; q < NS; q++) ksb[q] = ksn[q] = 0.0;
            trial(t, ksb, gs, sks);
            if (ok_decrease(gs, sks)) {
#pragma nounroll
                for (int k = 0; k < 20; k++) {
                    double gs2, sks2;
                    trial(t * kExtrap, ksn, gs2, sks2);
                    if (!ok_decrease(gs2, sks2)) break;
                    const bool same = gs2 == gs && sks2 == sks;
                    t *= kExtrap;
#pragma unroll
                    for (int q = 0; q < NS; q++) ksb[q] = ksn[q];
                    gs = gs2;
                    sks = sks2;
                    if (same) break;   // every moving variable has reached its bound
                }
            } else {
                int k = 0;
#pragma nounroll
                for (;;) {
                    t *= kInterp;
                    trial(t, ksb, gs, sks);
                    if (ok_decrease(gs, sks) || !(++k < kMaxTrials && gs < 0.0)) break;
                }
                if (!ok_decrease(gs, sks)) break;   // rounding floor: NN_EMAXIT
            }
            t_cauchy = t;
            bytes += 24.0 * dn;

            // ---- 3. c = P(c - t g), and Jacobi-PCG on the free face there
            double p[NS], q[NS], r[NS], w[NS];
            uint32_t fre = 0;     // free rows of this thread
            uint32_t live = 0;    // slices with a free row (uniform)
            double u[4] = {0.0, 0.0, 0.0, 0.0};
            int len[NS];
#pragma unroll
            for (int t2 = 0; t2 < NS; t2++) {
                const int i = mine(t2) ? i0 + t2 * T : 0;
                len[t2] = rp_in[i + 1] - rp_in[i];
            }
#pragma unroll
            for (int t2 = 0; t2 < NS; t2++) {
                const bool m = mine(t2);
                const double g0 = G[t2 * T];
                const double cv = proj_box(C[t2 * T] - t * g0, B);
                C[t2 * T] = m ? cv : 0.0;
                const double gi = g0 + ksb[t2];
                G[t2 * T] = m ? gi : 0.0;
                const bool fr = m && !((cv == B.lo && gi >= 0.0) || (cv == B.hi && gi <= 0.0));
                const double dmi = fr ? I[t2 * T] : 0.0;
                const double ri = fr ? -gi : 0.0;
                const double zi = dmi * ri;
                p[t2] = q[t2] = w[t2] = 0.0;
                r[t2] = ri;
                Y[t2 * T] = zi;
                u[0] += ri * zi;
                u[1] += ri * ri;
                u[2] += fr ? 1.0 : 0.0;
                u[3] += fr ? (double)len[t2] : 0.0;
                fre |= fr ? 1u << t2 : 0u;
                if (__ballot(fr) != 0) live |= 1u << t2;
                __builtin_amdgcn_sched_barrier(0);
            }
            wg_reduce<0u, kDirectFew>(u, shbuf, par);
            bytes += 88.0 * dn;
            // the CG's entries in registers
            double v[NS][RK];
            GlobalD val = (GlobalD)P.val;
            asm volatile("" : "+s"(val));
#pragma unroll
            for (int t2 = 0; t2 < NS; t2++) load(val, t2, LK, v[t2]);
            double rz = u[0], rr = u[1], rz_prev = 0.0;
            const double nf = u[2], nzf = u[3], rr_stop = O.rtol2 * u[1];
            int it = 0;
            bool cg_fail = false;
#pragma nounroll
            for (int j = 0;; j++) {
                if (!isfinite(rz) || !isfinite(rr)) {
                    status = NN_ENONFINITE;
                    cg_fail = true;
                    break;
                }
                if ((j == 0 && (rr == 0.0 || nf == 0.0)) || (j > 0 && rr <= rr_stop) ||
                    j >= O.max_cg || !(rz > 0.0))
                    break;
                const double beta = j == 0 ? 0.0 : rz / rz_prev;
                // p <- z + beta p, q <- K z + beta q on the free rows (K p by
                // linearity); the others keep p = q = 0 (z = 0 there)
                double pq[1] = {0.0};
                if constexpr (LK > 0) asm volatile("" : "+s"(val));
#pragma unroll
                for (int t2 = 0; t2 < NS; t2++) {
                    if (!((live >> t2) & 1)) continue;
                    double lv[LK > 0 ? LK : 1], zi, kz;
                    if constexpr (LK > 0) {
                        load(val, t2, 0, lv);
                        kz = row_sum(Y, t2, lv, v[t2], zi);
                    } else {
                        kz = row_sum(Y, t2, v[t2], v[t2], zi);
                    }
                    const double kf = (fre >> t2) & 1 ? kz : 0.0;
                    const double pi = fma(beta, p[t2], zi);
                    const double qi = fma(beta, q[t2], kf);
                    p[t2] = pi;
                    q[t2] = qi;
                    pq[0] += pi * qi;
                    __builtin_amdgcn_sched_barrier(0);   // one slice's gathers in registers at a time
                }
                wg_reduce<0u, kDirectFew>(pq, shbuf, par);
                if (!(pq[0] > 0.0 && isfinite(pq[0]))) {
                    status = isfinite(pq[0]) ? NN_ENOTSPD : NN_ENONFINITE;
                    cg_fail = true;
                    break;
                }
                const double alpha = rz / pq[0];
                asm volatile("" : "+s"(again));   // (nor 1 / diag here)
                double a2[2] = {0.0, 0.0};
#pragma unroll
                for (int t2 = 0; t2 < NS; t2++) {
                    const double ri = r[t2] - alpha * q[t2];
                    const double zi = I[again + t2 * T] * ri;   // (r = 0 off the free rows)
                    w[t2] += alpha * p[t2];
                    r[t2] = ri;
                    Y[t2 * T] = zi;
                    a2[0] += ri * zi;
                    a2[1] += ri * ri;
                }
                wg_reduce<0u, kDirectFew>(a2, shbuf, par);
                rz_prev = rz;
                rz = a2[0];
                rr = a2[1];
                it++;
                spmvs++;
                bytes += (dn + 4.0 * nf + 12.0 * nzf + 40.0 * nf) + (dn + 64.0 * nf);
            }
            cg_its += it;
            if (cg_fail) break;

            // ---- 4. projected search along w
            double b3[3];
            red_init<OPS3(OP_MIN, OP_SUM, OP_SUM), 3>(b3);
#pragma unroll
            for (int t2 = 0; t2 < NS; t2++) {
                // (w = 0 off the free rows: no crossing, nothing added)
                const double wi = w[t2], ci = C[t2 * T];
                const double room = wi < 0.0 ? ci - B.lo : B.hi - ci;
                const double brk = room / fabs(wi);
                b3[0] = wi != 0.0 ? fmin(b3[0], brk) : b3[0];
                b3[1] += G[t2 * T] * wi;
                b3[2] += wi * wi;
            }
            wg_reduce<OPS3(OP_MIN, OP_SUM, OP_SUM), kDirectFew>(b3, shbuf, par);
            bytes += 24.0 * dn;
            const double bmin = b3[0], gw = b3[1], wn = sqrt(b3[2]);
            if (it > 0 && gw < 0.0 && wn > 0.0) {
                double ts = 1.0;
                if (bmin < 1.0) {
#pragma nounroll
                    for (int k = 0; k < kMaxTrials; k++) {
#pragma unroll
                        for (int t2 = 0; t2 < NS; t2++) {
                            const double ci = C[t2 * T];
                            const double si = proj_box(ci + ts * w[t2], B) - ci;
                            Y[t2 * T] = mine(t2) ? si : 0.0;
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        __syncthreads();
                        double a3[2] = {0.0, 0.0};
                        product(Y, [&](int t2, double s, double si) {
                            const double sf = (fre >> t2) & 1 ? si : 0.0;
                            a3[0] += G[t2 * T] * sf;
                            a3[1] += sf * s;
                        });
                        wg_reduce<OPS2(OP_SUM, OP_SUM), kDirectFew>(a3, shbuf, par);
                        spmvs++;
                        strl++;
                        bytes += spmv_b + 16.0 * dn;
                        if (ok_decrease(a3[0], a3[1])) break;
                        ts *= kBack;
                        if (ts <= bmin) {
                            ts = bmin;   // no bound is crossed: decrease is guaranteed
                            break;
                        }
                    }
                }
                if (ts > 0.0) {
#pragma unroll
                    for (int t2 = 0; t2 < NS; t2++) {
                        const double cn = proj_box(C[t2 * T] + ts * w[t2], B);
                        C[t2 * T] = mine(t2) ? cn : 0.0;
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    bytes += 24.0 * dn;
                    __syncthreads();
                }
            }
        }
    }
finish:
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NS; t++) {
        if (!mine(t)) continue;
        const int i = i0 + t * T;
        const double ci = C[t * T];
        P.c[i] = ci;
        if (P.active) P.active[i] = ci == B.lo ? 1 : (ci == B.hi ? 2 : 0);
    }
    if (threadIdx.x == 0) {
        SoloOut S = {};
        S.kkt_rel = kkt_rel;
        S.kkt_nat_inf = kkt_nat;
        S.min_c = min_c;
        S.norm_f = normf;
        S.bytes = bytes;
        S.outer_its = outer;
        S.cg_its = cg_its;
        S.spmvs = spmvs;
        S.n_active = n_active;
        S.cauchy_trials = ctr;
        S.search_trials = strl;
        S.status = status;
        *P.out = S;
    }
}

template <int W, int NS, int RK>
__global__ __launch_bounds__(kSoloBlock, 2) void k_solo_diag(SoloDiag P, SoloOpts O, Box B)
{
    __shared__ __align__(16) double shbuf[2 * kSoloWaves * (kMaxRed + 1)];
    __shared__ double lds[2 * kSoloSpan + 2 * kSoloLdsRows];
    solo_solve_diag<W, NS, RK>(P, O, B, shbuf, lds);
}

template <int WMAX, int LDSV>
__global__ __launch_bounds__(kSoloBlock) void k_solo(SoloProb P, SoloOpts O, Box B)
{
    __shared__ __align__(16) double shbuf[2 * kSoloWaves * (kMaxRed + 1)];
    if constexpr (LDSV > 0) {
        __shared__ double lv[LDSV * solo_lds_rows(LDSV)];
        solo_solve<WMAX, LDSV>(P, O, B, shbuf, lv);
    } else {
        solo_solve<WMAX, 0>(P, O, B, shbuf, nullptr);
    }
}

}  // namespace

bool solo_eligible(const nn_matrix *A, const nn_opts *o)
{
    return A->n > 0 && A->n < ((int64_t)1 << 31) / kSlice && o->method == NN_TRON &&
           o->precision == NN_FP64 && !(o->delta0 > 0.0) && o->precond_degree <= 1 &&
           o->subspace == 0 && o->verbose == 0;
}

nn_status solo_solve_impl(nn_ctx *ctx, const nn_matrix *A, const double *vals,
                          const double *vals64p, const double *diag, const double *f, const nn_opts *o, double *c, uint8_t *active,
                          nn_stats *st)
{
    const int64_t n = A->n;
    nn_status rc = ensure_workspace(ctx, n);
    if (rc != NN_OK) return rc;
    Workspace &W = ctx->ws;
    SoloProb P;
    P.n = (int)n;
    P.nsl = (int)A->nslices;
    P.so = A->sl_off;
    P.sc = A->sl_col;
    P.rp = A->rowptr;
    P.v = vals;
    P.diag = diag;
    P.f = f;
    P.c = c;
    P.active = active;
    P.g = W.g;
    P.w = W.w;
    P.r = W.r;
    P.z = W.z;
    P.p = W.p0;
    P.q = W.q;
    P.ks[0] = W.ks0;
    P.ks[1] = W.ks1;
    P.dm = W.dm;
    P.mask = W.mask;
    // the report goes through the reduction partials (free between calls)
    P.out = reinterpret_cast<SoloOut *>(ctx->partials);
    SoloOpts O;
    O.tol = o->tol;
    O.rtol2 = o->inner_rtol * o->inner_rtol;
    O.c0v = std::min(std::max(o->c0_value, o->lower), o->upper);
    O.c0_mode = o->c0_mode == 1 ? 1 : 0;
    O.max_outer = o->max_outer;
    O.max_cg = o->max_cg;
    Box box;
    box.lo = o->lower;
    box.hi = o->upper;
    NN_HIP_TRY(ctx, hipEventRecord(ctx->ev0, ctx->stream));
    const int lds = n <= kSoloLdsRows5 ? 5 : (n <= kSoloLdsRows ? 4 : 0);
#define NN_SOLO_LAUNCH(WM)                                                                       \
    do {                                                                                         \
        if (lds == 5)                                                                            \
            hipLaunchKernelGGL((k_solo<WM, 5>), dim3(1), dim3(kSoloBlock), 0, ctx->stream, P,    \
                               O, box);                                                          \
        else if (lds == 4)                                                                       \
            hipLaunchKernelGGL((k_solo<WM, 4>), dim3(1), dim3(kSoloBlock), 0, ctx->stream, P,    \
                               O, box);                                                          \
        else                                                                                     \
            hipLaunchKernelGGL((k_solo<WM, 0>), dim3(1), dim3(kSoloBlock), 0, ctx->stream, P,    \
                               O, box);                                                          \
    } while (0)
    // The matrix in registers: one regular run over all slices, offsets inside
    // the LDS padding, at most eight slices per wavefront.  63^2 and 13^3 rows:
    // 1.93 and 0.86 ms, k_solo 5.69 and 1.55.
    // NS, the slices a thread has room for, is the smallest that fits, as every
    // pass works through all of them: 16 slices in all 0.58 ms at NS = 2, 0.78 at
    // 4, 1.31 at 8 (15-point rows: 0.39 at 2, 0.80 at 5, 1.19 at 8), 32 slices
    // 0.92 at 4, 1.50 at 8 (15-point, 35 slices: 0.86 at 5, 1.34 at 8).  Above
    // five slices a thread's 15-point rows leave no room for their first seven
    // entries.
    DiagReg reg{};
    const bool one_run = vals64p && n <= kSoloLdsRows && diag_one_run(A, &reg) &&
                         reg.h[A->wmax <= 8 ? 2 : 6] <= kSoloPad;
    const int ns = (P.nsl + kSoloWaves - 1) / kSoloWaves;
    const SoloDiag D{P.n, P.nsl, reg, vals64p, diag, f, A->rowptr, c, active, P.out, A->nnz};
#define NN_SOLO_DIAG(W, NS, RK)                                                                  \
    hipLaunchKernelGGL((k_solo_diag<W, NS, RK>), dim3(1), dim3(kSoloBlock), 0, ctx->stream, D, O, \
                       box)
    if (one_run && A->wmax <= 8) {
        if (ns <= 2) NN_SOLO_DIAG(7, 2, 7);
        else if (ns <= 4) NN_SOLO_DIAG(7, 4, 7);
        else NN_SOLO_DIAG(7, 8, 7);
    } else if (one_run) {
        if (ns <= 2) NN_SOLO_DIAG(15, 2, 15);
        else if (ns <= 5) NN_SOLO_DIAG(15, 5, 15);
        else NN_SOLO_DIAG(15, 8, 8);
    } else if (A->wmax <= 8) NN_SOLO_LAUNCH(8);
    else if (A->wmax <= 16) NN_SOLO_LAUNCH(16);
    else NN_SOLO_LAUNCH(32);
#undef NN_SOLO_DIAG
#undef NN_SOLO_LAUNCH
    NN_HIP_TRY(ctx, hipGetLastError());
    SoloOut R;
    NN_HIP_TRY(ctx, hipMemcpyAsync(&R, P.out, sizeof(SoloOut), hipMemcpyDeviceToHost, ctx->stream));
    NN_HIP_TRY(ctx, hipEventRecord(ctx->ev1, ctx->stream));
    NN_HIP_TRY(ctx, hipEventSynchronize(ctx->ev1));
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, ctx->ev0, ctx->ev1);
    nn_stats S;
    std::memset(&S, 0, sizeof(S));
    S.kkt_rel = R.kkt_rel;
    S.kkt_nat_inf = R.kkt_nat_inf;
    S.min_c = R.min_c;
    S.norm_f = R.norm_f;
    S.outer_its = R.outer_its;
    S.cg_its = R.cg_its;
    S.spmvs = R.spmvs;
    S.n_active = R.n_active;
    S.cauchy_trials = R.cauchy_trials;
    S.search_trials = R.search_trials;
    S.status = R.status;
    S.bytes_moved = R.bytes;
    S.seconds = ms * 1e-3;
    if (st) *st = S;
    switch (R.status) {
    case NN_OK:
        ctx->err.clear();
        return NN_OK;
    case NN_EMAXIT:
        return fail(ctx, NN_EMAXIT, "outer iteration cap or rounding floor reached");
    case NN_ENONFINITE:
        return fail(ctx, NN_ENONFINITE, "non-finite value in the solve");
    case NN_ENOTSPD:
        return fail(ctx, NN_ENOTSPD, "non-positive curvature in CG");
    default:
        return fail(ctx, (nn_status)R.status, "solve failed");
    }
}

}  // namespace nnqp
