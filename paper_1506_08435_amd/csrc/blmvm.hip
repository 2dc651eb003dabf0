// Bounded limited-memory variable-metric (BLMVM) solver for
//     min 1/2 c.Kc - c.f  subject to  lo <= c <= hi
// the gradient-only method the paper runs beside TRON through TAO (Sec. 3.1,
// Sec. 5.1; the objective and gradient callbacks of eq. S3_tao_objective and
// eq. S3_tao_gradient are all it uses).  The method is that of Benson & More
// (2001): an L-BFGS inverse-Hessian approximation H built from the steps s and
// the differences y of projected gradients, search direction d = -H pg, and a
// projected line search.  Here, for the quadratic objective:
//
//   1. Pair pass (one kernel over the rows): pg at the current point, the new
//      y = pg - pg_prev when a step was just taken, and every inner product
//      the compact representation needs (s_j.pg, y_j.pg, s_j.y, y_j.y, s.s).
//   2. Coefficient kernel (one block): accepts the new pair when
//      s.y > 1e-12 |s| |y| (else drops it; a full memory then loses its
//      oldest pair), sets gamma = s.y / y.y, and solves the small triangular
//      systems of the compact form (Byrd, Nocedal & Schnabel 1994)
//          H v = gamma v + S t - gamma Y p,  p = R^-1 S'v,
//          t = R^-T ((D + gamma Y'Y) p - gamma Y'v),
//      R the upper triangle of S'Y and D its diagonal (pairs oldest first).
//   3. Direction pass: d = -H pg from those coefficients, with every
//      component that points out of the box at a bound set to zero (the
//      projection would cancel it for any step), the first bound crossing
//      along d, g.d and d.d.
//   4. Line search: when no bound is crossed up to t = 1, one trial at t = 1
//      gives K d, and the step is the exact minimiser of the quadratic along
//      d (capped at the first crossing); otherwise projected backtracking
//      c(t) = P(c + t d), t = 1, 1/2, ..., until the sufficient-decrease test
//      holds, finishing with the exact step on the segment [0, crossing] if t
//      reaches it.  Each trial is one matrix pass that gathers P(c + t d), at
//      t = 1 as the direction pass left it, and
//      returns the gradient K c(t) - f at the trial point.
//   5. Step: c <- c(t), s stored in the next pair slot, g updated; done by
//      the next iteration's pair pass (one pass over the rows fewer), or by a
//      step kernel when a gradient refresh comes first.
// g is refreshed with a plain gradient pass every 50 iterations that did not
// end on a freshly computed gradient, and before convergence is accepted.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>

#include "nnqp_internal.hpp"
#include "diag.hpp"

namespace nnqp {

namespace {

constexpr int kLmMax = 8;                  // pair slots supported
constexpr int kLmNV = 4 * kLmMax + 3;      // values of the pair pass at kLmMax
static_assert(kLmMax * kLmMax <= 64, "one lane per table entry in the coefficient kernel");
constexpr double kLmMu = 0.01;             // sufficient-decrease constant
constexpr double kLmCurv = 1e-12;          // pair acceptance: s.y > kLmCurv |s| |y|
constexpr int kLmRefresh = 50;             // iterations between gradient refreshes
constexpr int kLmMaxTrials = 60;

struct LmState {
    int count;        // stored pairs
    int head;         // slot the next pair is written to
    int pending;      // a step was taken: its s is in slot head, its y is formed next
    int accepted;     // pairs accepted / rejected so far
    int rejected;
    double gamma;     // H0 = gamma I
    double pg2;       // |pg|^2 at the current point
    double nonfinite; // non-finite c or g entries at the current point
    double sy[kLmMax][kLmMax];   // s_a . y_b by slot (used for a older than or equal to b)
    double yy[kLmMax][kLmMax];   // y_a . y_b by slot
    double sc[kLmMax];           // coefficient of s_slot in H pg
    double yc[kLmMax];           // coefficient of y_slot in H pg
};

// slot j is live in the pair pass: a stored pair, or the pair being formed
__device__ __forceinline__ bool lm_live(int j, int M, int count, int head, int pending)
{
    const int age = (head - j + M) % M;   // 1 = newest stored pair, ..., M = oldest when full
    return (pending && j == head) || (age >= 1 && age <= count) || (count == M && j == head);
}

// The pair pass holds 4M + 3 accumulators per lane (95 VGPRs at M = 5), so
// one 1024-thread block fits a CU: it runs one block per CU and walks more
// slices per wavefront instead of queueing a second round of blocks.
constexpr int kPairBlocks = 256;

// Wavefront totals of NV sums: a[j] of the lanes 16 q .. 16 q + 15 becomes the
// total of value wave_sums_value<NV>(j, q), the bits wave_sum would give.  The
// levels 32 and 16 of the butterfly add the same pair in both its lanes, so
// two values share a register after each: a swap of half the lanes between
// them and one addition, and the last four levels run on a quarter of the
// values.  At 23 values a wavefront issues 130 instructions instead of 410; a
// full CU issues them for four wavefronts on each SIMD (pair pass of 166 k
// rows, five pairs: 11.4 -> 7.4 us).
template <int NV>
__host__ __device__ constexpr int wave_sums_regs() { return (NV + 3) / 4; }
template <int NV>
__device__ __forceinline__ int wave_sums_value(int j, int q)
{
    constexpr int G = wave_sums_regs<NV>();   // q = 0: j, 1: j + G, 2: j + 2G, 3: j + 3G
    return j + G * q;
}

__device__ __forceinline__ void swap32(double &a, double &b)   // a: low halves, b: high halves
{
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(h[0], l[0]);
    b = __hiloint2double(h[1], l[1]);
}
__device__ __forceinline__ void swap16(double &a, double &b)   // a: even rows, b: odd rows
{
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(h[0], l[0]);
    b = __hiloint2double(h[1], l[1]);
}

template <int NV>
__device__ __forceinline__ void wave_sums(double (&a)[NV])
{
    constexpr int G = wave_sums_regs<NV>();
    const auto add = [](double x, double y) { return x + y; };
#pragma unroll
    for (int j = 0; j < G; j++) {
        double v[4];
#pragma unroll
        for (int q = 0; q < 4; q++) v[q] = j + G * q < NV ? a[j + G * q] : 0.0;
        // lanes 0..31: values 0 and 1, lanes 32..63: values 2 and 3
        swap32(v[0], v[2]);
        swap32(v[1], v[3]);
        double x = v[0] + v[2], y = v[1] + v[3];
        swap16(x, y);
        x = x + y;
        x = wave_level<8>(x, add);
        x = wave_level<4>(x, add);
        x = wave_level<2>(x, add);
        a[j] = wave_level<1>(x, add);
    }
}

// Block total of NV sums (fixed order: butterfly within the wavefront, waves
// in order) stored as this block's partial part[k * kMaxBlocks + block].
template <int NV>
__device__ __forceinline__ void block_sums(double (&a)[NV], double *part, const Part &P)
{
    constexpr int G = wave_sums_regs<NV>();
    __shared__ double sh[kWaves][4 * G];
    const int lane = threadIdx.x & 63, wid = wave_id();
    wave_sums<NV>(a);
    if ((lane & 15) == 0)
#pragma unroll
        for (int j = 0; j < G; j++) sh[wid][wave_sums_value<NV>(j, lane >> 4)] = a[j];
    __syncthreads();
    for (int k = threadIdx.x; k < NV; k += kBlock) {
        double v = sh[0][k];
#pragma unroll
        for (int w = 1; w < kWaves; w++) v += sh[w][k];
        part[k * kMaxBlocks + block_id(P)] = v;
    }
}

// 1. pair pass (see the file comment); values: |pg|^2, #non-finite,
// s_j.pg, y_j.pg, s_j.y, y_j.y (j = 0..M-1 by slot), s.s.
// With `apply` the step of the previous iteration is taken here first (the
// step kernel fused in): c <- P(c + t d), s = c_new - c into slot head,
// g <- g + gscale (gn - g) (gscale = 1: gn itself), and the pair is formed
// from that s.
template <int M>
__global__ __launch_bounds__(kBlock) void kl_pairs(Part P, double *__restrict__ c,
                                                   double *__restrict__ g,
                                                   double *__restrict__ pg,
                                                   double *__restrict__ S,
                                                   double *__restrict__ Y, int64_t ld,
                                                   const LmState *__restrict__ st, Box B,
                                                   double *part, int apply,
                                                   const double *__restrict__ d, double t,
                                                   const double *__restrict__ gn, double gscale)
{
    constexpr int NV = 4 * M + 3;
    const int count = st->count, head = st->head, pending = apply || st->pending;
    bool live[M];
#pragma unroll
    for (int j = 0; j < M; j++) live[j] = lm_live(j, M, count, head, pending);
    double a[NV];
#pragma unroll
    for (int k = 0; k < NV; k++) a[k] = 0.0;
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        // every load of the row is issued here, before the state decides what
        // is used (slots that hold no pair hold finite numbers)
        double ci = c[i], gi = g[i], sn = 0.0;
        const double pg0 = pg[i];
        double di = 0.0, gni = 0.0;
        if (apply) {
            di = d[i];
            gni = gn[i];
        }
        double sv[M], yv[M];
#pragma unroll
        for (int j = 0; j < M; j++) {
            sv[j] = S[j * ld + i];
            yv[j] = Y[j * ld + i];
        }
        if (apply) {
            const double cn = proj_box(ci + t * di, B);
            sn = cn - ci;
            ci = cn;
            gi = gscale == 1.0 ? gni : gi + gscale * (gni - gi);
            c[i] = ci;
            g[i] = gi;
            S[head * ld + i] = sn;
        } else if (pending) {
#pragma unroll
            for (int j = 0; j < M; j++) sn = j == head ? sv[j] : sn;
        }
        const double pgi = ci > B.lo ? (ci < B.hi ? gi : fmax(gi, 0.0)) : fmin(gi, 0.0);
        a[0] += pgi * pgi;
        a[1] += (isfinite(ci) && isfinite(gi)) ? 0.0 : 1.0;
        double yn = 0.0;
        if (pending) {
            yn = pgi - pg0;
            Y[head * ld + i] = yn;
            a[2 + 4 * M] += sn * sn;
        }
        pg[i] = pgi;
#pragma unroll
        for (int j = 0; j < M; j++) {
            if (!live[j]) continue;
            const bool fresh = pending && j == head;
            const double sj = fresh ? sn : sv[j];
            const double yj = fresh ? yn : yv[j];
            a[2 + j] += sj * pgi;
            a[2 + M + j] += yj * pgi;
            if (pending) {
                a[2 + 2 * M + j] += sj * yn;
                a[2 + 3 * M + j] += yj * yn;
            }
        }
    });
    block_sums<NV>(a, part, P);
}

// 2. coefficient kernel: one block.  Each wavefront combines the block
// partials of a few of the pair pass's values (lane-strided sums, then a
// butterfly: fixed order) and the first one does the small algebra, every
// lane the same, in registers: the tables are read from LDS by age (oldest
// first) in one go, and loops over the pairs are unrolled with the bounds as
// conditions.  As one wavefront whose lane 0 indexed private arrays by age it
// spent 14.7 us on chains of scratch and LDS accesses (five pairs), now 4.2.
constexpr int kCoefWaves = 8;

template <int M>
__global__ __launch_bounds__(64 * kCoefWaves) void kl_coef(int nb, LmState *st, const double *part,
                                                           int applied)
{
    constexpr int NV = 4 * M + 3;
    __shared__ double t[NV];
    __shared__ double sy[M][M], yy[M][M];
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int count0 = st->count, head0 = st->head, pend0 = st->pending;
    const int acc0 = st->accepted, rej0 = st->rejected;
    const double gam0 = st->gamma;
    if (threadIdx.x < M * M) {
        sy[threadIdx.x / M][threadIdx.x % M] = st->sy[threadIdx.x / M][threadIdx.x % M];
        yy[threadIdx.x / M][threadIdx.x % M] = st->yy[threadIdx.x / M][threadIdx.x % M];
    }
    {
        constexpr int KW = (NV + kCoefWaves - 1) / kCoefWaves, R = kPairBlocks / 64;
        double x[KW][R];
#pragma unroll
        for (int q = 0; q < KW; q++)
#pragma unroll
            for (int r = 0; r < R; r++) {
                const int k = min(wid + q * kCoefWaves, NV - 1);
                x[q][r] = part[k * kMaxBlocks + lane + 64 * r];   // inside the array for every lane
            }
#pragma unroll
        for (int q = 0; q < KW; q++) {
            double v = 0.0;   // (an absent block adds +0.0, which changes no sum from +0.0)
#pragma unroll
            for (int r = 0; r < R; r++) v += lane + 64 * r < nb ? x[q][r] : 0.0;
            v = wave_sum(v);
            if (lane == 0 && wid + q * kCoefWaves < NV) t[wid + q * kCoefWaves] = v;
        }
    }
    __syncthreads();
    if (wid != 0) return;
    int count = count0, head = head0;
    double gam = gam0;
    const bool pending = pend0 || applied;
    bool ok = false;
    if (pending) {
        const double sny = t[2 + 2 * M + head], yny = t[2 + 3 * M + head], ss = t[2 + 4 * M];
        ok = isfinite(sny) && isfinite(yny) && yny > 0.0 && sny > kLmCurv * sqrt(ss) * sqrt(yny);
        if (ok) {
            // column `head` of S'Y and Y'Y against every pair that stays
            if (lane < M && lm_live(lane, M, count, head, 1)) {
                const double syv = t[2 + 2 * M + lane], yyv = t[2 + 3 * M + lane];
                sy[lane][head] = st->sy[lane][head] = syv;
                yy[lane][head] = st->yy[lane][head] = yyv;
                yy[head][lane] = st->yy[head][lane] = yyv;
            }
            count = count < M ? count + 1 : M;
            head = (head + 1) % M;
            gam = sny / yny;
        } else if (count == M) {
            count = M - 1;   // its oldest pair was overwritten
        }
    }
    // (one wavefront: its LDS writes precede its reads)
    __builtin_amdgcn_wave_barrier();
    // compact-form coefficients over the pairs, oldest first
    double R[M][M], Q[M][M], u[M], w[M], p[M], z[M], tp[M];
    int sl[M];
#pragma unroll
    for (int k = 0; k < M; k++) {
        sl[k] = (head - count + k + 2 * M) % M;
        u[k] = t[2 + sl[k]];
        w[k] = t[2 + M + sl[k]];
        p[k] = z[k] = tp[k] = 0.0;
    }
#pragma unroll
    for (int a = 0; a < M; a++)
#pragma unroll
        for (int b = 0; b < M; b++) {
            if (b >= a) R[a][b] = sy[sl[a]][sl[b]];
            Q[a][b] = yy[sl[a]][sl[b]];
        }
#pragma unroll
    for (int a = M - 1; a >= 0; a--)
        if (a < count) {
            double v = u[a];
#pragma unroll
            for (int b = a + 1; b < M; b++)
                if (b < count) v -= R[a][b] * p[b];
            p[a] = v / R[a][a];
        }
#pragma unroll
    for (int a = 0; a < M; a++)
        if (a < count) {
            double v = R[a][a] * p[a] - gam * w[a];
#pragma unroll
            for (int b = 0; b < M; b++)
                if (b < count) v += gam * Q[a][b] * p[b];
            z[a] = v;
        }
#pragma unroll
    for (int a = 0; a < M; a++)
        if (a < count) {
            double v = z[a];
#pragma unroll
            for (int b = 0; b < a; b++) v -= R[b][a] * tp[b];
            tp[a] = v / R[a][a];
        }
    if (lane < M) {
        // the lane's slot: its age, or none
        double scv = 0.0, ycv = 0.0;
#pragma unroll
        for (int a = 0; a < M; a++)
            if (a < count && sl[a] == lane) {
                scv = tp[a];
                ycv = -gam * p[a];
            }
        st->sc[lane] = scv;
        st->yc[lane] = ycv;
    }
    if (lane == 0) {
        st->pg2 = t[0];
        st->nonfinite = t[1];
        if (pending) {
            if (ok) st->accepted = acc0 + 1;
            else st->rejected = rej0 + 1;
            st->pending = 0;
        }
        st->count = count;
        st->head = head;
        st->gamma = gam;
    }
}

// What the host reads after a direction and its first trial, written straight
// into its pinned memory (a copy behind the kernel is one more launch in the chain).
struct LmHost {
    unsigned long long seq;      // number of the summary, stored last
    double gamma, pg2, nonfinite;
    double bmin, gd;             // direction: first bound crossing, g.d
    double gs, sks;              // trial at t = 1: g.s, s.(gn - g)
    int count;
};

// Combines the direction pass partials (SLOT_Q: first crossing, g.d) and the
// trial's (host slot: g.s, s.(gn - g)), one wavefront each (lane-strided, then
// a butterfly: fixed order).
__global__ __launch_bounds__(256) void kl_summary(int nb, const LmState *st, const double *partials,
                                                  LmHost *out, unsigned long long seq)
{
    const int lane = threadIdx.x & 63, wid = wave_id();
    const double *q = partials + (size_t)(wid < 2 ? SLOT_Q : SLOT_HOST) * kMaxRed * kMaxBlocks +
                      (wid & 1) * kMaxBlocks;
    constexpr int R = kMaxBlocks / 64;
    double x[R];
#pragma unroll
    for (int r = 0; r < R; r++) x[r] = q[lane + 64 * r];   // inside the slot for every lane
    if (threadIdx.x == 0) {
        out->count = st->count;
        out->gamma = st->gamma;
        out->pg2 = st->pg2;
        out->nonfinite = st->nonfinite;
    }
    if (wid == 0) {
        double v = INFINITY;
#pragma unroll
        for (int r = 0; r < R; r++)
            if (lane + 64 * r < nb) v = fmin(v, x[r]);
        v = wave_min(v);
        if (lane == 0) out->bmin = v;
    } else {
        double v = 0.0;
#pragma unroll
        for (int r = 0; r < R; r++) v += lane + 64 * r < nb ? x[r] : 0.0;
        v = wave_sum(v);
        if (lane == 0) (wid == 1 ? out->gd : wid == 2 ? out->gs : out->sks) = v;
    }
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(&out->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// drop every stored pair (before the coefficients are formed again)
__global__ void kl_forget(LmState *st) { st->count = 0; }

__global__ void kl_state_init(LmState *st, double gamma)
{
    st->count = 0;
    st->head = 0;
    st->pending = 0;
    st->accepted = 0;
    st->rejected = 0;
    st->gamma = gamma;
}

// 3. direction pass: d = -H pg, outward components at a bound zeroed;
// first crossing (min), g.d, d.d; ct: the point P(c + d) of the first trial
template <int M>
__global__ __launch_bounds__(kBlock) void kl_dir(Part P, const double *__restrict__ c,
                                                 const double *__restrict__ g,
                                                 const double *__restrict__ pg,
                                                 const double *__restrict__ S,
                                                 const double *__restrict__ Y, int64_t ld,
                                                 const LmState *__restrict__ st, Box B,
                                                 double *__restrict__ d, double *__restrict__ ct,
                                                 double *partials)
{
    const int count = st->count, head = st->head;
    const double gam = st->gamma;
    bool live[M];
    double sc[M], yc[M];
#pragma unroll
    for (int j = 0; j < M; j++) {
        live[j] = lm_live(j, M, count, head, 0) && count > 0;
        sc[j] = st->sc[j];
        yc[j] = st->yc[j];
    }
    constexpr uint32_t kOps = OPS3(OP_MIN, OP_SUM, OP_SUM);
    double a[3];
    red_init<kOps, 3>(a);
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        // (all loads first, as in the pair pass)
        const double pgi = pg[i], ci = c[i], gi = g[i];
        double sv[M], yv[M];
#pragma unroll
        for (int j = 0; j < M; j++) {
            sv[j] = S[j * ld + i];
            yv[j] = Y[j * ld + i];
        }
        double di = -gam * pgi;
#pragma unroll
        for (int j = 0; j < M; j++)
            if (live[j]) di -= sc[j] * sv[j] + yc[j] * yv[j];
        if ((ci <= B.lo && di < 0.0) || (ci >= B.hi && di > 0.0)) di = 0.0;
        d[i] = di;
        ct[i] = proj_box(ci + di, B);
        if (di < 0.0) a[0] = fmin(a[0], (ci - B.lo) / (-di));
        else if (di > 0.0) a[0] = fmin(a[0], (B.hi - ci) / di);
        a[1] += gi * di;
        a[2] += di * di;
    });
    block_partial<kOps, 3>(a, slot_ptr(partials, SLOT_Q), block_id(P));
}

// 4. trial: gathers c(t) = P(c + t d), writes gn = K c(t) - f; g.s, s.(gn - g), s.s
// with s = c(t) - c.  FIRST (t = 1, every iteration): the direction pass has
// written c(1), so one vector is gathered instead of two and no projection
// runs per entry (166 k rows: 10.0 -> 7.7 us); a backtracking step forms c(t)
// as it gathers.
template <int WMAX, class Cols, bool FIRST>
__global__ __launch_bounds__(kBlock, walk_waves<Cols>()) void kl_trial(Part P, const int *__restrict__ so, Cols cols,
                                                   const double *__restrict__ v,
                                                   const double *__restrict__ c,
                                                   const double *__restrict__ d,
                                                   const double *__restrict__ c1, double t,
                                                   const double *__restrict__ f,
                                                   const double *__restrict__ g,
                                                   double *__restrict__ gn, Box B,
                                                   double *partials)
{
    auto ct = [&](int ub, int l) {
        return FIRST ? (c1 + ub)[l] : proj_box((c + ub)[l] + t * (d + ub)[l], B);
    };
    constexpr uint32_t kOps = OPS3(OP_SUM, OP_SUM, OP_SUM);
    double a[3];
    red_init<kOps, 3>(a);
    walk_rows<WMAX, 5>(P, so, cols, v, AllRows(),
                    [&](int i) { return Three{ct(0, i) - c[i], f[i], g[i]}; }, ct,
                    [&](int i, double kc, Three x) {
                        const double gni = kc - x.b;
                        gn[i] = gni;
                        a[0] += x.c * x.a;
                        a[1] += x.a * (gni - x.c);
                        a[2] += x.a * x.a;
                    });
    block_partial<kOps, 3>(a, slot_ptr(partials, SLOT_HOST), block_id(P));
}

// 5. step: c <- P(c + t d), s -> slot head, g <- g + gscale (gn - g)
// (gscale = 1: the trial's gradient itself)
__global__ __launch_bounds__(kBlock) void kl_step(Part P, double *__restrict__ c,
                                                  const double *__restrict__ d, double t,
                                                  double *__restrict__ g,
                                                  const double *__restrict__ gn, double gscale,
                                                  double *__restrict__ S, int64_t ld,
                                                  LmState *st, Box B)
{
    const int head = st->head;
    for_rows(P, [&](int i, bool act) {
        if (!act) return;
        const double ci = c[i];
        const double cn = proj_box(ci + t * d[i], B);
        S[head * ld + i] = cn - ci;
        c[i] = cn;
        g[i] = gscale == 1.0 ? gn[i] : g[i] + gscale * (gn[i] - g[i]);
    });
    if (blockIdx.x == 0 && threadIdx.x == 0) st->pending = 1;
}

// Pair pass and coefficients; with apply, the pending step (t, gscale) is
// taken inside the pair pass.
template <int M>
void launch_pairs_coef(nn_ctx *ctx, const Part &P, double *c, double *g, Box B, bool apply,
                       double t, double gscale)
{
    LmWork &L = ctx->lm;
    const Part P1 = make_part(P.n, kPairBlocks);
    kl_pairs<M><<<P1.nb, kBlock, 0, ctx->stream>>>(P1, c, g, L.pg, L.S, L.Y, L.cap,
                                                   (const LmState *)L.state, B, L.part,
                                                   apply ? 1 : 0, L.d, t, L.gn, gscale);
    kl_coef<M><<<1, 64 * kCoefWaves, 0, ctx->stream>>>(P1.nb, (LmState *)L.state, L.part, apply ? 1 : 0);
}

template <int M>
void launch_coef(nn_ctx *ctx, const Part &P)
{
    const Part P1 = make_part(P.n, kPairBlocks);
    kl_coef<M><<<1, 64 * kCoefWaves, 0, ctx->stream>>>(P1.nb, (LmState *)ctx->lm.state, ctx->lm.part, 0);
}

template <int M>
void launch_dir(nn_ctx *ctx, const Part &P, const double *c, const double *g, Box B)
{
    LmWork &L = ctx->lm;
    kl_dir<M><<<P.nb, kBlock, 0, ctx->stream>>>(P, c, g, L.pg, L.S, L.Y, L.cap,
                                                (const LmState *)L.state, B, L.d,
                                                ctx->ws.q, ctx->partials);
}

#define NN_LM_DISPATCH(m, fn, ...)                  \
    switch (m) {                                    \
    case 1: fn<1>(__VA_ARGS__); break;              \
    case 2: fn<2>(__VA_ARGS__); break;              \
    case 3: fn<3>(__VA_ARGS__); break;              \
    case 4: fn<4>(__VA_ARGS__); break;              \
    case 5: fn<5>(__VA_ARGS__); break;              \
    case 6: fn<6>(__VA_ARGS__); break;              \
    case 7: fn<7>(__VA_ARGS__); break;              \
    default: fn<8>(__VA_ARGS__); break;             \
    }

nn_status ensure_lm(nn_ctx *ctx, int64_t n, int m)
{
    LmWork &L = ctx->lm;
    if (L.state && L.cap >= n && L.m >= m) return NN_OK;
    lm_release(ctx);
    const int64_t cap = std::max<int64_t>(n, 64);
    hipError_t e = dev_malloc(ctx->al, &L.S, sizeof(double) * cap * m);
    if (e == hipSuccess) e = dev_malloc(ctx->al, &L.Y, sizeof(double) * cap * m);
    if (e == hipSuccess) e = dev_malloc(ctx->al, &L.pg, sizeof(double) * cap);
    if (e == hipSuccess) e = dev_malloc(ctx->al, &L.d, sizeof(double) * cap);
    if (e == hipSuccess) e = dev_malloc(ctx->al, &L.gn, sizeof(double) * cap);
    if (e == hipSuccess) e = dev_malloc(ctx->al, &L.part, sizeof(double) * kLmNV * kMaxBlocks);
    if (e == hipSuccess) e = dev_malloc(ctx->al, &L.state, sizeof(LmState));
    if (e == hipSuccess) e = hipHostMalloc(&L.h_state, sizeof(LmHost), hipHostMallocCoherent);
    if (e != hipSuccess) {
        lm_release(ctx);
        return fail(ctx, NN_EOOM, std::string("BLMVM workspace: ") + hipGetErrorString(e));
    }
    // stale slots are never read as pairs, but keep them finite
    e = hipMemsetAsync(L.S, 0, sizeof(double) * cap * m, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(L.Y, 0, sizeof(double) * cap * m, ctx->stream);
    if (e != hipSuccess) return fail(ctx, NN_EHIP, hipGetErrorString(e));
    L.cap = cap;
    L.m = m;
    return NN_OK;
}

}  // namespace

void lm_release(nn_ctx *ctx)
{
    LmWork &L = ctx->lm;
    double *bufs[] = {L.S, L.Y, L.pg, L.d, L.gn, L.part};
    for (double *b : bufs) dev_free(ctx->al, b);
    dev_free(ctx->al, L.state);
    if (L.h_state) (void)hipHostFree(L.h_state);
    L = LmWork();
}

nn_status blmvm_impl(nn_ctx *ctx, const nn_matrix *A, const double *vals, const double *vals64p,
                     const double *f, const nn_opts *o, double *c, uint8_t *active, nn_stats *st)
{
    const int64_t n = A->n;
    nn_stats S;
    std::memset(&S, 0, sizeof(S));
    Box box;
    box.lo = o->lower;
    box.hi = o->upper;
    NN_HIP_TRY(ctx, hipEventRecord(ctx->ev0, ctx->stream));
    auto finish = [&](nn_status rc) -> nn_status {
        if (active && n > 0) launch_active(ctx, n, c, active, box);
        (void)hipEventRecord(ctx->ev1, ctx->stream);
        hipError_t e = hipEventSynchronize(ctx->ev1);
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, ctx->ev0, ctx->ev1);
        S.seconds = ms * 1e-3;
        prof_collect(ctx);
        if (e != hipSuccess) rc = fail(ctx, NN_EHIP, hipGetErrorString(e));
        S.status = (int32_t)rc;
        if (st) *st = S;
        return rc;
    };
    if (n == 0) return finish(NN_OK);
    const int M = std::min(std::max(o->lmm_vectors, 1), kLmMax);
    nn_status rc = ensure_workspace(ctx, n);
    if (rc != NN_OK) return rc;
    if ((rc = ensure_lm(ctx, n, M)) != NN_OK) return rc;
    Workspace &W = ctx->ws;
    LmWork &L = ctx->lm;
    LmHost &H = *(LmHost *)L.h_state;
    const Part P = make_part(n);
    const double nd = (double)n, nnz = (double)A->nnz;
    const double *vp64 = A->d16p ? vals64p : nullptr;
    const double eb = entry_bytes(A, 8.0, vp64, vp64);   // bytes per nonzero
    const double b_grad = 4.0 * (nd + 1) + eb * nnz + 32.0 * nd;
    const double b_trial = 4.0 * (nd + 1) + eb * nnz + 40.0 * nd;
    static const int kInitOps[4] = {OP_SUM, OP_MAX, OP_SUM, OP_SUM};
    static const int kGradOps[5] = {OP_SUM, OP_SUM, OP_MAX, OP_MIN, OP_SUM};
    static const int kTrialOps[3] = {OP_SUM, OP_SUM, OP_SUM};
    double red[kMaxRed];

    // ---- start point, load statistics, first gradient
    const double c0v = std::min(std::max(o->c0_value, box.lo), box.hi);
    prof_begin(ctx, KC_OTHER, 16.0 * n);
    launch_init(ctx, n, c, f, o->c0_mode == 1 ? 1 : 0, c0v, box);
    prof_end(ctx);
    if ((rc = host_reduce(ctx, n, 4, kInitOps, red)) != NN_OK) return rc;
    S.bytes_moved += 16.0 * n;
    const double normf = std::sqrt(red[0]), fmax = red[1];
    S.norm_f = normf;
    if (red[2] != 0.0 || red[3] != 0.0)
        return finish(fail(ctx, NN_ENONFINITE, "non-finite value in f or the initial c"));
    if (box.lo == 0.0 && !(fmax > 0.0)) {
        NN_HIP_TRY(ctx, hipMemsetAsync(c, 0, sizeof(double) * n, ctx->stream));
        S.n_active = (int32_t)n;
        return finish(NN_OK);
    }
    // gradient pass with the KKT report; true when the point is converged
    auto refresh = [&](bool &conv) -> nn_status {
        prof_begin(ctx, KC_GRAD, b_grad);
        launch_grad(ctx, A, vals, vp64, c, f, W.g, box);
        prof_end(ctx);
        S.spmvs++;
        S.bytes_moved += b_grad;
        nn_status r2 = host_reduce(ctx, n, 5, kGradOps, red);
        if (r2 != NN_OK) return r2;
        if (red[1] != 0.0) return fail(ctx, NN_ENONFINITE, "non-finite gradient");
        S.kkt_rel = std::sqrt(red[0]) / normf;
        S.kkt_nat_inf = red[2];
        S.min_c = red[3];
        S.n_active = (int32_t)red[4];
        conv = S.kkt_rel <= o->tol;
        return NN_OK;
    };
    bool conv = false;
    if ((rc = refresh(conv)) != NN_OK) return finish(rc);
    if (conv) return finish(NN_OK);
    kl_state_init<<<1, 1, 0, ctx->stream>>>((LmState *)L.state, 1.0);
    std::memset(L.h_state, 0, sizeof(LmHost));

    const double vp = 8.0 * n;   // bytes of one vector pass
    // Trial at step t along d: gathers P(c + t d), writes K c(t) - f; the
    // partials (g.s, s.(gn - g), s.s) stay in the host slot.
    auto launch_trial_t = [&](double t, bool after_dir) {
        prof_begin(ctx, KC_TRIAL, b_trial);
        auto go = [&](auto first, auto cols, const double *v) {
            NN_DISPATCH_W(A->wmax, (kl_trial<WM, decltype(cols), decltype(first)::value>), P.nb, P,
                          A->sl_off, cols, v, c, L.d, W.q, t, f, W.g, L.gn, box, ctx->partials);
        };
        auto pick = [&](auto first) {
            if (vp64 && A->diag_plan) go(first, diag_cols(A, A->d16p), vp64);
            else if (vp64) go(first, ColsD16P{A->d16p}, vp64);
            else go(first, ColsI32{A->sl_col}, vals);
        };
        if (after_dir) pick(std::true_type());
        else pick(std::false_type());
        prof_end(ctx);
        S.spmvs++;
        S.search_trials++;
        S.bytes_moved += b_trial;
    };
    auto read_trial = [&](double &gs, double &sks) -> nn_status {
        nn_status r2 = host_reduce(ctx, n, 3, kTrialOps, red);
        gs = red[0];
        sks = red[1];
        return r2;
    };
    // Direction pass (partials in SLOT_Q) and, without waiting for it, the
    // first trial t = 1 (both line searches start there); one synchronisation
    // returns the state, the direction summary and the trial.
    double bmin = INFINITY, gd = 0.0, gs1 = 0.0, sks1 = 0.0;
    unsigned long long n_summary = 0;
    auto direction_and_first_trial = [&]() -> nn_status {
        const double live = std::min(H.count + 1, M);
        prof_begin(ctx, KC_OTHER, vp * (4.0 + 2.0 * live));
        NN_LM_DISPATCH(M, launch_dir, ctx, P, c, W.g, box);
        prof_end(ctx);
        launch_trial_t(1.0, true);
        kl_summary<<<1, 256, 0, ctx->stream>>>(P.nb, (const LmState *)L.state, ctx->partials, &H, ++n_summary);
        NN_HIP_TRY(ctx, hipGetLastError());
        const nn_status r2 = flow_wait(
            ctx, [&] { return __atomic_load_n(&H.seq, __ATOMIC_ACQUIRE) == n_summary; });
        if (r2 != NN_OK) return r2;
        bmin = H.bmin;
        gd = H.gd;
        gs1 = H.gs;
        sks1 = H.sks;
        return NN_OK;
    };
    bool fresh = true;
    int since_fresh = 0;
    // the step of an iteration is taken by the next pair pass unless a
    // gradient refresh comes in between
    bool step_pending = false;
    double step_t = 0.0, step_gscale = 1.0;
    nn_status result = NN_EMAXIT;
    for (int it = 0;; it++) {
        // ---- 1-3. (pending step,) pairs, coefficients, direction (+ first trial)
        const double live = std::min(it, M);
        const double b_pairs = vp * (5.0 + 2.0 * live) + (step_pending ? vp * 3.0 : 0.0);
        prof_begin(ctx, KC_OTHER, b_pairs);
        NN_LM_DISPATCH(M, launch_pairs_coef, ctx, P, c, W.g, box, step_pending, step_t,
                       step_gscale);
        prof_end(ctx);
        S.bytes_moved += b_pairs + vp * (4.0 + 2.0 * live);
        step_pending = false;
        if ((rc = direction_and_first_trial()) != NN_OK) return finish(rc);
        if (H.nonfinite != 0.0) return finish(fail(ctx, NN_ENONFINITE, "non-finite iterate"));
        S.outer_its = it;
        const double rel = std::sqrt(H.pg2) / normf;
        if (rel <= o->tol) {
            if (fresh) {
                S.kkt_rel = rel;
                result = NN_OK;
                break;
            }
            if ((rc = refresh(conv)) != NN_OK) return finish(rc);
            fresh = true;
            since_fresh = 0;
            if (conv) {
                result = NN_OK;
                break;
            }
            continue;   // pairs and direction again from the fresh gradient
        }
        if (it >= o->max_lm_its) {
            fail(ctx, NN_EMAXIT, "BLMVM iteration cap reached");
            break;
        }
        if (!(gd < 0.0)) {
            // not a descent direction: forget the pairs, d = -gamma pg
            kl_forget<<<1, 1, 0, ctx->stream>>>((LmState *)L.state);
            NN_LM_DISPATCH(M, launch_coef, ctx, P);
            S.bytes_moved += vp * 4.0;
            S.refinements++;   // memory resets
            if ((rc = direction_and_first_trial()) != NN_OK) return finish(rc);
            if (!(gd < 0.0)) {
                fail(ctx, NN_EMAXIT, "no descent direction above the tolerance (rounding floor)");
                break;
            }
        }
        // ---- 4. line search (the trial at t = 1 is in gs1, sks1)
        double t, gscale, gs = gs1, sks = sks1;
        if (bmin >= 1.0) {
            if (!(sks > 0.0))
                return finish(fail(ctx, NN_ENOTSPD, "non-positive curvature along the direction"));
            t = std::min(-gs / sks, bmin);
            gscale = t;
        } else {
            t = 1.0;
            gscale = 1.0;
            for (int k = 0;; k++) {
                if (gs < 0.0 && gs + 0.5 * sks <= kLmMu * gs) break;
                t *= 0.5;
                if (t <= bmin || k + 1 >= kLmMaxTrials) {
                    // exact step on the segment before the first crossing
                    t = bmin;
                    launch_trial_t(t, false);
                    if ((rc = read_trial(gs, sks)) != NN_OK) return finish(rc);
                    if (!(sks > 0.0))
                        return finish(fail(ctx, NN_ENOTSPD, "non-positive curvature along the direction"));
                    gscale = std::min(-gs / sks, 1.0);
                    t *= gscale;
                    break;
                }
                launch_trial_t(t, false);
                if ((rc = read_trial(gs, sks)) != NN_OK) return finish(rc);
            }
        }
        // ---- 5. step: taken by the next pair pass, or here before a refresh
        fresh = gscale == 1.0;
        since_fresh = fresh ? 0 : since_fresh + 1;
        if (since_fresh >= kLmRefresh) {
            prof_begin(ctx, KC_OTHER, 56.0 * n);
            kl_step<<<P.nb, kBlock, 0, ctx->stream>>>(P, c, L.d, t, W.g, L.gn, gscale, L.S,
                                                      L.cap, (LmState *)L.state, box);
            prof_end(ctx);
            S.bytes_moved += 56.0 * n;
            if ((rc = refresh(conv)) != NN_OK) return finish(rc);
            fresh = true;
            since_fresh = 0;
        } else {
            step_pending = true;
            step_t = t;
            step_gscale = gscale;
        }
        if (o->verbose)
            std::fprintf(stderr, "nnqp blmvm %5d |pg|/|f| %.3e pairs %d gamma %.3g crossing %.3g step %.3g\n",
                         it, rel, H.count, H.gamma, bmin, t);
    }
    // final report from a fresh gradient
    if ((rc = refresh(conv)) != NN_OK) return finish(rc);
    if (result == NN_OK && !conv) result = NN_EMAXIT;
    if (result == NN_OK) ctx->err.clear();
    return finish(result);
}

}  // namespace nnqp
