// Diagonal layout of a sliced-ELL matrix (diag.hpp): which patterns have it,
// where its arrays lie, and the kernels that fill them.
//
// The offsets (column - row) a slice's rows use are collected on the device;
// consecutive slices with the same offsets form a run.  A run stores one
// array per offset >= 0 over all its rows.  The entry (i, i - d) is read as
// entry (i - d, i) where row i - d lies in the run (for a run that starts at
// row 0 zeros in front of the arrays stand for the rows before it); the first
// slices of a later run store their offsets < 0 themselves.  The arrays take
// the place of the matrix's paired or quad copies, so the layout is used
// where they fit in as many entries as the sliced-ELL arrays hold, where three
// quarters of the slices are regular (the unrolled stencil widths), and where
// K and M have the same bits on both sides of the diagonal; other patterns
// (unstructured numberings) keep the other layouts.
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "diag.hpp"

namespace nnqp {

namespace {

// The matrices whose patterns are looked over in one launch (blockIdx.y: which
// one): of a single-problem solve its own, of a batch every member's.  Their
// slices are numbered one after the other.
struct DiagJob {
    const int *so, *sc, *rp;
    const double *v, *m;     // values; capacity values or null
    int n, nsl, s0;          // rows, slices (0: nothing to do), first slice
    const int *srun;         // tables of the plan (kd_symmetric)
    const DiagRun *runs;
    const int *mirrored;
};
struct JobsOne {
    DiagJob j;
    __device__ __forceinline__ const DiagJob &operator[](int) const { return j; }
};
struct JobsMany {
    const DiagJob *j;
    __device__ __forceinline__ const DiagJob &operator[](int k) const { return j[k]; }
};

// Distinct offsets of each slice, ascending, at most kDiagMax: one wavefront
// per slice.  Each lane holds a cursor in its row (columns ascend), the next
// offset is the least of the lanes' current ones.  width[s] = 0: too many.
template <class Jobs>
__global__ __launch_bounds__(256) void kd_offsets(Jobs J, int *__restrict__ list,
                                                  int *__restrict__ width)
{
    const DiagJob &A = J[blockIdx.y];
    const int lane = threadIdx.x & 63;
    const int *__restrict__ sc = A.sc, *__restrict__ rp = A.rp;
    const int nw = gridDim.x * 4;
    for (int s = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)); s < A.nsl;
         s += nw) {
        const int row = s * kSlice + lane, off = A.so[s];
        const size_t at = (size_t)A.s0 + s;
        const int len = row < A.n ? rp[row + 1] - rp[row] : 0;
        constexpr int kNone = 0x7fffffff;
        int cur = 0;
        int d = len > 0 ? sc[off + lane] - row : kNone;
        int w = 0;
        for (;;) {
            int m = d;
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) m = min(m, __shfl_xor(m, o, 64));
            if (m == kNone) break;
            if (w == kDiagMax) {
                w = 0;
                break;
            }
            if (lane == 0) list[at * kDiagMax + w] = m;
            w++;
            if (d == m) {
                cur++;
                d = cur < len ? sc[off + cur * kSlice + lane] - row : kNone;
            }
        }
        if (lane == 0) width[at] = w;
    }
}

// start[s] = 1 where the offsets of slice s differ from those of slice s - 1
template <class Jobs>
__global__ __launch_bounds__(256) void kd_starts(Jobs J, const int *__restrict__ list,
                                                 const int *__restrict__ width,
                                                 int *__restrict__ start)
{
    const DiagJob &A = J[blockIdx.y];
    for (int sl = blockIdx.x * 256 + threadIdx.x; sl < A.nsl; sl += gridDim.x * 256) {
        const size_t s = (size_t)A.s0 + sl;
        int same = sl > 0 && width[s] == width[s - 1];
        for (int k = 0; same && k < width[s]; k++)
            same = list[s * kDiagMax + k] == list[(s - 1) * kDiagMax + k];
        // a slice with too many offsets is told to the host as -1
        start[s] = width[s] == 0 ? -1 : (same ? 0 : 1);
    }
}

// lists of the slices at[0], at[1], ... side by side
__global__ __launch_bounds__(64) void kd_pack(const int *__restrict__ at,
                                              const int *__restrict__ list, int *__restrict__ out)
{
    if (threadIdx.x < kDiagMax)
        out[(size_t)blockIdx.x * kDiagMax + threadIdx.x] =
            list[(size_t)at[blockIdx.x] * kDiagMax + threadIdx.x];
}

// The stored diagonals of a value array: entry k of row i at b_k + i, zero
// where the row has no such entry; offsets read through the opposite triangle
// are not stored.
template <class T>
__global__ __launch_bounds__(256) void kd_fill(Part P, const int *__restrict__ so,
                                               const int *__restrict__ sc,
                                               const int *__restrict__ rp, const int *__restrict__ srun,
                                               const DiagRun *__restrict__ runs,
                                               const int *__restrict__ mirrored,
                                               const T *__restrict__ src, T *__restrict__ dst)
{
    const int lane = threadIdx.x & 63;
    const int nw = gridDim.x * 4;
    for (int s = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)); s < P.nslices();
         s += nw) {
        const int row = s * kSlice + lane, off = so[s];
        const int len = row < P.n ? rp[row + 1] - rp[row] : 0;
        const DiagRun &r = runs[srun[s]];
        const bool mir = mirrored[srun[s]] != 0;
        int cur = 0;
        int d = len > 0 ? sc[off + lane] - row : 0x7fffffff;
        for (int k = 0; k < r.w; k++) {
            T v = T(0);
            if (d == r.d[k]) {
                v = src[off + cur * kSlice + lane];
                cur++;
                d = cur < len ? sc[off + cur * kSlice + lane] - row : 0x7fffffff;
            }
            if (!(mir && r.d[k] < 0)) dst[(ptrdiff_t)r.b[k] + row] = v;
        }
    }
}

// differ[blockIdx.y] = 1 where an entry (i, i - d) that would be read through
// the opposite triangle has other bits than (i - d, i), or only one of the two
// is there, in K or in M.
template <class Jobs>
__global__ __launch_bounds__(256) void kd_symmetric(Jobs J, int *__restrict__ differ)
{
    const DiagJob &A = J[blockIdx.y];
    const int *__restrict__ so = A.so, *__restrict__ sc = A.sc, *__restrict__ rp = A.rp;
    const double *__restrict__ v = A.v, *__restrict__ m = A.m;
    const int lane = threadIdx.x & 63;
    const int nw = gridDim.x * 4;
    auto bits = [](double x) { return __double_as_longlong(x); };
    int bad = 0;
    for (int s = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)); s < A.nsl;
         s += nw) {
        if (A.mirrored[A.srun[s]] == 0) continue;
        const DiagRun &r = A.runs[A.srun[s]];
        const int row = s * kSlice + lane, off = so[s];
        if (row >= A.n) continue;
        const int len = rp[row + 1] - rp[row];
        int cur = 0;
        for (int k = 0; k < r.w && r.d[k] < 0; k++) {
            const bool has = cur < len && sc[off + cur * kSlice + lane] - row == r.d[k];
            // row j = row + d lies in the run, or before row 0 (no entry)
            const int j = row + r.d[k];
            if (j < 0) continue;
            const int lj = j % kSlice, oj = so[j / kSlice];
            const int len_j = rp[j + 1] - rp[j];
            int e = -1;
            for (int q = 0; q < len_j && e < 0; q++)
                if (sc[oj + q * kSlice + lj] == row) e = oj + q * kSlice + lj;
            if (has != (e >= 0)) {
                bad = 1;
            } else if (has) {
                const int o = off + cur * kSlice + lane;
                if (bits(v[o]) != bits(v[e]) || (m && bits(m[o]) != bits(m[e]))) bad = 1;
            }
            if (has) cur++;
        }
    }
    if (bad) differ[blockIdx.y] = 1;
}

template <class T>
nn_status fill(nn_ctx *ctx, const nn_matrix *A, const void *index, const T *src, T *dst)
{
    const DiagPlan &D = *A->diag_plan;
    const Part P = make_part(A->n);
    const int *srun = (const int *)index;
    const DiagRun *runs = (const DiagRun *)(srun + D.srun.size());
    const int *mir = (const int *)(runs + D.runs.size());
    const int nb = std::max(1, std::min((P.nslices() + 3) / 4, 4096));
    // zeros: the rows before a run from row 0 on (the kernel writes the rest)
    if (D.runs[D.srun[0]].kind != DR_GENERAL || D.mirrored[D.srun[0]])
        NN_HIP_TRY(ctx, hipMemsetAsync(dst, 0, sizeof(T) * (size_t)D.entries, ctx->stream));
    kd_fill<T><<<nb, 256, 0, ctx->stream>>>(P, A->sl_off, A->sl_col, A->rowptr, srun, runs, mir, src,
                                            dst);
    NN_HIP_TRY(ctx, hipGetLastError());
    return NN_OK;
}

}  // namespace

ColsDiag diag_cols(const nn_matrix *A, const void *index)
{
    const DiagPlan &D = *A->diag_plan;
    ColsDiag c;
    c.srun = (const int *)index;
    c.runs = (const DiagRun *)(c.srun + D.srun.size());
    c.lo = D.lo;
    c.hi = D.hi;
    c.elo = D.elo;
    c.ehi = D.ehi;
    c.reg = D.main;
    return c;
}

// The tables of a plan as they lie in an index copy: run of each slice, runs,
// which runs read the opposite triangle.
static size_t table_bytes(const DiagPlan &D)
{
    return sizeof(int) * D.srun.size() + (sizeof(DiagRun) + sizeof(int)) * D.runs.size();
}
static void put_tables(const DiagPlan &D, char *p)
{
    const size_t a = sizeof(int) * D.srun.size(), b = sizeof(DiagRun) * D.runs.size();
    std::memcpy(p, D.srun.data(), a);
    std::memcpy(p + a, D.runs.data(), b);
    std::memcpy(p + a + b, D.mirrored.data(), sizeof(int) * D.mirrored.size());
}

nn_status diag_upload(nn_ctx *ctx, const nn_matrix *A, void *index)
{
    const DiagPlan &D = *A->diag_plan;
    char *p = (char *)index;
    const size_t a = sizeof(int) * D.srun.size(), b = sizeof(DiagRun) * D.runs.size(),
                 c = sizeof(int) * D.mirrored.size();
    NN_HIP_TRY(ctx, hipMemcpyAsync(p, D.srun.data(), a, hipMemcpyHostToDevice, ctx->stream));
    NN_HIP_TRY(ctx, hipMemcpyAsync(p + a, D.runs.data(), b, hipMemcpyHostToDevice, ctx->stream));
    NN_HIP_TRY(ctx, hipMemcpyAsync(p + a + b, D.mirrored.data(), c, hipMemcpyHostToDevice, ctx->stream));
    return NN_OK;
}

bool diag_one_run(const nn_matrix *A, DiagReg *reg)
{
    if (!A->diag_plan || A->diag_plan->elo != 0 || A->diag_plan->ehi != (int)A->nslices) return false;
    *reg = A->diag_plan->main;
    return true;
}

double diag_entries(const nn_matrix *A) { return A->diag_plan ? (double)A->diag_plan->entries : 0.0; }

nn_status diag_fill(nn_ctx *ctx, const nn_matrix *A, const void *index, const double *src,
                    double *dst)
{
    return fill(ctx, A, index, src, dst);
}

nn_status diag_fill(nn_ctx *ctx, const nn_matrix *A, const void *index, const float *src, float *dst)
{
    return fill(ctx, A, index, src, dst);
}

void diag_free(nn_matrix *A)
{
    delete A->diag_plan;
    A->diag_plan = nullptr;
}

// Looks P patterns over in four launches and three waits, whatever their number.
// send(job, J): the jobs to where the kernels take them from (J); scratch: two
// bytes per stored entry of all of them.
template <class Jobs, class Send>
static nn_status find(nn_ctx *ctx, nn_matrix *const *A, int P, char *scratch, Send send)
{
    hipStream_t st = ctx->stream;
    Jobs J;
    // 256 bytes per slice from two entries per row on, of which the lists take
    // 136 and an eighth of them again 17
    static_assert(2 * 2 * kSlice >= 4 * (kDiagMax + 2) + (4 * kDiagMax + 4) / 8,
                  "the lists fit in the index copy");
    std::vector<DiagJob> job((size_t)P);
    int64_t S = 0;
    int most = 0;   // slices
    for (int p = 0; p < P; p++) {
        const nn_matrix &K = *A[p];
        const bool look = K.nsell >= 2 * K.nslices * kSlice && K.wmax <= kDiagMax;
        job[p] = DiagJob{K.sl_off, K.sl_col, K.rowptr, K.val, K.mval, (int)K.n, look ? (int)K.nslices : 0,
                         (int)S, nullptr, nullptr, nullptr};
        S += job[p].nsl;
        most = std::max(most, job[p].nsl);
    }
    std::vector<std::unique_ptr<DiagPlan>> plan((size_t)P);
    if (S > 0) {
        int *list = (int *)scratch, *width = list + (size_t)S * kDiagMax, *start = width + S;
        NN_HIP_TRY(ctx, send(job, J));
        // (a slice per wavefront; many matrices share 65,536 blocks)
        const int gx = std::min((most + 3) / 4, std::max(64, 65536 / P));
        kd_offsets<<<dim3(P > 1 ? gx : (most + 3) / 4, P), 256, 0, st>>>(J, list, width);
        kd_starts<<<dim3((most + 255) / 256, P), 256, 0, st>>>(J, list, width, start);
        NN_HIP_TRY(ctx, hipGetLastError());
        std::vector<int> h(2 * (size_t)S);
        NN_HIP_TRY(ctx, hipMemcpyAsync(h.data(), width, sizeof(int) * 2 * S, hipMemcpyDeviceToHost, st));
        NN_HIP_TRY(ctx, hipStreamSynchronize(st));
        // segments: consecutive slices with the same offsets
        std::vector<int> at;                       // their first slices, of all matrices
        std::vector<size_t> seg((size_t)P + 1, 0);
        for (int p = 0; p < P; p++) {
            seg[p] = at.size();
            const int s0 = job[p].s0;
            for (int s = s0; s < s0 + job[p].nsl; s++) {
                if (h[S + s] < 0) {   // a slice with too many offsets
                    job[p].nsl = 0;
                    at.resize(seg[p]);
                    break;
                }
                if (h[S + s] > 0) at.push_back(s);
            }
        }
        seg[P] = at.size();
        // their lists: gathered behind the slices' own when they are few
        const size_t m = at.size();
        const bool some = 8 * m <= (size_t)S;
        std::vector<int> lists((some ? m : (size_t)S) * kDiagMax);
        if (m > 0) {
            const int *src = list;
            if (some) {
                int *d_at = start + S, *packed = d_at + m;
                NN_HIP_TRY(ctx, hipMemcpyAsync(d_at, at.data(), sizeof(int) * m, hipMemcpyHostToDevice, st));
                kd_pack<<<(unsigned)m, 64, 0, st>>>(d_at, list, packed);
                NN_HIP_TRY(ctx, hipGetLastError());
                src = packed;
            }
            NN_HIP_TRY(ctx, hipMemcpyAsync(lists.data(), src, sizeof(int) * lists.size(),
                                           hipMemcpyDeviceToHost, st));
            NN_HIP_TRY(ctx, hipStreamSynchronize(st));
        }
        std::vector<char> tables;
        std::vector<size_t> where((size_t)P, 0);
        bool any = false;
        for (int p = 0; p < P; p++) {
            DiagJob &j = job[p];
            if (j.nsl == 0) continue;
            std::vector<int> first(at.begin() + seg[p], at.begin() + seg[p + 1]);
            for (int &s : first) s -= j.s0;
            std::unique_ptr<DiagPlan> D(new DiagPlan());
            if (!diag_plan(A[p]->n, A[p]->nslices, A[p]->nsell, A[p]->wmax, first, h.data() + j.s0,
                           lists.data() + (some ? seg[p] : (size_t)j.s0) * kDiagMax, some, D.get())) {
                j.nsl = 0;
                continue;
            }
            where[p] = tables.size();
            tables.resize(tables.size() + table_bytes(*D));
            put_tables(*D, tables.data() + where[p]);
            plan[p] = std::move(D);
            any = true;
        }
        if (any) {
            for (int p = 0; p < P; p++) {
                if (!plan[p]) continue;
                char *t = scratch + where[p];
                job[p].srun = (const int *)t;
                job[p].runs = (const DiagRun *)(t + sizeof(int) * plan[p]->srun.size());
                job[p].mirrored = (const int *)(job[p].runs + plan[p]->runs.size());
            }
            // the flags go through the reduction partials, free between passes
            int *flag = reinterpret_cast<int *>(ctx->partials);
            std::vector<int> differ((size_t)P, 0);
            NN_HIP_TRY(ctx, hipMemcpyAsync(scratch, tables.data(), tables.size(), hipMemcpyHostToDevice, st));
            NN_HIP_TRY(ctx, hipMemsetAsync(flag, 0, sizeof(int) * P, st));
            NN_HIP_TRY(ctx, send(job, J));
            kd_symmetric<<<dim3(std::min(gx, 4096), P), 256, 0, st>>>(J, flag);
            NN_HIP_TRY(ctx, hipGetLastError());
            NN_HIP_TRY(ctx, hipMemcpyAsync(differ.data(), flag, sizeof(int) * P, hipMemcpyDeviceToHost, st));
            NN_HIP_TRY(ctx, hipStreamSynchronize(st));
            for (int p = 0; p < P; p++)
                if (differ[p]) plan[p].reset();
        }
    }
    for (int p = 0; p < P; p++) {
        A[p]->diag_plan = plan[p].release();
        A[p]->diag_tried = true;
    }
    return NN_OK;
}

nn_status diag_find(nn_ctx *ctx, nn_matrix *A, void *scratch)
{
    if (A->diag_tried) return NN_OK;
    try {
        return find<JobsOne>(ctx, &A, 1, (char *)scratch, [](const std::vector<DiagJob> &job, JobsOne &J) {
            J.j = job[0];
            return hipSuccess;
        });
    } catch (const std::bad_alloc &) {
        return fail(ctx, NN_EOOM, "host allocation");
    }
}

size_t diag_find_bytes(nn_matrix *const *A, int P)
{
    size_t b = 0;
    for (int p = 0; p < P; p++) b += sizeof(short) * (size_t)A[p]->nsell;
    return (b + 15) / 16 * 16 + sizeof(DiagJob) * (size_t)P;
}

nn_status diag_find_many(nn_ctx *ctx, nn_matrix *const *A, int P, void *scratch)
{
    static_assert(sizeof(double) * kSlots * kMaxBlocks * kMaxRed >= sizeof(int) * kDiagJobs, "flags");
    nn_status rc = NN_OK;
    try {
        for (int p = 0; p < P && rc == NN_OK; p += kDiagJobs) {
            const int m = std::min(P - p, kDiagJobs);
            DiagJob *d = (DiagJob *)((char *)scratch + diag_find_bytes(A, P) - sizeof(DiagJob) * (size_t)P);
            std::vector<DiagJob> kept;   // (the copy's source; find waits before it sends again)
            rc = find<JobsMany>(ctx, A + p, m, (char *)scratch,
                                [&](const std::vector<DiagJob> &job, JobsMany &J) {
                kept = job;
                J.j = d;
                return hipMemcpyAsync(d, kept.data(), sizeof(DiagJob) * (size_t)m, hipMemcpyHostToDevice,
                                      ctx->stream);
            });
        }
    } catch (const std::bad_alloc &) {
        rc = fail(ctx, NN_EOOM, "host allocation");
    }
    return rc;
}

}  // namespace nnqp
