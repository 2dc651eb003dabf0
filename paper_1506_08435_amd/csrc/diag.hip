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
#include <memory>
#include <new>
#include <vector>

#include "diag.hpp"

namespace nnqp {

namespace {

// Distinct offsets of each slice, ascending, at most kDiagMax: one wavefront
// per slice.  Each lane holds a cursor in its row (columns ascend), the next
// offset is the least of the lanes' current ones.  width[s] = 0: too many.
__global__ __launch_bounds__(256) void kd_offsets(Part P, const int *__restrict__ so,
                                                  const int *__restrict__ sc,
                                                  const int *__restrict__ rp,
                                                  int *__restrict__ list, int *__restrict__ width)
{
    const int lane = threadIdx.x & 63;
    const int s = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (s >= P.nslices()) return;
    const int row = s * kSlice + lane, off = so[s];
    const int len = row < P.n ? rp[row + 1] - rp[row] : 0;
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
        if (lane == 0) list[(size_t)s * kDiagMax + w] = m;
        w++;
        if (d == m) {
            cur++;
            d = cur < len ? sc[off + cur * kSlice + lane] - row : kNone;
        }
    }
    if (lane == 0) width[s] = w;
}

// start[s] = 1 where the offsets of slice s differ from those of slice s - 1
__global__ __launch_bounds__(256) void kd_starts(int nslices, const int *__restrict__ list,
                                                 const int *__restrict__ width,
                                                 int *__restrict__ start)
{
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= nslices) return;
    int same = s > 0 && width[s] == width[s - 1];
    for (int k = 0; same && k < width[s]; k++)
        same = list[(size_t)s * kDiagMax + k] == list[(size_t)(s - 1) * kDiagMax + k];
    // a slice with too many offsets is told to the host as -1
    start[s] = width[s] == 0 ? -1 : (same ? 0 : 1);
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

// *differ = 1 where an entry (i, i - d) that would be read through the
// opposite triangle has other bits than (i - d, i), or only one of the two is
// there.  m: capacity values or null.
__global__ __launch_bounds__(256) void kd_symmetric(Part P, const int *__restrict__ so,
                                                    const int *__restrict__ sc,
                                                    const int *__restrict__ rp,
                                                    const int *__restrict__ srun,
                                                    const DiagRun *__restrict__ runs,
                                                    const int *__restrict__ mirrored,
                                                    const double *__restrict__ v,
                                                    const double *__restrict__ m,
                                                    int *__restrict__ differ)
{
    const int lane = threadIdx.x & 63;
    const int nw = gridDim.x * 4;
    auto bits = [](double x) { return __double_as_longlong(x); };
    int bad = 0;
    for (int s = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)); s < P.nslices();
         s += nw) {
        if (mirrored[srun[s]] == 0) continue;
        const DiagRun &r = runs[srun[s]];
        const int row = s * kSlice + lane, off = so[s];
        if (row >= P.n) continue;
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
    if (bad) *differ = 1;
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

static nn_status upload(nn_ctx *ctx, const DiagPlan &D, void *index)
{
    char *p = (char *)index;
    const size_t a = sizeof(int) * D.srun.size(), b = sizeof(DiagRun) * D.runs.size(),
                 c = sizeof(int) * D.mirrored.size();
    NN_HIP_TRY(ctx, hipMemcpyAsync(p, D.srun.data(), a, hipMemcpyHostToDevice, ctx->stream));
    NN_HIP_TRY(ctx, hipMemcpyAsync(p + a, D.runs.data(), b, hipMemcpyHostToDevice, ctx->stream));
    NN_HIP_TRY(ctx, hipMemcpyAsync(p + a + b, D.mirrored.data(), c, hipMemcpyHostToDevice, ctx->stream));
    return NN_OK;
}

nn_status diag_upload(nn_ctx *ctx, const nn_matrix *A, void *index)
{
    return upload(ctx, *A->diag_plan, index);
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

nn_status diag_find(nn_ctx *ctx, nn_matrix *A, void *scratch)
{
    if (A->diag_tried) return NN_OK;
    const int64_t ns = A->nslices;
    // the scratch is an index copy to be (2 bytes per entry): 256 bytes per
    // slice from two entries per row on, of which the lists take 136 and an
    // eighth of them again 17
    if (A->nsell < 2 * ns * kSlice || A->wmax > kDiagMax) {
        A->diag_tried = true;
        return NN_OK;
    }
    int *list = (int *)scratch, *width = list + (size_t)ns * kDiagMax, *start = width + ns;
    static_assert(2 * 2 * kSlice >= 4 * (kDiagMax + 2) + (4 * kDiagMax + 4) / 8,
                  "the lists fit in the index copy");
    const Part P = make_part(A->n);
    kd_offsets<<<(unsigned)((ns + 3) / 4), 256, 0, ctx->stream>>>(P, A->sl_off, A->sl_col, A->rowptr,
                                                                  list, width);
    kd_starts<<<(unsigned)((ns + 255) / 256), 256, 0, ctx->stream>>>((int)ns, list, width, start);
    NN_HIP_TRY(ctx, hipGetLastError());
    try {
        std::vector<int> h(2 * (size_t)ns);
        NN_HIP_TRY(ctx, hipMemcpyAsync(h.data(), width, sizeof(int) * 2 * ns, hipMemcpyDeviceToHost,
                                       ctx->stream));
        NN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        // segments: consecutive slices with the same offsets
        std::vector<int> first;
        for (int64_t s = 0; s < ns; s++) {
            if (h[ns + s] < 0) {   // a slice with too many offsets
                A->diag_tried = true;
                return NN_OK;
            }
            if (h[ns + s] > 0) first.push_back((int)s);
        }
        // their lists: gathered behind the slices' own when they are few
        const size_t m = first.size();
        std::vector<int> lists;
        const bool some = 8 * m <= (size_t)ns;
        lists.resize((some ? m : (size_t)ns) * kDiagMax);
        if (some) {
            int *at = start + ns, *packed = at + m;
            NN_HIP_TRY(ctx, hipMemcpyAsync(at, first.data(), sizeof(int) * m, hipMemcpyHostToDevice,
                                           ctx->stream));
            kd_pack<<<(unsigned)m, 64, 0, ctx->stream>>>(at, list, packed);
            NN_HIP_TRY(ctx, hipGetLastError());
            NN_HIP_TRY(ctx, hipMemcpyAsync(lists.data(), packed, sizeof(int) * lists.size(),
                                           hipMemcpyDeviceToHost, ctx->stream));
        } else {
            NN_HIP_TRY(ctx, hipMemcpyAsync(lists.data(), list, sizeof(int) * lists.size(),
                                           hipMemcpyDeviceToHost, ctx->stream));
        }
        NN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        std::unique_ptr<DiagPlan> D(new DiagPlan());
        bool fits = diag_plan(A->n, ns, A->nsell, A->wmax, first, h.data(), lists.data(), some, D.get());
        if (fits) {
            // the flag goes through the reduction partials, free between passes
            int *flag = reinterpret_cast<int *>(ctx->partials), differ = 0;
            nn_status rc = upload(ctx, *D, scratch);
            if (rc != NN_OK) return rc;
            const int *srun = (const int *)scratch;
            const DiagRun *runs = (const DiagRun *)(srun + D->srun.size());
            NN_HIP_TRY(ctx, hipMemsetAsync(flag, 0, sizeof(int), ctx->stream));
            kd_symmetric<<<std::max(1, std::min((P.nslices() + 3) / 4, 4096)), 256, 0, ctx->stream>>>(
                P, A->sl_off, A->sl_col, A->rowptr, srun, runs, (const int *)(runs + D->runs.size()),
                A->val, A->mval, flag);
            NN_HIP_TRY(ctx, hipGetLastError());
            NN_HIP_TRY(ctx, hipMemcpyAsync(&differ, flag, sizeof(int), hipMemcpyDeviceToHost,
                                           ctx->stream));
            NN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
            fits = differ == 0;
        }
        if (fits) A->diag_plan = D.release();
    } catch (const std::bad_alloc &) {
        return fail(ctx, NN_EOOM, "host allocation");
    }
    A->diag_tried = true;
    return NN_OK;
}

}  // namespace nnqp
