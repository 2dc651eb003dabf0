// Diagonal layout of a sliced matrix, and the row walks that read it.
//
// On a mesh whose nodes are numbered along grid lines the 64 rows of a slice
// share a handful of column offsets (the 7 or 15 of a P1 stencil; a row next
// to a Dirichlet boundary lacks some of them).  The layout keeps, per run of
// consecutive slices with the same offsets, one array of values per offset,
// so entry k of row i is val[b_k + i] in column i + d_k with b_k and d_k
// uniform over the wavefront: no column index is read per entry, and the
// addresses of all loads are scalar.  K is symmetric, so inside a run the
// entry (i, i - d) is not stored again: it is read as entry (i - d, i), in the
// array of the offset +d.  A 15-point row then takes 64 B of values from
// memory instead of 150 B of values and int16 offsets; the other seven values
// come from the caches (row i - d is at most a grid plane back).  Solves of
// 127^3, 100^3 (mixed) and 80^3 (Galerkin) rows: 209 -> 149, 51.6 -> 37.2 and
// 20.0 -> 12.3 ms against the paired and quad copies (Galerkin: int32 columns).
//
// Entries a row does not have are stored as zeros and added as 0 * x: with
// finite x the sum is bitwise the one of the general walk (the columns are
// in ascending order in both).  What is read through this layout are the
// solvers' passes, whose reductions end a solve at the first non-finite value.
#pragma once

#include "rows.hpp"

namespace nnqp {

// Unrolled entries of a walk: the offsets of a regular row.
template <int WMAX>
constexpr int diag_width() { return diag_regular(WMAX); }

// The layout as Cols of walk_rows.  Slices [elo, ehi) are the main run, whose
// offsets and bases are kernel arguments (no lookup); [lo, hi) are its slices
// with every column inside [0, n).
struct ColsDiag {
    const int *srun;
    const DiagRun *runs;
    int lo, hi, elo, ehi;
    DiagReg reg;
};

// A slice's kind and, when it is regular, its offsets and bases, in scalar
// registers.
template <int W>
struct DiagTab {
    int kind, b0, stride;
    int h[W / 2];
};

template <int W>
__device__ __forceinline__ DiagTab<W> diag_tab(const ColsDiag &D, int s)
{
    DiagTab<W> t;
    if (s >= D.elo && s < D.ehi) {
        t.kind = s >= D.lo && s < D.hi ? DR_REGULAR : DR_EDGE;
        t.b0 = D.reg.b0;
        t.stride = D.reg.stride;
#pragma unroll
        for (int u = 0; u < W / 2; u++) t.h[u] = D.reg.h[u];
    } else {
        const DiagRun &r = D.runs[D.srun[s]];
        t.kind = r.kind;
        t.b0 = r.reg.b0;
        t.stride = r.reg.stride;
#pragma unroll
        for (int u = 0; u < W / 2; u++) t.h[u] = r.reg.h[u];
    }
    return t;
}

// Entry k of a regular row (ascending columns): where its value and its
// column are for the slice's first row.
template <int W>
__device__ __forceinline__ void diag_entry(const DiagTab<W> &t, int k, int &d, int &b)
{
    constexpr int H = W / 2;
    const int u = k < H ? H - 1 - k : k - H - 1;   // index into h (k != H)
    d = k == H ? 0 : (k < H ? -t.h[u] : t.h[u]);
    b = t.b0 + (k == H ? 0 : (u + 1) * t.stride) + (k < H ? d : 0);
}

// The general walk of a slice: any offsets, columns held inside [0, n) (an
// offset that leaves it for some row is a zero entry there).
template <int NT, class XT, class VT, class X>
__device__ __forceinline__ void diag_row_gen(const ColsDiag &D, const VT *__restrict__ v, int n,
                                             int s, X x, double (&acc)[NT])
{
    const int lane = threadIdx.x & 63, row0 = s * kSlice;
    const DiagRun &r = D.runs[D.srun[s]];
    const int w = r.w;
    constexpr int PH = 4;
#pragma nounroll
    for (int h = 0; h < w; h += PH) {
        VT vv[PH];
        XT xv[PH][NT];
#pragma unroll
        for (int k = 0; k < PH; k++) {
            vv[k] = (v + ((ptrdiff_t)r.b[h + k] + row0))[lane];
            x(0, min(max(row0 + lane + r.d[h + k], 0), n - 1), xv[k]);
        }
#pragma unroll
        for (int k = 0; k < PH; k++)
#pragma unroll
            for (int q = 0; q < NT; q++) {
                const double y = __builtin_fma((double)vv[k], (double)xv[k][q], acc[q]);
                acc[q] = h + k < w ? y : acc[q];
            }
    }
}

// Row sums of NT products over a regular slice: PH entries per load phase.
// EDGE: columns held inside [0, n).
template <int W, int NT, int PH, bool EDGE, class XT, class VT, class X>
__device__ __forceinline__ void diag_row_reg(const DiagTab<W> &t, const VT *__restrict__ v, int n,
                                             int row0, X x, double (&acc)[NT])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 0; h < W; h += PH) {
        VT vv[PH];
        XT xv[PH][NT];
#pragma unroll
        for (int k = 0; k < PH; k++) {
            if (h + k >= W) continue;
            int d, b;
            diag_entry<W>(t, h + k, d, b);
            vv[k] = (v + (ptrdiff_t)(b + row0))[lane];
            if constexpr (EDGE) x(0, min(max(row0 + d + lane, 0), n - 1), xv[k]);
            else x(row0 + d, lane, xv[k]);
        }
#pragma unroll
        for (int k = 0; k < PH; k++) {
            if (h + k >= W) continue;
#pragma unroll
            for (int q = 0; q < NT; q++)
                acc[q] = __builtin_fma((double)vv[k], (double)xv[k][q], acc[q]);
        }
    }
}

template <int W, int NT, int PH, class XT, class VT, class X>
__device__ __forceinline__ void diag_row(const ColsDiag &D, const VT *__restrict__ v, int n, int s,
                                         X x, double (&acc)[NT])
{
    const DiagTab<W> t = diag_tab<W>(D, s);
    if (t.kind == DR_REGULAR) diag_row_reg<W, NT, PH, false, XT>(t, v, n, s * kSlice, x, acc);
    else if (t.kind == DR_EDGE)
        diag_row_reg<W, NT, (PH < 4 ? PH : 4), true, XT>(t, v, n, s * kSlice, x, acc);
    else diag_row_gen<NT, XT>(D, v, n, s, x, acc);
}

// sell_rows on the diagonal layout, PH entries per load phase.
template <int WMAX, int PH, class VT, class Act, class Pre, class X, class Epi>
__device__ __forceinline__ void diag_rows(const Part &P, const ColsDiag &D,
                                          const VT *__restrict__ v, Act active, Pre pre, X x,
                                          Epi epi)
{
    using PV = decltype(pre(0));
    constexpr int W = diag_width<WMAX>();
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int nw = P.nb * kWaves;
    using XT = decltype(x(0, 0));
    auto x1 = [&](int ub, int l, XT (&out)[1]) { out[0] = x(ub, l); };
    for (int s = block_id(P) * kWaves + wid; s < P.nslices(); s += nw) {
        const int row = s * kSlice + lane;
        const bool act = row < P.n && active(row);
        const PV pv = act ? pre(row) : PV();
        if (__ballot(act) == 0) continue;
        double acc[1] = {0.0};
        diag_row<W, 1, PH, XT>(D, v, P.n, s, x1, acc);
        if (act) epi(row, acc[0], pv);
    }
}

template <int WMAX, int NT, class VT, class Pre, class X, class Epi>
__device__ __forceinline__ void diag_rows_n(const Part &P, const ColsDiag &D,
                                            const VT *__restrict__ v, Pre pre, X x, Epi epi)
{
    using PV = decltype(pre(0));
    constexpr int W = diag_width<WMAX>();
    const int lane = threadIdx.x & 63, wid = wave_id();
    const int nw = P.nb * kWaves;
    for (int s = block_id(P) * kWaves + wid; s < P.nslices(); s += nw) {
        const int row = s * kSlice + lane;
        const bool act = row < P.n;
        const PV pv = act ? pre(row) : PV();
        double acc[NT];
#pragma unroll
        for (int q = 0; q < NT; q++) acc[q] = 0.0;
        diag_row<W, NT, 5, double>(D, v, P.n, s, x, acc);
        if (act) epi(row, acc, pv);
    }
}

// sell_rows and sell_rows_n on any layout.  x(ub, l) is the gathered value of
// row ub + l, ub uniform over the wavefront (the diagonal walk passes the
// column of its first lane, the others 0): the row is addressed as
// (vector + ub)[l], a scalar base and a lane offset.
// PH: entries per load phase of the diagonal walk (what 64 VGPRs hold).
template <int WMAX, int PH = 8, class VT, class Cols, class Act, class Pre, class X, class Epi>
__device__ __forceinline__ void walk_rows(const Part &P, const int *__restrict__ so, const Cols &sc,
                                          const VT *__restrict__ sv, Act active, Pre pre, X x,
                                          Epi epi)
{
    if constexpr (std::is_same<Cols, ColsDiag>::value)
        diag_rows<WMAX, PH>(P, sc, sv, active, pre, x, epi);
    else
        sell_rows<WMAX>(P, so, sc, sv, active, pre, [&](int j) { return x(0, j); }, epi);
}

template <int WMAX, int NT, int PHASE, class VT, class Cols, class Pre, class X, class Epi>
__device__ __forceinline__ void walk_rows_n(const Part &P, const int *__restrict__ so,
                                            const Cols &sc, const VT *__restrict__ sv, Pre pre, X x,
                                            Epi epi)
{
    if constexpr (std::is_same<Cols, ColsDiag>::value) {
        diag_rows_n<WMAX, NT>(P, sc, sv, pre, x, epi);
    } else {
        auto x0 = [&](int j, double (&out)[NT]) { x(0, j, out); };
        sell_rows_n<WMAX, NT, VT, Cols, Pre, decltype(x0), Epi, PHASE>(P, so, sc, sv, pre, x0, epi);
    }
}

// Waves per SIMD a kernel on Cols is compiled for: the walks of the diagonal
// layout issue as many loads ahead as registers allow, so the bound is given
// (eight waves, 64 VGPRs: two blocks per CU; without it the float64 passes
// took 80-104 VGPRs and ran one block per CU).  The other walks keep theirs.
template <class Cols>
constexpr int walk_waves() { return std::is_same<Cols, ColsDiag>::value ? 8 : 4; }

// Host side: the layout of A as a kernel argument, from the index copy
// (d16p or d16q) the pass reads.
ColsDiag diag_cols(const nn_matrix *A, const void *index);

}  // namespace nnqp
