// P1 assembly of the stiffness matrix K, capacity matrix M and load F.
//
// The mesh is uploaded once and everything after the size checks runs on the
// device (a 96 x 96 x 24 slab with K and M, 208 k rows: 4.1 ms, 1.1 of them in
// kernels and most of the rest in the transfer of 48 MB; 38 ms with a symbolic
// phase on the host's threads): validation, free-DOF numbering (scan),
// node-to-element incidence (count, scan, fill, sort each node's few elements),
// row lengths and slice widths (scans), and a row-gather numeric phase.  The host waits twice before
// it, for the flags of the validation with the number of free nodes and for
// the sizes of the matrix.  A mesh with a row of more than kRowMax columns
// or kIncMax elements takes the host's symbolic phase and k_assemble instead,
// behind the device's, which finds that row (a square of 500^2 cells beside a hub
// of 200 triangles 16.0 ms, one of 1,000^2 38.3; 16.7 and 47.0 before there was a
// device phase to run first).
//
// Numeric phase: one thread owns one free row i and walks the elements
// incident to its node in increasing element order; for each it forms the P1
// gradients and adds the row's element entries
//     K^e_ab = |e| grad phi_a . D_e grad phi_b,
//     M^e_ab = |e| (1 + delta_ab) / ((d+1)(d+2)),   F^e_a = |e| f_e / (d+1)
// (bilinear form B and functional L of Sec. 2.1.2; capacity matrix of
// Sec. 2.2.2) into the row's own slots.  No two threads write the same slot,
// so no atomics are needed and the result is reproducible; the stiffness
// entry is evaluated with a form symmetric in (a, b), so K is bitwise
// symmetric.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <thread>
#include <vector>

#include "nnqp_internal.hpp"

namespace nnqp {

namespace {

template <class F>
void parallel_for(int64_t n, F &&fn)
{
    unsigned nt = std::thread::hardware_concurrency();
    if (nt == 0) nt = 1;
    if (nt > 32) nt = 32;
    if (n < 4096) nt = 1;
    if (nt == 1) {
        fn(0, n, 0);
        return;
    }
    std::vector<std::thread> th;
    int64_t per = (n + nt - 1) / nt;
    for (unsigned t = 0; t < nt; t++) {
        int64_t a = (int64_t)t * per, b = std::min<int64_t>(n, a + per);
        if (a >= b) break;
        th.emplace_back([&, a, b, t] { fn(a, b, (int)t); });
    }
    for (auto &x : th) x.join();
}

// A scratch device buffer of one call, taken from and returned to the
// context's allocator.
struct DevBuf {
    const nnqp::DevAlloc &al;
    void *p = nullptr;
    explicit DevBuf(const nnqp::DevAlloc &a) : al(a) {}
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    ~DevBuf() { nnqp::dev_free(al, p); }
};

}  // namespace

// ---------------------------------------------------------------- device side
struct AsmArgs {
    int dim;
    int nfree;
    const int *free_node;   // [nfree] node id of each free row
    const int64_t *inc_ptr; // [n_nodes + 1]
    const int *inc_elem;    // incident elements, ascending per node
    const int *elems;       // [ne * (dim+1)]
    const double *coords;   // [nn * dim]
    const double *D;        // [nD * dim * dim]
    int per_elem_D;
    const double *kscale;   // [ne] or null
    const double *f;        // [ne]
    const double *dval;     // [nn] Dirichlet values or null (homogeneous)
    const int *dof;         // [nn]
    const int *rowptr;
    const int *col;
    double *val;
    double *mval;           // or null
    double *F;
};

// K^e_ab without contraction and in an order symmetric in (a, b).
template <int DIM>
__device__ __forceinline__ double stiff_entry(const double *Dm, const double *ga, const double *gb)
{
#pragma clang fp contract(off)
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; k++) s += Dm[k * DIM + k] * (ga[k] * gb[k]);
#pragma unroll
    for (int k = 0; k < DIM; k++)
#pragma unroll
        for (int l = k + 1; l < DIM; l++) s += Dm[k * DIM + l] * (ga[k] * gb[l] + ga[l] * gb[k]);
    return s;
}

// One element as a row's thread needs it: vertices, gradients of the
// barycentric functions, volume and tensor.
template <int DIM>
struct Elem {
    int vid[DIM + 1];
    double gr[DIM + 1][DIM];
    double vol;
    double Dm[DIM * DIM];
};

template <int DIM>
__device__ __forceinline__ void load_elem(const AsmArgs &A, int e, Elem<DIM> &E)
{
    constexpr int NV = DIM + 1;
    double x[NV][DIM];
#pragma unroll
    for (int a = 0; a < NV; a++) E.vid[a] = A.elems[(int64_t)e * NV + a];
#pragma unroll
    for (int a = 0; a < NV; a++)
#pragma unroll
        for (int k = 0; k < DIM; k++) x[a][k] = A.coords[(int64_t)E.vid[a] * DIM + k];
    auto &gr = E.gr;
    if constexpr (DIM == 2) {
        const double e1x = x[1][0] - x[0][0], e1y = x[1][1] - x[0][1];
        const double e2x = x[2][0] - x[0][0], e2y = x[2][1] - x[0][1];
        const double det = e1x * e2y - e1y * e2x;
        gr[1][0] = e2y / det;
        gr[1][1] = -e2x / det;
        gr[2][0] = -e1y / det;
        gr[2][1] = e1x / det;
        gr[0][0] = -(gr[1][0] + gr[2][0]);
        gr[0][1] = -(gr[1][1] + gr[2][1]);
        E.vol = fabs(det) * 0.5;
    } else {
        // edge vectors e_k = x_k - x_0 and cross products e2 x e3, e3 x e1, e1 x e2
        double ev[3][3], cr[3][3];
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int k = 0; k < 3; k++) ev[a][k] = x[a + 1][k] - x[0][k];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const double *u = ev[(a + 1) % 3], *w = ev[(a + 2) % 3];
            cr[a][0] = u[1] * w[2] - u[2] * w[1];
            cr[a][1] = u[2] * w[0] - u[0] * w[2];
            cr[a][2] = u[0] * w[1] - u[1] * w[0];
        }
        const double det = ev[0][0] * cr[0][0] + ev[0][1] * cr[0][1] + ev[0][2] * cr[0][2];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            gr[1][k] = cr[0][k] / det;
            gr[2][k] = cr[1][k] / det;
            gr[3][k] = cr[2][k] / det;
            gr[0][k] = -(gr[1][k] + gr[2][k] + gr[3][k]);
        }
        E.vol = fabs(det) / 6.0;
    }
    const double *Ds = A.D + (A.per_elem_D ? (int64_t)e * DIM * DIM : 0);
    const double ks = A.kscale ? A.kscale[e] : 1.0;
#pragma unroll
    for (int k = 0; k < DIM * DIM; k++) E.Dm[k] = ks * Ds[k];
}

// The element's contributions to the row of `node`: add(j, kab, mass) for each
// free vertex (DOF j) in vertex order, and the load into Frow.
template <int DIM, class Add>
__device__ __forceinline__ void add_elem(const AsmArgs &A, int e, const Elem<DIM> &E, int node,
                                         double &Frow, Add add)
{
    constexpr int NV = DIM + 1;
    double gl[DIM];
    int la = 0;
#pragma unroll
    for (int k = 0; k < DIM; k++) gl[k] = E.gr[0][k];
#pragma unroll
    for (int a = 1; a < NV; a++)
        if (E.vid[a] == node) {
            la = a;
#pragma unroll
            for (int k = 0; k < DIM; k++) gl[k] = E.gr[a][k];
        }
    Frow += E.vol * A.f[e] / (double)NV;
    const double mdiag = E.vol * 2.0 / (double)(NV * (NV + 1));
    const double moff = E.vol / (double)(NV * (NV + 1));
#pragma unroll
    for (int b = 0; b < NV; b++) {
        const int j = A.dof[E.vid[b]];
        if (j < 0) {
            // Dirichlet neighbour: its prescribed value moves to the load
            if (A.dval) Frow -= E.vol * stiff_entry<DIM>(E.Dm, gl, E.gr[b]) * A.dval[E.vid[b]];
            continue;
        }
        add(j, E.vol * stiff_entry<DIM>(E.Dm, gl, E.gr[b]), (b == la) ? mdiag : moff);
    }
}

// The general numeric phase: the row's slots in global memory (CSR order).
template <int DIM>
__global__ __launch_bounds__(kBlock) void k_assemble(AsmArgs A)
{
    const int row = blockIdx.x * kBlock + threadIdx.x;
    if (row >= A.nfree) return;
    const int node = A.free_node[row];
    const int s0 = A.rowptr[row], s1 = A.rowptr[row + 1];
    double Frow = 0.0;
    for (int64_t t = A.inc_ptr[node]; t < A.inc_ptr[node + 1]; t++) {
        const int e = A.inc_elem[t];
        Elem<DIM> E;
        load_elem<DIM>(A, e, E);
        add_elem<DIM>(A, e, E, node, Frow, [&](int j, double kab, double m) {
            int slot = s0;
            while (slot < s1 && A.col[slot] != j) slot++;
            if (slot >= s1) return;   // cannot happen: the pattern holds every element pair
            A.val[slot] += kab;
            if (A.mval) A.mval[slot] += m;
        });
    }
    A.F[row] = Frow;
}

// ---------------------------------------------------------------- symbolic phase on the device
// What the device phase takes: the columns of a row (64 rows of them with K and
// M sums fill 60 of the 64 KB of LDS a block has by default) and the elements at
// its node (one thread sorts and walks them).  Rows of the structured meshes
// have 7 columns of 6 elements (squares) and 15 of 24 (cubes); a tetrahedral
// node with 48 columns has at most 90 elements.
constexpr int kRowMax = 48;
constexpr int kIncMax = 96;

// What the host reads back: set by the checks and the size kernels.
struct AsmFlags {
    int bad_elem, bad_coord, bad_D, bad_dval;
    int first_f, first_ks;        // first element with a bad source, scale (INT_MAX: none)
    int long_row, max_row, wmax;
    int pad;
    int64_t n, inc, nnz, nsell;   // totals of the scans
};

// Element ids inside the mesh, finite inputs (the caller's arrays as uploaded).
__global__ __launch_bounds__(256) void ka_check(int64_t nn, int64_t ne, int dim, int64_t nD,
                                                const int *__restrict__ elems,
                                                const double *__restrict__ coords,
                                                const double *__restrict__ D,
                                                const double *__restrict__ ks,
                                                const double *__restrict__ f,
                                                const uint8_t *__restrict__ dirichlet,
                                                const double *__restrict__ dv, AsmFlags *F)
{
    const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x, nt = (int64_t)gridDim.x * 256;
    bool be = false, bc = false, bd = false, bv = false;
    for (int64_t t = t0; t < ne * (dim + 1); t += nt) be = be || elems[t] < 0 || elems[t] >= nn;
    for (int64_t t = t0; t < nn * dim; t += nt) bc = bc || !isfinite(coords[t]);
    for (int64_t t = t0; t < nD * dim * dim; t += nt) bd = bd || !isfinite(D[t]);
    int ff = 0x7fffffff, fk = 0x7fffffff;
    for (int64_t e = t0; e < ne; e += nt) {
        if (!isfinite(f[e])) ff = min(ff, (int)e);
        if (ks && !(isfinite(ks[e]) && ks[e] > 0.0)) fk = min(fk, (int)e);
    }
    if (dv)
        for (int64_t v = t0; v < nn; v += nt) bv = bv || (dirichlet[v] && !isfinite(dv[v]));
    if (be) F->bad_elem = 1;
    if (bc) F->bad_coord = 1;
    if (bd) F->bad_D = 1;
    if (bv) F->bad_dval = 1;
    if (ff != 0x7fffffff) atomicMin(&F->first_f, ff);
    if (fk != 0x7fffffff) atomicMin(&F->first_ks, fk);
}

// Exclusive scan of get(i), i < n, into put(i, sum before i): kScan items per
// block, the blocks' sums scanned by one block in between.
constexpr int kScan = 2048;   // 256 threads x 8

template <class Get>
__global__ __launch_bounds__(256) void ka_scan_sums(int64_t n, Get get, int64_t *__restrict__ sums)
{
    __shared__ int64_t sh[4];
    const int64_t base = (int64_t)blockIdx.x * kScan + threadIdx.x * 8;
    int64_t a = 0;
#pragma unroll
    for (int k = 0; k < 8; k++)
        if (base + k < n) a += get(base + k);
    for (int o = 32; o >= 1; o >>= 1) a += __shfl_xor(a, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// sums -> exclusive prefix sums, one block; the total goes to *total
__global__ __launch_bounds__(1024) void ka_scan_top(int nb, int64_t *__restrict__ sums, int64_t *total)
{
    __shared__ int64_t sh[1024];
    int64_t carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        const int64_t v = b < nb ? sums[b] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const int64_t w = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += w;
            __syncthreads();
        }
        if (b < nb) sums[b] = carry + sh[threadIdx.x] - v;
        carry += sh[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

template <class Get, class Put>
__global__ __launch_bounds__(256) void ka_scan_put(int64_t n, Get get, Put put,
                                                   const int64_t *__restrict__ sums)
{
    __shared__ int64_t sh[256];
    const int64_t base = (int64_t)blockIdx.x * kScan + threadIdx.x * 8;
    int64_t v[8], a = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        v[k] = base + k < n ? (int64_t)get(base + k) : 0;
        a += v[k];
    }
    sh[threadIdx.x] = a;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const int64_t w = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
        __syncthreads();
        sh[threadIdx.x] += w;
        __syncthreads();
    }
    int64_t at = sums[blockIdx.x] + sh[threadIdx.x] - a;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        if (base + k < n) put(base + k, at);
        at += v[k];
    }
}

template <class Get, class Put>
void scan(hipStream_t st, int64_t n, Get get, Put put, int64_t *sums, int64_t *total)
{
    const int nb = (int)std::max<int64_t>(1, (n + kScan - 1) / kScan);
    ka_scan_sums<<<nb, 256, 0, st>>>(n, get, sums);
    ka_scan_top<<<1, 1024, 0, st>>>(nb, sums, total);
    ka_scan_put<<<nb, 256, 0, st>>>(n, get, put, sums);
}

// elements at each node (cnt zero on entry), and the place of each in its
// node's list (in any order): 149 us for 5.3 M, the rate of the atomics, which
// the fill behind it then does without (218 -> 20 us)
__global__ __launch_bounds__(256) void ka_count(int64_t m, const int *__restrict__ elems,
                                                int *__restrict__ cnt, int *__restrict__ place)
{
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < m; t += (int64_t)gridDim.x * 256)
        place[t] = atomicAdd(&cnt[elems[t]], 1);
}

// every element into its nodes' lists
template <int NV>
__global__ __launch_bounds__(256) void ka_fill(int64_t m, const int *__restrict__ elems,
                                               const int64_t *__restrict__ ptr,
                                               const int *__restrict__ place, int *__restrict__ list)
{
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < m; t += (int64_t)gridDim.x * 256)
        list[ptr[elems[t]] + place[t]] = (int)(t / NV);
}

__device__ __forceinline__ void insertion_sort(int *x, int n)
{
    for (int i = 1; i < n; i++) {
        const int e = x[i];
        int k = i;
        while (k > 0 && x[k - 1] > e) {
            x[k] = x[k - 1];
            k--;
        }
        x[k] = e;
    }
}

// Each node's elements in increasing order (insertion: the lists are short and
// nearly sorted; a longer one has no row here, or sends the mesh to the host).
// The lists of a block's 256 nodes are one range: it goes through LDS when it
// fits (32 elements a node), where the sort's dependent accesses are cheap
// (228 k nodes of 24 elements: 167 -> 50 us).
constexpr int kSortLds = 256 * 32;

__global__ __launch_bounds__(256) void ka_sort(int64_t nn, const int64_t *__restrict__ ptr,
                                               int *__restrict__ list)
{
    __shared__ int s[kSortLds];
    const int64_t v0 = (int64_t)blockIdx.x * 256, v = v0 + threadIdx.x;
    const int64_t r0 = ptr[v0], r1 = ptr[min(v0 + 256, nn)];
    const int64_t a = v < nn ? ptr[v] : r1, b = v < nn ? ptr[v + 1] : r1;
    const int len = b - a > kIncMax ? 0 : (int)(b - a);
    if (r1 - r0 <= kSortLds) {
        const int m = (int)(r1 - r0);
        for (int i = threadIdx.x; i < m; i += 256) s[i] = list[r0 + i];
        __syncthreads();
        insertion_sort(s + (a - r0), len);
        __syncthreads();
        for (int i = threadIdx.x; i < m; i += 256) list[r0 + i] = s[i];
    } else {
        insertion_sort(list + a, len);
    }
}

constexpr int kPatBlock = 64;   // one slice per block

// Sorted distinct columns of a free row in a strip of LDS (entry k of a thread
// at c[k * kPatBlock]); returns their number, or cap + 1 when they do not fit.
template <int DIM>
__device__ __forceinline__ int row_columns(const AsmArgs &A, int node, int *c, int cap)
{
    constexpr int NV = DIM + 1, T = kPatBlock;
    int len = 0;
    const int64_t t1 = A.inc_ptr[node + 1];
    for (int64_t t = A.inc_ptr[node]; t < t1; t++) {
        const int64_t e = A.inc_elem[t];
        int j[NV];
#pragma unroll
        for (int b = 0; b < NV; b++) j[b] = A.dof[A.elems[e * NV + b]];
#pragma unroll
        for (int b = 0; b < NV; b++) {
            if (j[b] < 0) continue;
            int k = len;
            while (k > 0 && c[(k - 1) * T] > j[b]) k--;
            if (k > 0 && c[(k - 1) * T] == j[b]) continue;
            if (len == cap) return cap + 1;
            for (int q = len; q > k; q--) c[q * T] = c[(q - 1) * T];
            c[k * T] = j[b];
            len++;
        }
    }
    return len;
}

// row lengths and slice widths
template <int DIM>
__global__ __launch_bounds__(kPatBlock) void ka_rows(AsmArgs A, int *__restrict__ rowlen,
                                                     int *__restrict__ width, AsmFlags *F)
{
    __shared__ int c[kRowMax * kPatBlock];
    const int row = blockIdx.x * kPatBlock + threadIdx.x;
    int len = 0;
    if (row < A.nfree) {
        const int node = A.free_node[row];
        if (A.inc_ptr[node + 1] - A.inc_ptr[node] > kIncMax) len = kRowMax + 1;
        else len = row_columns<DIM>(A, node, c + threadIdx.x, kRowMax);
        if (len > kRowMax) F->long_row = 1;
        rowlen[row] = len;
    }
    int w = len;
    for (int o = 32; o >= 1; o >>= 1) w = max(w, __shfl_xor(w, o, 64));
    if (threadIdx.x == 0) {
        width[blockIdx.x] = w;
        atomicMax(&F->wmax, w);
    }
}

// The numeric phase with the row's columns and sums in LDS: CSR columns, and
// the sliced-ELL arrays of nn_matrix (padding: own row, value 0; rows past the
// last one: column 0, value 0).  cap: the longest row.
// What bounds it is the latency of the gathers (element, DOFs, vertices) of one
// row's 24 elements: 0.52 ms for the 208 k rows of a 96 x 96 x 24 slab with K
// and M, where k_assemble, whose additions into global slots wait for one
// another, took 2.2 ms and a layout pass behind it.  LDS holds exactly the
// longest row (19 KB a block at 15 columns, eight blocks on a CU).
template <int DIM, bool MASS>
__global__ __launch_bounds__(kPatBlock) void ka_numeric(AsmArgs A, const int *__restrict__ so,
                                                        int *__restrict__ col, int *__restrict__ sc,
                                                        double *__restrict__ sv,
                                                        double *__restrict__ smv, int cap)
{
    extern __shared__ double lds[];   // cap x kPatBlock: K sums, M sums, columns
    constexpr int T = kPatBlock;
    double *ks = lds, *ms = lds + cap * T;
    int *cs = reinterpret_cast<int *>(lds + (MASS ? 2 : 1) * cap * T);
    const int tid = threadIdx.x;
    const int row = blockIdx.x * T + tid;
    const int off = so[blockIdx.x], w = (so[blockIdx.x + 1] - off) / kSlice;
    if (row >= A.nfree) {
        for (int k = 0; k < w; k++) {
            const int e = off + k * kSlice + tid;
            sc[e] = 0;
            sv[e] = 0.0;
            if (MASS) smv[e] = 0.0;
        }
        return;
    }
    const int node = A.free_node[row];
    int *c = cs + tid;
    double *kk = ks + tid, *mm = ms + tid;
    const int len = row_columns<DIM>(A, node, c, cap);
    for (int k = 0; k < len; k++) {
        kk[k * T] = 0.0;
        if (MASS) mm[k * T] = 0.0;
    }
    double Frow = 0.0;
    for (int64_t t = A.inc_ptr[node]; t < A.inc_ptr[node + 1]; t++) {
        const int e = A.inc_elem[t];
        Elem<DIM> E;
        load_elem<DIM>(A, e, E);
        add_elem<DIM>(A, e, E, node, Frow, [&](int j, double kab, double m) {
            int lo = 0, hi = len - 1;   // the row holds j
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (c[mid * T] < j) lo = mid + 1;
                else hi = mid;
            }
            kk[lo * T] += kab;
            if (MASS) mm[lo * T] += m;
        });
    }
    A.F[row] = Frow;
    const int p0 = A.rowptr[row];
    for (int k = 0; k < w; k++) {
        const int e = off + k * kSlice + tid;
        const bool real = k < len;
        if (real) col[p0 + k] = c[k * T];
        sc[e] = real ? c[k * T] : row;
        sv[e] = real ? kk[k * T] : 0.0;
        if (MASS) smv[e] = real ? mm[k * T] : 0.0;
    }
}

// first row whose diagonal is not finite or not positive: 2 row + (not finite)
__global__ __launch_bounds__(256) void ka_diag(int64_t n, const double *__restrict__ d,
                                               unsigned long long *first)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const bool nf = !isfinite(d[i]);
    if (nf || !(d[i] > 0.0)) atomicMin(first, 2ull * (unsigned long long)i + (nf ? 1 : 0));
}

// ---------------------------------------------------------------- host side
void sell_offsets(const int64_t *rowptr, int64_t n, std::vector<int64_t> &off, int &wmax)
{
    const int64_t ns = (n + kSlice - 1) / kSlice;
    off.assign(ns + 1, 0);
    wmax = 0;
    for (int64_t s = 0; s < ns; s++) {
        int w = 0;
        for (int64_t i = s * kSlice; i < std::min<int64_t>(n, (s + 1) * kSlice); i++)
            w = std::max<int>(w, (int)(rowptr[i + 1] - rowptr[i]));
        off[s + 1] = off[s] + (int64_t)w * kSlice;
        wmax = std::max(wmax, w);
    }
}

nn_status sell_build(nn_ctx *ctx, nn_matrix *A, const int64_t *rowptr_host, const double *csr_val,
                     const double *csr_mval)
{
    std::vector<int64_t> off;
    int wmax = 0;
    sell_offsets(rowptr_host, A->n, off, wmax);
    const int64_t ns = (int64_t)off.size() - 1;
    const int64_t nsell = off.back();
    if (nsell >= ((int64_t)1 << 31)) return fail(ctx, NN_EINVAL, "sliced-ELL size exceeds 32-bit offsets");
    A->nslices = ns;
    A->nsell = nsell;
    A->wmax = wmax;
    std::vector<int> off32(off.begin(), off.end());
    const size_t ne = (size_t)std::max<int64_t>(nsell, 1);
    hipError_t e = dev_malloc(A->al, &A->sl_off, sizeof(int) * (ns + 1));
    if (e == hipSuccess) e = dev_malloc(A->al, &A->sl_col, sizeof(int) * ne);
    if (e == hipSuccess) e = dev_malloc(A->al, &A->val, sizeof(double) * ne);
    if (e == hipSuccess && csr_mval) e = dev_malloc(A->al, &A->mval, sizeof(double) * ne);
    if (e != hipSuccess) return fail(ctx, NN_EOOM, "sliced-ELL allocation failed");
    NN_HIP_TRY(ctx, hipMemcpyAsync(A->sl_off, off32.data(), sizeof(int) * (ns + 1),
                                   hipMemcpyHostToDevice, ctx->stream));
    if (A->n > 0) launch_csr_to_sell(ctx, A, csr_val, csr_mval);
    NN_HIP_TRY(ctx, hipGetLastError());
    NN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    return NN_OK;
}

nn_status finish_matrix(nn_ctx *ctx, nn_matrix *A)
{
    if (A->n > 0) {
        // int16 column offsets for the float32-value passes, kept only when
        // every |col - row| fits
        short *sd = nullptr;
        if (dev_malloc(A->al, &sd, sizeof(short) * std::max<int64_t>(A->nsell, 1)) != hipSuccess)
            return fail(ctx, NN_EOOM, "int16 offset allocation failed");
        launch_sell_d16(ctx, A, sd);
        static const int kMaxOp[1] = {OP_MAX};
        double span = 0.0;
        nn_status rc = host_reduce(ctx, A->n, 1, kMaxOp, &span);
        if (rc != NN_OK) {
            dev_free(A->al, sd);
            return rc;
        }
        if (span <= 32767.0) A->sl_d16 = sd;
        else dev_free(A->al, sd);
        if (dev_malloc(A->al, &A->diag, sizeof(double) * A->n) != hipSuccess)
            return fail(ctx, NN_EOOM, "diagonal allocation failed");
        launch_diag(ctx, A, A->val, A->diag);
        // (the result goes through the reduction partials, free between passes)
        unsigned long long *first = reinterpret_cast<unsigned long long *>(ctx->partials);
        unsigned long long none = ~0ull, bad = none;
        NN_HIP_TRY(ctx, hipMemsetAsync(first, 0xff, sizeof(none), ctx->stream));
        ka_diag<<<(unsigned)((A->n + 255) / 256), 256, 0, ctx->stream>>>(A->n, A->diag, first);
        NN_HIP_TRY(ctx, hipGetLastError());
        NN_HIP_TRY(ctx, hipMemcpyAsync(&bad, first, sizeof(bad), hipMemcpyDeviceToHost, ctx->stream));
        NN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        if (bad != none) {
            if (bad & 1) return fail(ctx, NN_ENONFINITE, "non-finite diagonal entry");
            return fail(ctx, NN_ENOTSPD, "non-positive diagonal entry at row " + std::to_string(bad / 2));
        }
    }
    return NN_OK;
}

// The host's symbolic phase and the general numeric phase (a mesh with rows of
// more than kRowMax columns); the arguments have been checked.
static nn_status assemble_host(nn_ctx *ctx, const nn_mesh *mesh, const double *D, int64_t nD,
                               const double *kscale, const double *f_elem, const uint8_t *dirichlet,
                               const double *dvals, int with_mass, nn_matrix **K_out, double *F_dev,
                               int64_t *dof_of_node)
{
    const int dim = mesh->dim;
    const int64_t nn = mesh->n_nodes, ne = mesh->n_elems;
    const int nv = dim + 1;

    // ---- free-DOF numbering
    std::vector<int> dof(nn);
    std::vector<int> free_node;
    free_node.reserve(nn);
    for (int64_t v = 0; v < nn; v++) {
        if (dirichlet[v]) {
            dof[v] = -1;
        } else {
            dof[v] = (int)free_node.size();
            free_node.push_back((int)v);
        }
    }
    const int64_t n = (int64_t)free_node.size();
    if (dof_of_node)
        for (int64_t v = 0; v < nn; v++) dof_of_node[v] = dof[v];

    // ---- node -> element incidence (elements ascending per node)
    std::vector<int64_t> inc_ptr(nn + 1, 0);
    for (int64_t t = 0; t < ne * nv; t++) inc_ptr[mesh->elems[t] + 1]++;
    for (int64_t v = 0; v < nn; v++) inc_ptr[v + 1] += inc_ptr[v];
    std::vector<int> inc_elem(std::max<int64_t>(inc_ptr[nn], 1));
    {
        std::vector<int64_t> pos(inc_ptr.begin(), inc_ptr.end() - 1);
        for (int64_t e = 0; e < ne; e++)
            for (int a = 0; a < nv; a++) inc_elem[pos[mesh->elems[e * nv + a]]++] = (int)e;
    }

    // ---- CSR pattern of the free rows
    std::vector<int> rowlen(n);
    auto row_cols = [&](int node, std::vector<int> &buf) {
        buf.clear();
        for (int64_t t = inc_ptr[node]; t < inc_ptr[node + 1]; t++) {
            const int e = inc_elem[t];
            for (int b = 0; b < nv; b++) {
                const int j = dof[mesh->elems[(int64_t)e * nv + b]];
                if (j >= 0) buf.push_back(j);
            }
        }
        std::sort(buf.begin(), buf.end());
        buf.erase(std::unique(buf.begin(), buf.end()), buf.end());
    };
    parallel_for(n, [&](int64_t a, int64_t b, int) {
        std::vector<int> buf;
        for (int64_t r = a; r < b; r++) {
            row_cols(free_node[r], buf);
            rowlen[r] = (int)buf.size();
        }
    });
    std::vector<int64_t> rp64(n + 1, 0);
    for (int64_t r = 0; r < n; r++) rp64[r + 1] = rp64[r] + rowlen[r];
    const int64_t nnz = rp64[n];
    if (nnz >= ((int64_t)1 << 31)) return fail(ctx, NN_EINVAL, "nnz exceeds 32-bit row pointers");
    std::vector<int> rowptr(n + 1), col(std::max<int64_t>(nnz, 1));
    for (int64_t r = 0; r <= n; r++) rowptr[r] = (int)rp64[r];
    parallel_for(n, [&](int64_t a, int64_t b, int) {
        std::vector<int> buf;
        for (int64_t r = a; r < b; r++) {
            row_cols(free_node[r], buf);
            std::copy(buf.begin(), buf.end(), col.begin() + rowptr[r]);
        }
    });

    // ---- device numeric phase
    nn_matrix *M = new (std::nothrow) nn_matrix();
    if (!M) return fail(ctx, NN_EOOM, "host allocation");
    M->al = ctx->al;
    M->n = n;
    M->nnz = nnz;
    auto cleanup = [&](nn_status st) {
        nn_matrix_free(ctx, M);
        return st;
    };
    const DevAlloc &ta = ctx->al;   // scratch of this call
    DevBuf d_free(ta), d_incp(ta), d_ince(ta), d_elems(ta), d_coords(ta), d_D(ta), d_ks(ta),
        d_f(ta), d_dv(ta), d_dof(ta), d_F(ta), d_val(ta), d_mval(ta);
    auto up = [&](DevBuf &b, const void *src, size_t bytes) -> hipError_t {
        hipError_t e = dev_malloc(ta, &b.p, bytes > 0 ? bytes : 8);
        if (e != hipSuccess) return e;
        if (src && bytes > 0) e = hipMemcpyAsync(b.p, src, bytes, hipMemcpyHostToDevice, ctx->stream);
        return e;
    };
#define NN_UP(buf, src, bytes)                                                              \
    do {                                                                                    \
        hipError_t e_ = up(buf, src, bytes);                                                \
        if (e_ != hipSuccess) {                                                             \
            fail(ctx, e_ == hipErrorOutOfMemory ? NN_EOOM : NN_EHIP,                        \
                 std::string("assembly upload: ") + hipGetErrorString(e_));                 \
            return cleanup(e_ == hipErrorOutOfMemory ? NN_EOOM : NN_EHIP);                  \
        }                                                                                   \
    } while (0)
    NN_UP(d_free, free_node.data(), sizeof(int) * n);
    NN_UP(d_incp, inc_ptr.data(), sizeof(int64_t) * (nn + 1));
    NN_UP(d_ince, inc_elem.data(), sizeof(int) * inc_elem.size());
    NN_UP(d_elems, mesh->elems, sizeof(int) * ne * nv);
    NN_UP(d_coords, mesh->coords, sizeof(double) * nn * dim);
    NN_UP(d_D, D, sizeof(double) * nD * dim * dim);
    if (kscale) NN_UP(d_ks, kscale, sizeof(double) * ne);
    NN_UP(d_f, f_elem, sizeof(double) * ne);
    if (dvals) NN_UP(d_dv, dvals, sizeof(double) * nn);
    NN_UP(d_dof, dof.data(), sizeof(int) * nn);
    {
        hipError_t e = dev_malloc(M->al, &M->rowptr, sizeof(int) * (n + 1));
        if (e == hipSuccess) e = dev_malloc(M->al, &M->col, sizeof(int) * std::max<int64_t>(nnz, 1));
        if (e == hipSuccess) e = dev_malloc(ta, &d_val.p, sizeof(double) * std::max<int64_t>(nnz, 1));
        if (e == hipSuccess && with_mass)
            e = dev_malloc(ta, &d_mval.p, sizeof(double) * std::max<int64_t>(nnz, 1));
        if (e == hipSuccess && !F_dev) e = dev_malloc(ta, &d_F.p, sizeof(double) * std::max<int64_t>(n, 1));
        if (e != hipSuccess) {
            fail(ctx, NN_EOOM, std::string("matrix allocation: ") + hipGetErrorString(e));
            return cleanup(NN_EOOM);
        }
    }
    NN_HIP_TRY(ctx, hipMemcpyAsync(M->rowptr, rowptr.data(), sizeof(int) * (n + 1),
                                   hipMemcpyHostToDevice, ctx->stream));
    if (nnz > 0) {
        NN_HIP_TRY(ctx, hipMemcpyAsync(M->col, col.data(), sizeof(int) * nnz, hipMemcpyHostToDevice,
                                       ctx->stream));
        NN_HIP_TRY(ctx, hipMemsetAsync(d_val.p, 0, sizeof(double) * nnz, ctx->stream));
        if (d_mval.p) NN_HIP_TRY(ctx, hipMemsetAsync(d_mval.p, 0, sizeof(double) * nnz, ctx->stream));
    }
    AsmArgs args;
    args.dim = dim;
    args.nfree = (int)n;
    args.free_node = (const int *)d_free.p;
    args.inc_ptr = (const int64_t *)d_incp.p;
    args.inc_elem = (const int *)d_ince.p;
    args.elems = (const int *)d_elems.p;
    args.coords = (const double *)d_coords.p;
    args.D = (const double *)d_D.p;
    args.per_elem_D = nD == 1 ? 0 : 1;
    args.kscale = (const double *)d_ks.p;
    args.f = (const double *)d_f.p;
    args.dval = (const double *)d_dv.p;
    args.dof = (const int *)d_dof.p;
    args.rowptr = M->rowptr;
    args.col = M->col;
    args.val = (double *)d_val.p;
    args.mval = (double *)d_mval.p;
    args.F = F_dev ? F_dev : (double *)d_F.p;
    if (n > 0) {
        const int64_t nb = (n + kBlock - 1) / kBlock;
        if (dim == 2) k_assemble<2><<<(unsigned)nb, kBlock, 0, ctx->stream>>>(args);
        else k_assemble<3><<<(unsigned)nb, kBlock, 0, ctx->stream>>>(args);
        NN_HIP_TRY(ctx, hipGetLastError());
    }
    NN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    nn_status st = sell_build(ctx, M, rp64.data(), (const double *)d_val.p, (const double *)d_mval.p);
    if (st == NN_OK) st = finish_matrix(ctx, M);
    if (st != NN_OK) return cleanup(st);
    int mr = 0;
    for (int64_t r = 0; r < n; r++) mr = std::max(mr, rowlen[r]);
    M->max_row = mr;
    *K_out = M;
    return NN_OK;
#undef NN_UP
}

nn_status assemble_impl(nn_ctx *ctx, const nn_mesh *mesh, const double *D, int64_t nD,
                        const double *kscale, const double *f_elem, const uint8_t *dirichlet,
                        const double *dvals, int with_mass, nn_matrix **K_out, double *F_dev,
                        int64_t *dof_of_node)
{
    if (!mesh || !K_out || !D || !f_elem || !dirichlet)
        return fail(ctx, NN_EINVAL, "null argument to nn_assemble");
    const int dim = mesh->dim;
    if (dim != 2 && dim != 3) return fail(ctx, NN_EINVAL, "mesh dim must be 2 or 3");
    const int64_t nn = mesh->n_nodes, ne = mesh->n_elems;
    if (nn < 0 || ne < 0 || (nn > 0 && !mesh->coords) || (ne > 0 && !mesh->elems))
        return fail(ctx, NN_EINVAL, "bad mesh sizes or arrays");
    if (nn >= (int64_t)1 << 31 || ne >= (int64_t)1 << 31)
        return fail(ctx, NN_EINVAL, "mesh too large for 32-bit indices");
    if (nD != 1 && nD != ne) return fail(ctx, NN_EINVAL, "nD must be 1 or n_elems");
    const int nv = dim + 1;
    hipStream_t st = ctx->stream;

    // ---- scratch of the call, one allocation
    struct Part {
        size_t off, bytes;
    };
    size_t total = 0;
    auto part = [&](size_t bytes) {
        const Part p{total, bytes};
        total += (bytes + 255) / 256 * 256;
        return p;
    };
    const size_t un = (size_t)nn, ue = (size_t)ne;
    const Part pe = part(4 * ue * nv), pc = part(8 * un * dim), pD = part(8 * (size_t)nD * dim * dim),
               pk = part(kscale ? 8 * ue : 0), pf = part(8 * ue), pv = part(dvals ? 8 * un : 0),
               pm = part(un), pdof = part(4 * un), pfree = part(4 * un), pcnt = part(4 * un),
               pptr = part(8 * (un + 1)), pinc = part(4 * ue * nv), pplace = part(4 * ue * nv),
               plen = part(4 * un), pwid = part(4 * (un / kSlice + 2)), psum = part(8 * (un / kScan + 2)),
               pfl = part(sizeof(AsmFlags)), pF = part(F_dev ? 0 : 8 * un);
    DevBuf buf(ctx->al);
    if (dev_malloc(ctx->al, &buf.p, total) != hipSuccess) return fail(ctx, NN_EOOM, "assembly scratch");
    struct Drain {   // no buffer goes back before the work on it has ended
        hipStream_t st;
        ~Drain() { (void)hipStreamSynchronize(st); }
    } drain{st};
    char *base = static_cast<char *>(buf.p);
    auto at = [&](const Part &p) -> void * { return p.bytes ? base + p.off : nullptr; };
    AsmFlags *flags = (AsmFlags *)(base + pfl.off);
    AsmFlags h{};
    h.first_f = h.first_ks = 0x7fffffff;
    auto up = [&](const Part &p, const void *src) -> hipError_t {
        return p.bytes ? hipMemcpyAsync(base + p.off, src, p.bytes, hipMemcpyHostToDevice, st) : hipSuccess;
    };
    auto sizes = [&]() -> hipError_t {   // the flags as the kernels left them
        const hipError_t e = hipMemcpyAsync(&h, flags, sizeof(h), hipMemcpyDeviceToHost, st);
        return e == hipSuccess ? hipStreamSynchronize(st) : e;
    };

    // ---- upload, validation, free-DOF numbering
    NN_HIP_TRY(ctx, up(pfl, &h));
    NN_HIP_TRY(ctx, up(pm, dirichlet));
    NN_HIP_TRY(ctx, up(pe, mesh->elems));
    NN_HIP_TRY(ctx, up(pc, mesh->coords));
    NN_HIP_TRY(ctx, up(pD, D));
    if (kscale) NN_HIP_TRY(ctx, up(pk, kscale));
    NN_HIP_TRY(ctx, up(pf, f_elem));
    if (dvals) NN_HIP_TRY(ctx, up(pv, dvals));
    const uint8_t *mask = (const uint8_t *)at(pm);
    int *dof = (int *)at(pdof), *free_node = (int *)at(pfree), *cnt = (int *)at(pcnt);
    int *list = (int *)at(pinc), *place = (int *)at(pplace), *rowlen = (int *)at(plen), *width = (int *)at(pwid);
    int64_t *ptr = (int64_t *)at(pptr), *sums = (int64_t *)at(psum);
    const int *elems = (const int *)at(pe);
    AsmArgs args;
    args.dim = dim;
    args.free_node = free_node;
    args.inc_ptr = ptr;
    args.inc_elem = list;
    args.elems = elems;
    args.coords = (const double *)at(pc);
    args.D = (const double *)at(pD);
    args.per_elem_D = nD == 1 ? 0 : 1;
    args.kscale = (const double *)at(pk);
    args.f = (const double *)at(pf);
    args.dval = (const double *)at(pv);
    args.dof = dof;
    args.rowptr = nullptr;
    args.col = nullptr;
    args.val = args.mval = nullptr;
    args.F = F_dev ? F_dev : (double *)at(pF);
    auto grid = [](int64_t m) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((m + 255) / 256, 8192)); };
    ka_check<<<grid(ne * nv), 256, 0, st>>>(nn, ne, dim, nD, elems, args.coords, args.D, args.kscale,
                                            args.f, mask, args.dval, flags);
    scan(st, nn, [mask] __device__(int64_t v) { return mask[v] ? 0 : 1; },
         [mask, dof, free_node] __device__(int64_t v, int64_t k) {
             dof[v] = mask[v] ? -1 : (int)k;
             if (!mask[v]) free_node[k] = (int)v;
         },
         sums, &flags->n);
    NN_HIP_TRY(ctx, hipGetLastError());
    NN_HIP_TRY(ctx, sizes());
    if (h.bad_elem) return fail(ctx, NN_EINVAL, "element node id out of range");
    if (h.bad_coord) return fail(ctx, NN_ENONFINITE, "non-finite coordinate");
    if (h.bad_D) return fail(ctx, NN_ENONFINITE, "non-finite diffusivity");
    if (h.first_f != 0x7fffffff && h.first_f <= h.first_ks)
        return fail(ctx, NN_ENONFINITE, "non-finite source");
    if (h.first_ks != 0x7fffffff) return fail(ctx, NN_ENONFINITE, "kscale must be finite and positive");
    if (h.bad_dval) return fail(ctx, NN_ENONFINITE, "non-finite Dirichlet value");
    const int64_t n = h.n, ns = (n + kSlice - 1) / kSlice;
    args.nfree = (int)n;

    // ---- incidence (elements ascending per node), row lengths, slice widths
    nn_matrix *M = new (std::nothrow) nn_matrix();
    if (!M) return fail(ctx, NN_EOOM, "host allocation");
    M->al = ctx->al;
    M->n = n;
    auto cleanup = [&](nn_status rc) {
        (void)hipStreamSynchronize(st);
        nn_matrix_free(ctx, M);
        return rc;
    };
    auto hip = [&](hipError_t e, const char *what) -> nn_status {
        if (e == hipSuccess) return NN_OK;
        return fail(ctx, e == hipErrorOutOfMemory ? NN_EOOM : NN_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    };
    nn_status rc = NN_OK;
    hipError_t e = dev_malloc(M->al, &M->rowptr, sizeof(int) * (n + 1));
    if (e == hipSuccess) e = dev_malloc(M->al, &M->sl_off, sizeof(int) * (ns + 1));
    if ((rc = hip(e, "matrix allocation")) != NN_OK) return cleanup(rc);
    int *rowptr = M->rowptr, *so = M->sl_off;
    e = hipMemsetAsync(cnt, 0, sizeof(int) * un, st);
    if (e == hipSuccess && ne > 0) ka_count<<<grid(ne * nv), 256, 0, st>>>(ne * nv, elems, cnt, place);
    scan(st, nn, [cnt] __device__(int64_t v) { return cnt[v]; },
         [cnt, ptr, nn] __device__(int64_t v, int64_t k) {
             ptr[v] = k;
             if (v == nn - 1) ptr[nn] = k + cnt[v];
         },
         sums, &flags->inc);
    if (ne > 0) {
        if (dim == 2) ka_fill<3><<<grid(ne * nv), 256, 0, st>>>(ne * nv, elems, ptr, place, list);
        else ka_fill<4><<<grid(ne * nv), 256, 0, st>>>(ne * nv, elems, ptr, place, list);
        ka_sort<<<(unsigned)((nn + 255) / 256), 256, 0, st>>>(nn, ptr, list);
    }
    if (n > 0) {
        if (dim == 2) ka_rows<2><<<(unsigned)ns, kPatBlock, 0, st>>>(args, rowlen, width, flags);
        else ka_rows<3><<<(unsigned)ns, kPatBlock, 0, st>>>(args, rowlen, width, flags);
    }
    // (a row pointer or slice offset past 31 bits is refused below)
    scan(st, n, [rowlen] __device__(int64_t i) { return rowlen[i]; },
         [rowlen, rowptr, n] __device__(int64_t i, int64_t k) {
             rowptr[i] = (int)k;
             if (i == n - 1) rowptr[n] = (int)(k + rowlen[i]);
         },
         sums, &flags->nnz);
    scan(st, ns, [width] __device__(int64_t s) { return (int64_t)width[s] * kSlice; },
         [width, so, ns] __device__(int64_t s, int64_t k) {
             so[s] = (int)k;
             if (s == ns - 1) so[ns] = (int)(k + (int64_t)width[s] * kSlice);
         },
         sums, &flags->nsell);
    if (n == 0) {
        e = hipMemsetAsync(rowptr, 0, sizeof(int), st);
        if (e == hipSuccess) e = hipMemsetAsync(so, 0, sizeof(int), st);
    }
    // the numbering for the caller, while the device works
    if (dof_of_node) {
        int64_t k = 0;
        for (int64_t v = 0; v < nn; v++) dof_of_node[v] = dirichlet[v] ? -1 : k++;
    }
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = sizes();
    if ((rc = hip(e, "assembly")) != NN_OK) return cleanup(rc);
    if (h.long_row) {
        (void)cleanup(NN_OK);
        dev_free(ctx->al, buf.p);
        buf.p = nullptr;
        return assemble_host(ctx, mesh, D, nD, kscale, f_elem, dirichlet, dvals, with_mass, K_out, F_dev,
                             dof_of_node);
    }
    if (h.nnz >= ((int64_t)1 << 31)) return cleanup(fail(ctx, NN_EINVAL, "nnz exceeds 32-bit row pointers"));
    if (h.nsell >= ((int64_t)1 << 31))
        return cleanup(fail(ctx, NN_EINVAL, "sliced-ELL size exceeds 32-bit offsets"));
    M->nnz = h.nnz;
    M->nslices = ns;
    M->nsell = h.nsell;
    M->wmax = h.wmax;
    M->max_row = h.wmax;

    // ---- numeric phase
    const size_t nz = (size_t)std::max<int64_t>(M->nnz, 1), nse = (size_t)std::max<int64_t>(M->nsell, 1);
    e = dev_malloc(M->al, &M->col, sizeof(int) * nz);
    if (e == hipSuccess) e = dev_malloc(M->al, &M->sl_col, sizeof(int) * nse);
    if (e == hipSuccess) e = dev_malloc(M->al, &M->val, sizeof(double) * nse);
    if (e == hipSuccess && with_mass) e = dev_malloc(M->al, &M->mval, sizeof(double) * nse);
    if ((rc = hip(e, "matrix allocation")) != NN_OK) return cleanup(rc);
    args.rowptr = M->rowptr;
    if (n > 0) {
        const size_t lds = (size_t)h.wmax * kPatBlock * (with_mass ? 20 : 12);
        auto go = [&](auto k) {
            k<<<(unsigned)ns, kPatBlock, lds, st>>>(args, M->sl_off, M->col, M->sl_col, M->val, M->mval, h.wmax);
        };
        if (dim == 2) with_mass ? go(ka_numeric<2, true>) : go(ka_numeric<2, false>);
        else with_mass ? go(ka_numeric<3, true>) : go(ka_numeric<3, false>);
    }
    if ((rc = hip(hipGetLastError(), "assembly")) != NN_OK) return cleanup(rc);
    if ((rc = finish_matrix(ctx, M)) != NN_OK) return cleanup(rc);
    if ((rc = hip(hipStreamSynchronize(st), "assembly")) != NN_OK) return cleanup(rc);
    *K_out = M;
    return NN_OK;
}

}  // namespace nnqp
