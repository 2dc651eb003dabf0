// Host side of the diagonal layout (diag.hpp): from the column offsets that
// each slice of a matrix uses, the runs of slices, what kind of walk reads them
// and where their value arrays lie.  Plain C++ without device code, so that a
// host test can compare what a plan reads with the matrix.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace nnqp {

constexpr int kSlice = 64;      // rows of a slice
constexpr int kDiagMax = 32;    // offsets of a run
constexpr int kDiagHalf = 7;    // offsets > 0 of a regular run (3D P1)
constexpr int kDiagRunsMax = 4096;
enum { DR_REGULAR = 0, DR_EDGE = 1, DR_GENERAL = 2 };
// Regular runs: offsets 0, +-h[0], ..., ascending h; the array of offset h[u]
// starts at b0 + (u + 1) stride (that of offset 0 at b0), counted from row 0.
struct DiagReg {
    int b0, stride;
    int h[kDiagHalf];
};
struct DiagRun {
    int w;      // offsets, ascending; slots past w repeat offset 0
    int kind;   // regular, regular with columns that would leave [0, n), general
    DiagReg reg;
    int d[kDiagMax];
    int b[kDiagMax];
};

struct DiagPlan {
    std::vector<int> srun;        // run of each slice
    std::vector<DiagRun> runs;
    std::vector<int> mirrored;    // run: offsets < 0 read through the opposite triangle
    int64_t entries = 0;          // length of a value array
    int lo = 0, hi = 0, elo = 0, ehi = 0;   // slices of the main run (ColsDiag)
    DiagReg main{};
};

// Offsets of a regular row in the kernels' instance for slices of up to wmax
// entries (diag_width): a 2D P1 stencil has 7, a 3D one 15.
constexpr int diag_regular(int wmax) { return wmax <= 8 ? 7 : 15; }

struct PatternRun {
    int s0, s1;
    std::vector<int> d;
};

// Bases of the runs' arrays.  False when the arrays or tables do not fit or
// too few slices are regular.
inline bool lay_out(int64_t n, int64_t nslices, int64_t nsell, int wmax,
                    const std::vector<PatternRun> &pat, DiagPlan *D)
{
    const int W = diag_regular(wmax);
    D->srun.assign((size_t)nslices, 0);
    int64_t regular = 0;
    for (const PatternRun &p : pat) {
        const int w = (int)p.d.size();
        const int64_t rows = (int64_t)(p.s1 - p.s0) * kSlice;
        bool sym = true;
        for (int d : p.d)
            if (d < 0 && !std::binary_search(p.d.begin(), p.d.end(), -d)) sym = false;
        const int dmin = p.d.front(), dmax = p.d.back();
        // slices that store their offsets < 0: all without the opposite
        // offsets, none in a run from row 0 on, else those whose row i - d may
        // lie before the run
        const int64_t reach = (-(int64_t)std::min(dmin, 0) + kSlice - 1) / kSlice;
        const bool front = sym && p.s0 == 0;
        const int head = !sym ? p.s1 - p.s0 : (front ? 0 : (int)std::min<int64_t>(p.s1 - p.s0, reach));
        // arrays of the offsets >= 0: equal lengths (zeros in front when the
        // run starts at row 0), so that their bases are b0 + u stride
        const int64_t pad = front ? reach * kSlice : 0;
        const int64_t stride = rows + pad;
        const int64_t b0 = D->entries + pad - (int64_t)p.s0 * kSlice;
        int nup = 0;
        for (int d : p.d) nup += d >= 0;
        D->entries += nup * stride;
        std::vector<int64_t> base(w);
        for (int k = 0, u = 0; k < w; k++) {
            if (p.d[k] >= 0) {
                base[k] = b0 + stride * u++;
            } else {
                base[k] = D->entries - (int64_t)p.s0 * kSlice;   // (head slices only)
                D->entries += (int64_t)head * kSlice;
            }
        }
        if (D->entries > nsell) return false;
        // regular: 0, +-h[0], +-h[1], ...  (the last rows of a run may reach
        // into the next one with offsets whose opposite no row of the run has)
        bool reg = w == W;
        for (int k = 0; reg && k < w; k++) reg = p.d[k] == -p.d[w - 1 - k];
        auto edge = [&](int s) {
            return (int64_t)s * kSlice + dmin < 0 || (int64_t)s * kSlice + kSlice - 1 + dmax >= n;
        };
        auto kind = [&](int s) {
            if (!reg || s < p.s0 + head) return (int)DR_GENERAL;
            return edge(s) ? (int)DR_EDGE : (int)DR_REGULAR;
        };
        DiagReg g{};
        g.b0 = (int)b0;
        g.stride = (int)stride;
        if (reg)
            for (int u = 0; u < W / 2; u++) g.h[u] = p.d[W / 2 + 1 + u];
        // sub-runs: consecutive slices of one kind, stored or mirrored alike
        int e0 = p.s0 + head, in0 = 0, in1 = 0;
        for (int s = p.s0; s < p.s1;) {
            const bool in_head = s < p.s0 + head;
            int t = s + 1;
            while (t < p.s1 && (t < p.s0 + head) == in_head && kind(t) == kind(s)) t++;
            DiagRun r{};
            r.w = w;
            r.kind = kind(s);
            r.reg = g;
            int64_t zero = b0;
            for (int k = 0; k < w; k++) {
                int64_t b = base[k];
                if (p.d[k] < 0 && !in_head)
                    b = base[std::lower_bound(p.d.begin(), p.d.end(), -p.d[k]) - p.d.begin()] + p.d[k];
                r.d[k] = p.d[k];
                r.b[k] = (int)b;
                if (p.d[k] == 0) zero = b;
            }
            for (int k = w; k < kDiagMax; k++) {
                r.d[k] = 0;
                r.b[k] = (int)zero;
            }
            if (r.kind != DR_GENERAL) regular += t - s;
            if (r.kind == DR_REGULAR && t - s > in1 - in0) {
                in0 = s;
                in1 = t;
            }
            const int id = (int)D->runs.size();
            if (id >= kDiagRunsMax) return false;
            D->runs.push_back(r);
            D->mirrored.push_back(in_head ? 0 : 1);
            for (int q = s; q < t; q++) D->srun[q] = id;
            s = t;
        }
        if (reg && p.s1 - e0 > D->ehi - D->elo) {   // the main run: the longest regular one
            D->elo = e0;
            D->ehi = p.s1;
            D->lo = in0;
            D->hi = in1;
            D->main = g;
        }
    }
    const size_t bytes = sizeof(int) * D->srun.size() + (sizeof(DiagRun) + sizeof(int)) * D->runs.size();
    return bytes <= sizeof(short) * (size_t)nsell && 4 * regular >= 3 * nslices;
}

// The plan of a pattern.  first: the slices whose offsets differ from those of the
// slice before; width: offsets of each slice; lists: kDiagMax offsets of each
// of `first` side by side (packed), or of every slice.  False: no diagonal layout.
inline bool diag_plan(int64_t n, int64_t nslices, int64_t nsell, int wmax,
                      const std::vector<int> &first, const int *width, const int *lists, bool packed,
                      DiagPlan *D)
{
    const int W = diag_regular(wmax);
    // runs: a segment joins the run before it when one's offsets contain
    // the other's (whole slices in the first line of a grid plane lack
    // the offsets to the line before), up to the regular width: slices
    // where the numbering shifts hold the offsets of both sides
    std::vector<PatternRun> pat;
    for (size_t q = 0; q < first.size(); q++) {
        const int s0 = first[q], s1 = q + 1 < first.size() ? first[q + 1] : (int)nslices;
        const int *l = &lists[(packed ? q : (size_t)s0) * kDiagMax], *e = l + width[s0];
        if (!pat.empty() && (int)pat.back().d.size() <= W &&
            std::includes(pat.back().d.begin(), pat.back().d.end(), l, e)) {
            pat.back().s1 = s1;
        } else if (!pat.empty() && width[s0] <= W &&
                   std::includes(l, e, pat.back().d.begin(), pat.back().d.end())) {
            pat.back().s1 = s1;
            pat.back().d.assign(l, e);
        } else {
            PatternRun p;
            p.s0 = s0;
            p.s1 = s1;
            p.d.assign(l, e);
            pat.push_back(p);
        }
    }
    return lay_out(n, nslices, nsell, wmax, pat, D);
}

}  // namespace nnqp
