// The diagonal layout of a CSR matrix on the CPU: the plan that
// csrc/diag_plan.hpp makes, its arrays filled as the device kernels fill them,
// and a product that reads them as the device walks do, with every index
// checked.  Built and called by test_diag_plan.py.
#include <cmath>
#include <cstring>
#include <set>

#include "diag_plan.hpp"

using namespace nnqp;

namespace {
struct Walk {
    const DiagPlan &D;
    const std::vector<double> &v;
    const double *x;
    int64_t n;
    bool ok = true;
    double val(int64_t at)
    {
        if (at < 0 || at >= (int64_t)v.size()) return ok = false, 0.0;
        return v[at];
    }
    double col(int64_t j)
    {
        if (j < 0 || j >= n) return ok = false, 0.0;
        return x[j];
    }
    int64_t clamp(int64_t j) const { return std::min(std::max<int64_t>(j, 0), n - 1); }
    // entries of a regular row, columns in ascending order
    double regular(const DiagReg &r, int W, int64_t row, bool edge)
    {
        const int H = W / 2;
        double acc = 0.0;
        for (int k = 0; k < W; k++) {
            const int u = k < H ? H - 1 - k : k - H - 1;
            const int d = k == H ? 0 : (k < H ? -r.h[u] : r.h[u]);
            const int64_t b = r.b0 + (int64_t)(k == H ? 0 : (u + 1) * (int64_t)r.stride) + (k < H ? d : 0);
            const double a = val(b + row), y = col(edge ? clamp(row + d) : row + d);
            acc = std::fma(a, y, acc);
        }
        return acc;
    }
    double general(const DiagRun &r, int64_t row)
    {
        double acc = 0.0;
        for (int h = 0; h < r.w; h += 4)
            for (int k = h; k < h + 4; k++) {
                const double a = val(r.b[k] + row), y = col(clamp(row + r.d[k]));
                if (k < r.w) acc = std::fma(a, y, acc);
            }
        return acc;
    }
};
}  // namespace

// y = K x through the layout.  Returns 0: the pattern has no layout, 1: it has,
// 2: in one regular run (y1: the product as the engines that hold one run read
// it, zeros outside [0, n)), -1: an index out of range, -2: a place of an array
// filled twice with different values.  info: runs, regular slices, main run's.
extern "C" int diag_product(int64_t n, const int64_t *rp, const int *col, const double *val,
                            const double *x, double *y, double *y1, int64_t *info)
{
    const int64_t ns = (n + kSlice - 1) / kSlice;
    int64_t nsell = 0;
    int wmax = 0;
    for (int64_t s = 0; s < ns; s++) {
        int w = 0;
        for (int64_t i = s * kSlice; i < std::min(n, (s + 1) * kSlice); i++)
            w = std::max(w, (int)(rp[i + 1] - rp[i]));
        nsell += (int64_t)w * kSlice;
        wmax = std::max(wmax, w);
    }
    if (nsell < 2 * ns * kSlice || wmax > kDiagMax) return 0;
    std::vector<int> width(ns), first, lists, all((size_t)ns * kDiagMax, 0);
    for (int64_t s = 0; s < ns; s++) {
        std::set<int> d;
        for (int64_t i = s * kSlice; i < std::min(n, (s + 1) * kSlice); i++)
            for (int64_t k = rp[i]; k < rp[i + 1]; k++) d.insert((int)(col[k] - i));
        if ((int)d.size() > kDiagMax) return 0;
        width[s] = (int)d.size();
        std::copy(d.begin(), d.end(), all.begin() + s * kDiagMax);
        if (s == 0 || width[s] != width[s - 1] ||
            !std::equal(d.begin(), d.end(), all.begin() + (s - 1) * kDiagMax))
            first.push_back((int)s);
    }
    const bool packed = 8 * first.size() <= (size_t)ns;
    for (int s : first) lists.insert(lists.end(), all.begin() + (int64_t)s * kDiagMax, all.begin() + (int64_t)(s + 1) * kDiagMax);
    DiagPlan D;
    if (!diag_plan(n, ns, nsell, wmax, first, width.data(), packed ? lists.data() : all.data(), packed, &D))
        return 0;
    auto find = [&](int64_t i, int64_t j) -> const double * {
        for (int64_t k = rp[i]; k < rp[i + 1]; k++)
            if (col[k] == j) return val + k;
        return nullptr;
    };
    // entries that would be read through the opposite triangle
    for (int64_t s = 0; s < ns; s++) {
        if (!D.mirrored[D.srun[s]]) continue;
        const DiagRun &r = D.runs[D.srun[s]];
        for (int64_t i = s * kSlice; i < std::min(n, (s + 1) * kSlice); i++)
            for (int k = 0; k < r.w && r.d[k] < 0; k++) {
                const int64_t j = i + r.d[k];
                if (j < 0) continue;
                const double *a = find(i, j), *b = find(j, i);
                if (!a != !b || (a && std::memcmp(a, b, sizeof(double)) != 0)) return 0;
            }
    }
    const bool zeros = D.runs[D.srun[0]].kind != DR_GENERAL || D.mirrored[D.srun[0]];
    std::vector<double> v((size_t)D.entries, zeros ? 0.0 : NAN);
    std::vector<char> set((size_t)D.entries, 0);
    for (int64_t s = 0; s < ns; s++) {
        const DiagRun &r = D.runs[D.srun[s]];
        for (int64_t i = s * kSlice; i < (s + 1) * kSlice; i++)
            for (int k = 0; k < r.w; k++) {
                if (D.mirrored[D.srun[s]] && r.d[k] < 0) continue;
                const double *a = i < n ? find(i, i + r.d[k]) : nullptr;
                const int64_t at = r.b[k] + i;
                if (at < 0 || at >= D.entries) return -1;
                if (set[at]) return -2;
                set[at] = 1;
                v[at] = a ? *a : 0.0;
            }
    }
    const int W = diag_regular(wmax);
    Walk w{D, v, x, n};
    info[0] = (int64_t)D.runs.size();
    info[1] = 0;
    info[2] = D.ehi - D.elo;
    for (int64_t s = 0; s < ns; s++) {
        const bool main = s >= D.elo && s < D.ehi;
        const DiagRun &r = D.runs[D.srun[s]];
        const int kind = main ? (s >= D.lo && s < D.hi ? DR_REGULAR : DR_EDGE) : r.kind;
        info[1] += kind != DR_GENERAL;
        for (int64_t i = s * kSlice; i < (s + 1) * kSlice; i++) {
            const double a = kind == DR_GENERAL ? w.general(r, i)
                                                : w.regular(main ? D.main : r.reg, W, i, kind == DR_EDGE);
            if (i < n) y[i] = a;
        }
    }
    if (!w.ok) return -1;
    if (D.elo != 0 || D.ehi != ns) return 1;
    std::vector<double> padded(ns * kSlice + 2 * (size_t)D.main.h[W / 2 - 1], 0.0);
    std::copy(x, x + n, padded.begin() + D.main.h[W / 2 - 1]);
    Walk o{D, v, padded.data() + D.main.h[W / 2 - 1], 0};
    for (int64_t i = 0; i < n; i++) {
        double acc = 0.0;
        for (int k = 0; k < W; k++) {
            const int H = W / 2, u = k < H ? H - 1 - k : k - H - 1;
            const int d = k == H ? 0 : (k < H ? -D.main.h[u] : D.main.h[u]);
            const int64_t b = D.main.b0 + (int64_t)(k == H ? 0 : (u + 1) * (int64_t)D.main.stride) + (k < H ? d : 0);
            acc = std::fma(o.val(b + i), o.x[i + d], acc);
        }
        y1[i] = acc;
    }
    return o.ok ? 2 : -1;
}
