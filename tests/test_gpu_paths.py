"""Kernel paths at the sizes where they can go wrong (edges of slices, blocks
and grids), through the C ABI, against numpy and the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_1506_08435_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0)
    yield c
    c.close()


# one row, the edges of a wavefront's 64 rows and of a block's 1024, more
# blocks than one wavefront combines (64 x 1024 rows), more than the grid holds
# (512 x 1024 rows)
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 65537, 525000])
@pytest.mark.parametrize("path", ["multi", "one", "batch"])
def test_reductions_of_a_diagonal_problem(ctx, n, path):
    """K = diag(k): the minimiser is max(f, 0) / k, so every reported reduction
    (|f|, the active count, the KKT norms) has a closed form.  The sum of n
    squares in double, in any order, is within n ulp of the exact one."""
    import torch
    if path == "one" and n > 4096:
        pytest.skip("the one-workgroup engine's range")
    rng = np.random.default_rng(n)
    k = rng.uniform(0.5, 2.0, n)
    f = rng.uniform(-1.0, 1.0, n)
    f[n // 2] = 1.0
    K = ctx.matrix_from_csr(np.arange(n + 1), np.arange(n, dtype=np.int32), k)
    F = torch.from_numpy(f).to(ctx.device)
    if path == "batch":
        cs, acts, sts, rc = ctx.solve_batch([K], [F], tol=1e-12)
        c, act, st = cs[0], acts[0], sts[0]
        assert rc == 0
    else:
        c, act, st = ctx.solve_nonneg(K, F, tol=1e-12, engine=1 if path == "multi" else 2)
    ref = np.maximum(f, 0.0) / k
    eps = np.finfo(float).eps
    nf = float(np.sqrt(np.sum(f.astype(np.longdouble) ** 2)))
    assert abs(st["norm_f"] - nf) <= n * eps * nf
    assert st["kkt_rel"] <= 1e-12
    # |c - ref| <= |g| / k, |g| <= tol |f|
    assert np.abs(c.cpu().numpy() - ref).max() <= 2.1e-12 * nf
    c = c.cpu().numpy()
    assert st["n_active"] == int((c == 0.0).sum()) == int((act.cpu().numpy() == 1).sum())
    assert np.all(c[f <= 0.0] == 0.0)
    assert st["min_c"] == c.min()
    K.free()


def _with_zeros(rowptr, col, vals, seed, extra=2):
    """The same matrix with `extra` explicit zero entries per row at random
    columns (and their transposes): every 64-row slice then has more distinct
    column offsets than the diagonal layout takes, and a sum in column order
    keeps its bits (0 * x adds nothing to a finite sum)."""
    n = rowptr.size - 1
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(n), np.diff(rowptr))
    r, c = np.repeat(np.arange(n), extra), rng.integers(0, n, extra * n)
    key = np.concatenate([rows * n + col, r * n + c, c * n + r])
    data = [np.concatenate([v, np.zeros(2 * extra * n)]) for v in vals]
    # the first of equal keys is the real entry
    uniq, first = np.unique(key, return_index=True)
    rp = np.concatenate([[0], np.cumsum(np.bincount(uniq // n, minlength=n))])
    return rp, (uniq % n).astype(np.int32), [d[first] for d in data]


_DIAG = {
    # one slice and a bit; slices that span grid lines; slices inside a line;
    # a line longer than two slices; 3D with fewer and more rows than an
    # offset reaches; a numbering that shifts (runs); offsets past int16
    "square_9": lambda: W.square2d(9), "square_33": lambda: W.square2d(33),
    "square_65": lambda: W.square2d(65), "square_201": lambda: W.square2d(201),
    "cube_5": lambda: W.cube3d(5), "cube_12": lambda: W.cube3d(12), "cube_21": lambda: W.cube3d(21),
    "cube_66": lambda: W.cube3d(66), "hole_3": lambda: W.cube_hole(3),
    "slab": lambda: W.config_transient3d(20, 18, 9, ell=3.0),
    "wide": lambda: W.box_problem("wide", (200, 170, 3), 1 / 200, W.aniso3d_tensor()),
}


@pytest.mark.parametrize("name", sorted(_DIAG))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_diagonal_layout_keeps_the_bits(ctx, name, precision):
    """Solves that read the diagonal layout and solves of the same matrix in a
    pattern without one (explicit zeros) give the same bits: TRON, with a
    Chebyshev preconditioner, with a trust radius, BLMVM, Galerkin, a
    backward-Euler step and products."""
    import torch
    from paper_1506_08435_amd import nnqp
    p = _DIAG[name]()
    K, F, _ = ctx.assemble(p, with_mass=True)
    rp, col, val, mval = ctx.matrix_export(K)
    rpz, colz, (valz, mvalz) = _with_zeros(rp, col, [val, mval], 5)
    Z = ctx.matrix_from_csr(rpz, colz, valz, mvalz)
    assert Z.n == K.n and Z.nnz > K.nnz
    prec = nnqp.NN_MIXED if precision == "mixed" else nnqp.NN_FP64
    kw = dict(tol=1e-8, inner_rtol=0.3, precision=prec, engine=1, lower=0.0)
    calls = [lambda A: ctx.solve_nonneg(A, F, **kw)[:2],
             lambda A: ctx.solve_nonneg(A, F, **kw, precond_degree=3)[:2],
             lambda A: ctx.solve_nonneg(A, F, **kw, delta0=1e-3 * (K.n ** 0.5))[:2],
             lambda A: ctx.step_transient(A, 1e-3, F, torch.zeros(K.n, dtype=torch.float64, device=ctx.device),
                                          **kw)[:2]]
    if precision == "fp64":
        x = torch.from_numpy(np.random.default_rng(3).standard_normal(K.n)).to(ctx.device)
        calls += [lambda A: ctx.solve_nonneg(A, F, tol=1e-6, method=nnqp.NN_BLMVM)[:2],
                  lambda A: ctx.solve_galerkin(A, F, tol=1e-8, max_cg=20000)[:1],
                  lambda A: (ctx.matvec(A, x), ctx.matvec(A, x, which=1))]
    for k, call in enumerate(calls):
        a, b = call(K), call(Z)
        torch.cuda.synchronize()
        for u, w in zip(a, b):
            assert torch.equal(u, w), (name, precision, k, (u != w).sum().item())
    K.free()
    Z.free()


def test_matrix_with_one_unequal_pair_matches_oracle(ctx):
    """K[i, j] and K[j, i] one ulp apart: the entries cannot be shared across
    the diagonal, every stored value counts.  Products are exact to rounding
    against numpy in long double, and the solve matches the oracle."""
    import torch
    p = W.cube3d(12)
    S = oracle.assemble(p)
    val = S.K.copy()
    rows = np.repeat(np.arange(S.n), np.diff(S.rowptr))
    off = np.flatnonzero(rows == S.col + 1)[500]
    val[off] *= 1.0 + 1e-3            # one side only: a visible difference in the product
    K = ctx.matrix_from_csr(S.rowptr, S.col, val)
    x = np.random.default_rng(1).standard_normal(S.n)
    y = ctx.matvec(K, torch.from_numpy(x).to(ctx.device)).cpu().numpy()
    ref = np.zeros(S.n, dtype=np.longdouble)
    np.add.at(ref, rows, val.astype(np.longdouble) * x[S.col])
    mag = np.zeros(S.n)
    np.add.at(mag, rows, np.abs(val * x[S.col]))
    assert np.all(np.abs(y - ref) <= 16 * np.finfo(float).eps * mag)
    # the solver's gradient reads every stored value: the residual of a
    # one-iteration solve reports |pg| of K c0 - f with K as given
    F = torch.from_numpy(S.F).to(ctx.device)
    c0 = torch.from_numpy(np.abs(x)).to(ctx.device)
    _, _, st = ctx.solve_nonneg(K, F, c=c0.clone(), c0_mode=1, max_outer=0, tol=1e-12, engine=1,
                                allow_maxit=True)
    g = np.zeros(S.n, dtype=np.longdouble)
    np.add.at(g, rows, val.astype(np.longdouble) * np.abs(x)[S.col])
    g = (g - S.F).astype(float)
    want = np.sqrt(np.sum(g * g)) / np.sqrt(np.sum(S.F ** 2))
    assert abs(st["kkt_rel"] - want) <= 1e-12 * want
    K.free()


_SOLO = {f"square_{n}": (lambda n=n: W.square2d(n)) for n in (3, 9, 17, 23, 33, 46, 47, 64, 65)}
_SOLO.update({f"cube_{n}": (lambda n=n: W.cube3d(n)) for n in (4, 9, 11, 12, 14, 15, 17)})
# offsets that reach further than the padding of the vectors in LDS
_SOLO["thin"] = lambda: W.box_problem("thin", (700, 4), 1 / 700, W.aniso2d_tensor())


@pytest.mark.parametrize("name", sorted(_SOLO))
def test_one_workgroup_engine_with_the_matrix_in_registers(ctx, name):
    """One to eight slices per wavefront, 7- and 15-point rows, rows past the
    last one: the same bits and counts as the engine that reads the matrix from
    memory (the same matrix with explicit zeros), for the non-negative problem,
    bounds that exclude zero, bounds on both sides, a warm start and a
    backward-Euler step."""
    import torch
    p = _SOLO[name]()
    K, F, _ = ctx.assemble(p, with_mass=True)
    rp, col, val, mval = ctx.matrix_export(K)
    rpz, colz, (valz, mvalz) = _with_zeros(rp, col, [val, mval], 7, extra=3)
    Z = ctx.matrix_from_csr(rpz, colz, valz, mvalz)
    # (3 x 3 cells hold no source: a load on every row)
    F = F + torch.from_numpy(np.random.default_rng(4).uniform(-0.2, 1.0, K.n) / K.n).to(ctx.device)
    top = float(ctx.solve_nonneg(K, F, tol=1e-8, engine=1)[0].max())
    warm = torch.from_numpy(np.random.default_rng(2).uniform(0, top, K.n)).to(ctx.device)
    for k, kw in enumerate([dict(tol=1e-9, inner_rtol=0.5), dict(tol=1e-9, lower=0.1 * top),
                            dict(tol=1e-9, lower=-0.2 * top, upper=0.5 * top),
                            dict(tol=1e-9, c0_mode=1)]):
        out = []
        for A in (K, Z):
            out.append(ctx.solve_nonneg(A, F, engine=2, c=warm.clone(), allow_maxit=True, **kw))
        (c, a, s), (cz, az, sz) = out
        assert torch.equal(c, cz) and torch.equal(a, az), (name, k)
        for key in ("kkt_rel", "kkt_nat_inf", "min_c", "norm_f", "outer_its", "cg_its", "spmvs",
                    "n_active", "cauchy_trials", "search_trials", "status"):
            assert s[key] == sz[key], (name, k, key)
    c, cz = warm.clone(), warm.clone()
    for _ in range(2):
        ctx.step_transient(K, 1e-3, F, c, tol=1e-9, engine=2)
        ctx.step_transient(Z, 1e-3, F, cz, tol=1e-9, engine=2)
    assert torch.equal(c, cz)
    K.free()
    Z.free()
