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


def _fan(m, every):
    """A free hub with m ring nodes, every `every`-th of them free, inside a
    Dirichlet ring: the hub's row has 1 + ceil(m / every) columns of m
    triangles.  A small square beside it holds ordinary rows."""
    from paper_1506_08435_amd.workloads import Problem
    sq = W.square2d(9)
    a = 2 * np.pi * np.arange(m) / m
    ring = np.stack([np.cos(a), np.sin(a)], 1)
    xy = np.concatenate([sq.coords, [[5.0, 5.0]], 5.0 + ring, 5.0 + 2.0 * ring])
    s = len(sq.coords)
    hub, r0, q0 = s, s + 1, s + 1 + m
    i = np.arange(m)
    j = (i + 1) % m
    el = np.concatenate([
        np.stack([r0 + i, r0 + j, hub + 0 * i], 1),
        np.stack([r0 + i, q0 + i, q0 + j], 1),
        np.stack([q0 + j, r0 + j, r0 + i], 1),
        sq.elems])
    fixed = np.concatenate([sq.dirichlet, [0], (i % every != 0).astype(np.uint8), np.ones(m, np.uint8)])
    rng = np.random.default_rng(m)
    D = np.array([[[2.0, 0.3], [0.3, 1.0]]])
    return Problem(name="fan", dim=2, coords=xy, elems=el.astype(np.int32), D=D,
                   kscale=np.concatenate([rng.uniform(0.5, 2.0, 3 * m),
                                          np.random.default_rng(1).uniform(0.5, 2.0, len(sq.elems))]),
                   f_elem=rng.uniform(-1, 1, len(el)),
                   dirichlet=fixed.astype(np.uint8), cells=(1, 1), h=1.0,
                   dirichlet_values=rng.uniform(0, 1, len(xy)))


# the longest row and the most elements at a node that the device phase takes,
# one more of each, and a hub far past both
@pytest.mark.parametrize("m,every", [(47, 1), (48, 1), (96, 3), (97, 3), (300, 1)])
@pytest.mark.parametrize("mass", [False, True])
def test_assembly_with_a_hub(ctx, m, every, mass):
    """Sums of at most 300 products of float64: within 300 ulp of the largest."""
    p = _fan(m, every)
    K, F, dof = ctx.assemble(p, with_mass=mass)
    S = oracle.assemble(p, with_mass=mass)
    out = ctx.matrix_export(K)
    assert np.array_equal(out[0], S.rowptr) and np.array_equal(out[1], S.col)
    assert np.array_equal(dof, S.dof)
    tol = 300 * np.finfo(np.float64).eps
    assert np.abs(out[2] - S.K).max() <= tol * np.abs(S.K).max()
    if mass:
        assert np.abs(out[3] - S.M).max() <= tol * np.abs(S.M).max()
    assert np.abs(F.cpu().numpy() - S.F).max() <= tol * max(np.abs(S.F).max(), np.abs(S.K).max())
    # rows of the same mesh without the hub: the same bits on either path
    q = _fan(40, 1)
    Q, _, _ = ctx.assemble(q, with_mass=mass)
    qr, qc, qv = ctx.matrix_export(Q)[:3]
    n = int((W.square2d(9).dirichlet == 0).sum())
    k = qr[n]
    assert np.array_equal(out[0][: n + 1], qr[: n + 1]) and np.array_equal(out[1][:k], qc[:k])
    assert np.array_equal(out[2][:k], qv[:k])
    Q.free()
    K.free()


@pytest.mark.parametrize("what", ["node", "coord", "D", "f", "ks", "dval", "order", "none"])
def test_assembly_refusals(ctx, what):
    """Each kind of bad input is refused with its own status, and the node
    ids before everything else; the outcome of a mesh without elements or
    nodes stays what it was."""
    from paper_1506_08435_amd import nnqp
    import dataclasses
    p = W.config_transient3d(5, 4, 3, ell=2.0)
    p = dataclasses.replace(p, coords=p.coords.copy(), elems=p.elems.copy(), D=p.D.copy(),
                            f_elem=p.f_elem.copy(), kscale=np.ones(len(p.elems)),
                            dirichlet=p.dirichlet.copy(), dirichlet_values=np.zeros(len(p.coords)))
    p.dirichlet[0] = 1
    status, text = nnqp.NN_ENONFINITE, None
    if what in ("node", "order"):
        p.elems[-1, 1] = len(p.coords)
        status, text = nnqp.NN_EINVAL, "out of range"
    if what in ("coord", "order"):
        p.coords[-1, 0] = np.nan
        text = text or "coordinate"
    if what == "D":
        p.D[0, 0, 0] = np.inf
        text = "diffusivity"
    if what in ("f", "order"):
        p.f_elem[3] = np.nan
        text = text or "source"
    if what in ("ks", "f"):
        p.kscale[3] = 0.0          # the same element: its source is looked at first
        text = text or "kscale"
    if what == "dval":
        p.dirichlet_values[0] = -np.inf
        text = "Dirichlet"
    if what == "none":
        q = dataclasses.replace(p, elems=p.elems[:0], f_elem=p.f_elem[:0], kscale=p.kscale[:0])
        with pytest.raises(nnqp.NnError) as e:
            ctx.assemble(q)
        assert e.value.status == nnqp.NN_ENOTSPD and "row 0" in str(e.value)
        return
    with pytest.raises(nnqp.NnError) as e:
        ctx.assemble(p)
    assert e.value.status == status and text in str(e.value)


# every memory size the pair pass, the coefficients and the direction are
# compiled for, and more rows than the pair pass has lanes (256 x 1024)
@pytest.mark.parametrize("mesh,m", [("square", m) for m in range(1, 9)] + [("cube", 5)])
def test_blmvm_memories(ctx, mesh, m):
    """Both methods end with |pg| <= 1e-11 |f|: the minimisers differ by at
    most that times the condition number, about n^(2/d) times the anisotropy
    (1e3): 1e-11 * 4e3 * 1e3 * 0.1 (pg is far from the worst direction)."""
    from paper_1506_08435_amd import nnqp
    p = W.square2d(33) if mesh == "square" else W.cube3d(66)
    K, F, _ = ctx.assemble(p)
    ref = ctx.solve_nonneg(K, F, tol=1e-11)[0].cpu().numpy().copy()
    tol = 1e-11 if mesh == "square" else 1e-8
    c, _, st = ctx.solve_nonneg(K, F, tol=tol, method=nnqp.NN_BLMVM, lmm_vectors=m)
    c = c.cpu().numpy()
    assert st["kkt_rel"] <= tol and c.min() >= 0.0
    assert np.abs(c - ref).max() <= (4e-6 if mesh == "square" else 4e-3) * np.abs(ref).max()
    K.free()


# iterations enqueued ahead of the device (solves), steps of a chunk (batch):
# the same bits for any number, with a trust region (early ends) and without
@pytest.mark.parametrize("what", ["tron", "radius", "mixed", "cheb", "galerkin", "batch"])
def test_work_enqueued_ahead_does_not_matter(ctx, what):
    from paper_1506_08435_amd import nnqp
    kw = {"radius": {"delta0": 1e-3}, "mixed": {"precision": nnqp.NN_MIXED},
          "cheb": {"precond_degree": 3}}.get(what, {})
    if what == "batch":
        members = [ctx.assemble(W.batch_problem(i, n_range=(8, 40)))[:2] for i in range(5)]
    else:
        K, F, _ = ctx.assemble(W.cube3d(19))
    got = []
    for chunk in (1, 2, 16, 0):
        if what == "batch":
            c = ctx.solve_batch([m[0] for m in members], [m[1] for m in members], tol=1e-10,
                                cg_chunk=chunk)[0]
            got.append((b"".join(x.cpu().numpy().tobytes() for x in c),))
        elif what == "galerkin":
            c, st = ctx.solve_galerkin(K, F, tol=1e-10, cg_chunk=chunk)[:2]
            got.append((c.cpu().numpy().tobytes(), st["cg_its"], st["spmvs"], st["bytes_moved"]))
        else:
            c, _, st = ctx.solve_nonneg(K, F, tol=1e-10, cg_chunk=chunk, **kw)
            got.append((c.cpu().numpy().tobytes(), st["cg_its"], st["spmvs"], st["search_trials"],
                        st["bytes_moved"], st["n_active"]))
    assert all(g == got[0] for g in got), [g[1:] for g in got]


def test_solves_on_several_threads(ctx):
    """One context, stream and matrix per thread, several solves each at the
    same time: the bits of a solve alone."""
    import threading
    import torch
    from paper_1506_08435_amd import nnqp
    sizes = [21, 24, 27]
    alone = []
    for n in sizes:
        K, F, _ = ctx.assemble(W.cube3d(n))
        alone.append(ctx.solve_nonneg(K, F, tol=1e-10)[0].cpu().numpy().copy())
        K.free()
    got, errors = {}, []

    def work(i):
        try:
            c = nnqp.Context(0, stream=torch.cuda.Stream(0))
            K, F, _ = c.assemble(W.cube3d(sizes[i]))
            got[i] = [c.solve_nonneg(K, F, tol=1e-10)[0].cpu().numpy().copy() for _ in range(4)]
            K.free()
            c.close()
        except Exception as e:   # noqa: BLE001 (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i in range(3):
        assert all(np.array_equal(x, alone[i]) for x in got[i]), i


@pytest.mark.parametrize("what", ["galerkin", "blmvm", "one"])
def test_solves_without_the_copies(what):
    """Solves that read a matrix's copies only for speed: with every further
    allocation refused a fresh matrix is solved from its sliced-ELL arrays, to
    the same bits."""
    import torch
    from paper_1506_08435_amd import nnqp
    refuse = [False]

    def alloc(nbytes):
        if refuse[0]:
            return None
        return torch.cuda.caching_allocator_alloc(nbytes, 0, torch.cuda.current_stream(0))

    c = nnqp.Context(0, allocator=(alloc, torch.cuda.caching_allocator_delete))
    p = W.cube3d(10 if what == "one" else 20)

    def solve(K, F):
        if what == "galerkin":
            return c.solve_galerkin(K, F, tol=1e-10)[0].cpu().numpy().copy()
        kw = {"method": nnqp.NN_BLMVM} if what == "blmvm" else {}
        return c.solve_nonneg(K, F, tol=1e-10, **kw)[0].cpu().numpy().copy()

    K1, F1, _ = c.assemble(p)
    K2, F2, _ = c.assemble(p)
    a = solve(K1, F1)
    refuse[0] = True
    b = solve(K2, F2)
    assert np.array_equal(a, b)
    refuse[0] = False
    assert np.array_equal(a, solve(K2, F2))
    K1.free()
    K2.free()
    c.close()
