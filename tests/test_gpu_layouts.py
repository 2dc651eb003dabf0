"""Which layout of the matrix a solve reads, and the same bits from each."""
import numpy as np
import pytest

from paper_1506_08435_amd import workloads as W
from test_diag_plan import _band_then_grid, _csr
from test_gpu_paths import _DIAG, _SOLO, _with_zeros

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0)
    yield c
    c.close()


def _read(n, nnz, moved, ends):
    """Layout from the bytes per stored entry of one gradient pass: `moved` of a
    solve that stops at its first gradient, less `ends` bytes a row."""
    per = (moved - 4.0 * (n + 1) - ends * n) / nnz
    return {10.0: "pairs", 12.0: "int32"}.get(round(per, 9), "diagonal" if per < 9.9 else per)


def _layout(ctx, K, F):
    st = ctx.solve_nonneg(K, F, tol=1e-14, max_outer=0, engine=1, allow_maxit=True)[2]
    return _read(K.n, K.nnz, st["bytes_moved"], 48.0)


# too few rows for the arrays; two planes of a grid, whose rows have no common
# offsets (and columns past int16)
_OTHER = {"square_3": "pairs", "square_9": "pairs", "cube_4": "pairs", "cube_5": "pairs", "wide": "int32"}


@pytest.mark.parametrize("name", sorted({**_DIAG, **_SOLO}))
def test_layout_of_the_bitwise_cases(ctx, name):
    """The matrices that test_gpu_paths compares bitwise have the layout that
    their comparison is about, and the matrix with explicit zeros has not."""
    import torch
    K, F, _ = ctx.assemble({**_DIAG, **_SOLO}[name]())
    F = torch.ones_like(F)
    assert _layout(ctx, K, F) == _OTHER.get(name, "diagonal")
    rp, col, val, _ = ctx.matrix_export(K)
    rpz, colz, (valz,) = _with_zeros(rp, col, [val], 5)
    Z = ctx.matrix_from_csr(rpz, colz, valz)
    assert _layout(ctx, Z, F) in ("pairs", "int32")
    K.free()
    Z.free()


def _same_bits(ctx, K, Z, F, precision):
    """Every kind of solve on two forms of one matrix, steps at two time steps
    (the transient values formed, formed anew and formed back)."""
    import torch
    from paper_1506_08435_amd import nnqp
    kw = dict(tol=1e-8, inner_rtol=0.3, engine=1,
              precision=nnqp.NN_MIXED if precision == "mixed" else nnqp.NN_FP64)
    calls = [lambda A: ctx.solve_nonneg(A, F, **kw)[:2],
             lambda A: ctx.solve_nonneg(A, F, **kw, precond_degree=3)[:2],
             lambda A: ctx.solve_nonneg(A, F, **kw, subspace=1)[:2]]
    if K.has_mass:
        def steps(A):
            c = torch.zeros(K.n, dtype=torch.float64, device=ctx.device)
            return [ctx.step_transient(A, dt, F, c, **kw)[0].clone() for dt in (1e-3, 2e-3, 1e-3)]
        calls.append(steps)
    if precision == "fp64":
        calls += [lambda A: ctx.solve_nonneg(A, F, tol=1e-6, method=nnqp.NN_BLMVM)[:2],
                  lambda A: ctx.solve_galerkin(A, F, tol=1e-8, max_cg=20000)[:1]]
        if K.has_mass:
            def lm_steps(A):
                c = torch.zeros(K.n, dtype=torch.float64, device=ctx.device)
                return [ctx.step_transient(A, dt, F, c, tol=1e-8, method=nnqp.NN_BLMVM)[0].clone()
                        for dt in (1e-3, 2e-3)]
            calls.append(lm_steps)
    for k, call in enumerate(calls):
        for u, w in zip(call(K), call(Z)):
            assert torch.equal(u, w), (k, (u != w).sum().item())


# columns past int16 with the diagonal layout (one run, its planes wider than
# the offsets); a numbering that shifts: runs past row 0, mirrored
@pytest.mark.parametrize("name,p", [("wide", lambda: W.box_problem("wide", (185, 185, 12), 1 / 185, W.aniso3d_tensor())),
                                    ("hole_4", lambda: W.cube_hole(4))])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_runs_and_far_columns_keep_the_bits(ctx, name, p, precision):
    K, F, _ = ctx.assemble(p(), with_mass=True)
    rp, col, val, mval = ctx.matrix_export(K)
    far = int(np.abs(col - np.repeat(np.arange(K.n), np.diff(rp))).max()) > 32767
    assert far == (name == "wide")
    rpz, colz, (valz, mvalz) = _with_zeros(rp, col, [val, mval], 5)
    Z = ctx.matrix_from_csr(rpz, colz, valz, mvalz)
    assert _layout(ctx, K, F) == "diagonal" and _layout(ctx, Z, F) == "int32"
    _same_bits(ctx, K, Z, F, precision)
    K.free()
    Z.free()


@pytest.mark.parametrize("reach", [(70, 90), (65, 1000)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_run_that_reaches_into_the_next_one(ctx, reach, precision):
    """A band coupled to a grid: seven offsets that are not symmetric are no
    regular rows."""
    import torch
    n, pairs = _band_then_grid(reach)
    rp, col, val = _csr(n, pairs, np.random.default_rng(2))
    rows = np.repeat(np.arange(n), np.diff(rp))
    val = -np.abs(val)
    val[rows == col] = 0.0
    val[rows == col] = 1e-3 - np.bincount(rows, val, minlength=n)
    K = ctx.matrix_from_csr(rp, col, val)
    rpz, colz, (valz,) = _with_zeros(rp, col, [val], 5)
    Z = ctx.matrix_from_csr(rpz, colz, valz)
    F = torch.from_numpy(np.random.default_rng(3).uniform(-0.5, 1.0, n)).to(ctx.device)
    assert _layout(ctx, K, F) == "diagonal" and _layout(ctx, Z, F) != "diagonal"
    _same_bits(ctx, K, Z, F, precision)
    K.free()
    Z.free()


# one ulp between an entry and its opposite: every stored value counts, also
# where only the capacity matrix has such a pair
@pytest.mark.parametrize("which", ["K", "M"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_one_ulp_off_the_opposite_entry(ctx, which, precision):
    p = W.cube3d(12)
    K0, F, _ = ctx.assemble(p, with_mass=True)
    assert _layout(ctx, K0, F) == "diagonal"
    rp, col, val, mval = ctx.matrix_export(K0)
    rows = np.repeat(np.arange(K0.n), np.diff(rp))
    v = val if which == "K" else mval
    at = np.flatnonzero((rows == col + 1) & (v != 0.0))[500]
    v[at] = np.nextafter(v[at], 1.0)
    K = ctx.matrix_from_csr(rp, col, val, mval)
    rpz, colz, (valz, mvalz) = _with_zeros(rp, col, [val, mval], 5)
    Z = ctx.matrix_from_csr(rpz, colz, valz, mvalz)
    assert _layout(ctx, K, F) == "pairs"
    _same_bits(ctx, K, Z, F, precision)
    for A in (K0, K, Z):
        A.free()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_layouts_keep_the_bits(ctx, precision):
    """The same members in a batch where all have the diagonal layout, beside a
    member without it (pairs of float64 values, quads of float32), and beside one
    without int16 offsets (int32): equal bits, solves and steps at two dt."""
    import torch
    from paper_1506_08435_amd import nnqp
    kw = dict(tol=1e-9, inner_rtol=0.3, precision=nnqp.NN_MIXED if precision == "mixed" else nnqp.NN_FP64)
    names = [W.square2d(40), W.square2d(33), W.cube3d(9), W.cube3d(17), W.square2d(65)]
    beside = {"diagonal": [], "pairs": [W.square2d(9)],
              "int32": [W.box_problem("wide", (200, 170, 3), 1 / 200, W.aniso3d_tensor())]}
    m, want = len(names), None
    for layout, more in beside.items():
        Ks, Fs = map(list, zip(*[ctx.assemble(p, with_mass=True)[:2] for p in names + more]))
        st = ctx.solve_batch(Ks, Fs, allow_fail=True, **{**kw, "tol": 1e-15, "max_outer": 0})[2]
        assert [_read(K.n, K.nnz, s["bytes_moved"], 48.0) for K, s in zip(Ks[:m], st)] == [layout] * m
        got = list(ctx.solve_batch(Ks, Fs, **kw)[0][:m])
        cs = [torch.zeros(K.n, dtype=torch.float64, device=ctx.device) for K in Ks]
        for dt in (1e-3, 2e-3):
            ctx.step_transient_batch(Ks, dt, Fs, cs, **kw)
            got += [c.clone() for c in cs[:m]]
        if want is None:
            want = got
        assert all(torch.equal(u, w) for u, w in zip(got, want)), layout
        for K in Ks:
            K.free()
