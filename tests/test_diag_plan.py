"""The host side of the diagonal layout: whatever pattern a plan is made for, a
product read through it is the matrix's, and no index leaves an array (on the
CPU, diag_plan_check.cpp)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_1506_08435_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1506_08435_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("diag") / "libdiagplan.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-ffp-contract=off", "-Wall", "-Werror",
                    "-I", CSRC, "-o", out, os.path.join(HERE, "diag_plan_check.cpp")], check=True)
    return ctypes.CDLL(out)


def _layout(lib, n, rp, col, val, x):
    """(outcome, product, product of one run, info) of diag_product."""
    rp, col, val, x = (np.ascontiguousarray(a, dtype=t) for a, t in
                       ((rp, np.int64), (col, np.int32), (val, np.float64), (x, np.float64)))
    y, y1, info = np.full(n, np.nan), np.full(n, np.nan), np.zeros(3, np.int64)
    p = [a.ctypes.data_as(ctypes.c_void_p) for a in (rp, col, val, x, y, y1, info)]
    return lib.diag_product(ctypes.c_int64(n), *p), y, y1, info


def _csr(n, pairs, rng):
    """Symmetric CSR with the diagonal and random values at the (i, j), i < j."""
    a = np.unique(np.asarray(sorted(pairs), dtype=np.int64).reshape(-1, 2), axis=0)
    v = rng.standard_normal(len(a))
    i = np.concatenate([a[:, 0], a[:, 1], np.arange(n)])
    j = np.concatenate([a[:, 1], a[:, 0], np.arange(n)])
    w = np.concatenate([v, v, rng.uniform(1, 2, n)])
    o = np.lexsort((j, i))
    return np.concatenate([[0], np.cumsum(np.bincount(i, minlength=n))]), j[o], w[o]


def _check(lib, n, rp, col, val, seed=0):
    x = np.random.default_rng(seed).standard_normal(n)
    got, y, y1, info = _layout(lib, n, rp, col, val, x)
    assert got >= 0, got
    if got == 0:
        return got, info
    # a sum of w fused multiply-adds is within w eps of the exact one
    rows = np.repeat(np.arange(n), np.diff(rp))
    ref = np.zeros(n, np.longdouble)
    np.add.at(ref, rows, val.astype(np.longdouble) * x[col])
    mag = np.zeros(n)
    np.add.at(mag, rows, np.abs(val * x[col]))
    w = int(np.diff(rp).max())
    for z in (y, y1) if got == 2 else (y,):
        assert np.all(np.abs(z - ref) <= 2 * w * np.finfo(float).eps * mag)
    return got, info


_MESH = {
    "square_33": lambda: W.square2d(33), "square_65": lambda: W.square2d(65), "square_100": lambda: W.square2d(100),
    "cube_12": lambda: W.cube3d(12), "cube_21": lambda: W.cube3d(21), "slab": lambda: W.config_transient3d(20, 18, 9),
}


@pytest.mark.parametrize("name", sorted(_MESH))
def test_grid_numberings_have_one_run(lib, name):
    S = oracle.assemble(_MESH[name]())
    got, info = _check(lib, S.n, S.rowptr, S.col, S.K)
    assert got == 2 and info[1] == info[2] == (S.n + 63) // 64


@pytest.mark.parametrize("k", [3, 4])
def test_numbering_that_shifts_has_several_runs(lib, k):
    S = oracle.assemble(W.cube_hole(k))
    got, info = _check(lib, S.n, S.rowptr, S.col, S.K)
    assert got == 1 and info[0] > 3


@pytest.mark.parametrize("name,p", [("square_9", W.square2d(9)), ("cube_5", W.cube3d(5))])
def test_arrays_longer_than_the_matrix_are_refused(lib, name, p):
    S = oracle.assemble(p)
    assert _check(lib, S.n, S.rowptr, S.col, S.K)[0] == 0


def _band_then_grid(reach):
    """A band (offsets +-1, +-2) whose last slice reaches into a grid (7-point
    rows) at two offsets: the band's run has seven offsets, none of them the
    opposite of those two."""
    n1, side = 64 * 4, 60
    n = n1 + side * side
    pairs = [(i, i + d) for i in range(n1) for d in (1, 2) if i + d < n1]
    at = n1 + np.arange(side * side).reshape(side, side)
    pairs += list(zip(at[:, :-1].ravel(), at[:, 1:].ravel())) + list(zip(at[:-1].ravel(), at[1:].ravel()))
    pairs += list(zip(at[:-1, :-1].ravel(), at[1:, 1:].ravel()))
    pairs += [(n1 - 1, n1 - 1 + r) for r in reach]
    return n, pairs


@pytest.mark.parametrize("reach", [(70, 90), (65, 1000)])
def test_run_that_reaches_into_the_next_one(lib, reach):
    n, pairs = _band_then_grid(reach)
    rp, col, val = _csr(n, pairs, np.random.default_rng(1))
    assert _check(lib, n, rp, col, val)[0] == 1


def test_joined_stencils(lib):
    """Segments of different stencils (2D and 3D rows, bands, a numbering that
    changes its stride) one behind the other, with couplings across."""
    seen = {0: 0, 1: 0, 2: 0}
    for seed in range(400):
        rng = np.random.default_rng(seed)
        half = int(rng.choice([3, 7]))
        pairs, a = [], 0
        for _ in range(int(rng.integers(1, 5))):
            m = int(rng.integers(1, 30)) * 64 + (int(rng.integers(0, 64)) if rng.random() < 0.5 else 0)
            k = half if rng.random() < 0.7 else int(rng.integers(1, half + 1))
            h = np.unique(rng.integers(1, int(rng.choice([8, 70, 300])), size=k))
            for d in h:
                i = np.arange(a, a + m)
                i = i[rng.random(m) < rng.choice([1.0, 0.9])]
                cross = rng.random() < 0.5
                pairs += [(p, p + d) for p in i if cross or p + d < a + m]
            a += m
            for _ in range(int(rng.integers(0, 3))):   # single couplings
                i = int(rng.integers(0, a))
                pairs.append((i, i + int(rng.integers(1, 200))))
        n = a
        pairs = [p for p in pairs if p[1] < n]
        rp, col, val = _csr(n, pairs, rng)
        seen[_check(lib, n, rp, col, val, seed)[0]] += 1
    assert seen[1] > 20 and seen[2] > 20, seen


def test_unequal_pair_is_refused(lib):
    S = oracle.assemble(W.square2d(33))
    val = S.K.copy()
    rows = np.repeat(np.arange(S.n), np.diff(S.rowptr))
    k = np.flatnonzero(rows == S.col + 1)[500]
    val[k] = np.nextafter(val[k], 0.0)
    assert _layout(lib, S.n, S.rowptr, S.col, val, np.ones(S.n))[0] == 0
