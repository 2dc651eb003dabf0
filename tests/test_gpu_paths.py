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
