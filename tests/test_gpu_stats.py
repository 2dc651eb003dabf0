"""What a solve reports of its work, against the launches that were timed."""
import pytest

from paper_1506_08435_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_every_search_pass_is_counted():
    """The matrix passes of the projected search, from the products reported
    (all of them, less gradients, CG and Cauchy trials) and from the timed
    launches of the class (less the ladders and the single Cauchy trials): the
    same, also where a first trial was made that was not needed."""
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0)
    surplus = 0
    for p in (W.cube3d(20), W.cube3d(27), W.square2d(60), W.square2d(120), W.cube_hole(3)):
        K, F, _ = c.assemble(p)
        for kw in (dict(inner_rtol=0.5), dict(inner_rtol=0.1), dict(inner_rtol=0.5, precision=nnqp.NN_MIXED),
                   dict(inner_rtol=0.1, lower=-10.0)):   # (no bound is reached: no search)
            kw = dict(tol=1e-9, engine=1, lower=p.bounds[0], upper=p.bounds[1]) | kw
            c.solve_nonneg(K, F, **kw)
            c.set_profiling(True, classes=["grad", "trial"])
            c.kernel_times(reset=True)
            st = c.solve_nonneg(K, F, **kw)[2]
            t = c.kernel_times(reset=True)
            c.set_profiling(False)
            ladders = st["outer_its"] + 1
            assert t["grad"]["count"] == ladders
            singles = st["cauchy_trials"] - 3 * st["outer_its"]
            passes = t["trial"]["count"] - ladders - singles
            assert st["spmvs"] - ladders - st["cg_its"] - st["cauchy_trials"] == passes
            assert passes >= st["search_trials"]
            surplus += passes - st["search_trials"]
        K.free()
    assert surplus > 0
    c.close()


def test_more_iterations_enqueued_ahead_than_a_solve_has():
    """cg_chunk far beyond the iterations of any CG solve, and the launches past
    its end: the same bits and counts."""
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0)
    K, F, _ = c.assemble(W.cube3d(19))
    for kw in ({}, {"delta0": 1e-3}, {"precision": nnqp.NN_MIXED}, {"precond_degree": 3}):
        a, b = (c.solve_nonneg(K, F, tol=1e-10, engine=1, cg_chunk=k, **kw) for k in (2, 300))
        assert (a[0] == b[0]).all() and all(a[2][k] == b[2][k] for k in ("cg_its", "spmvs", "outer_its"))
    K.free()
    c.close()
