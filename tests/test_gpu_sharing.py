"""One matrix read by several contexts, each on its thread and stream."""
import threading

import numpy as np
import pytest

from paper_1506_08435_amd import workloads as W

pytestmark = pytest.mark.gpu


def _call(nnqp, what, c, K, F):
    import torch
    kw = dict(tol=1e-10)
    if what == "galerkin":
        return c.solve_galerkin(K, F, **kw)[0]
    if what == "step":
        c0 = torch.zeros(K.n, dtype=torch.float64, device=c.device)
        torch.cuda.current_stream(0).synchronize()
        return c.step_transient(K, 1e-3, F, c0, **kw)[0]
    if what in ("batch", "batch_mixed"):
        if what == "batch_mixed":
            kw.update(precision=nnqp.NN_MIXED)
        return c.solve_batch([K], [F], **kw)[0][0]
    if what == "blmvm":
        kw.update(method=nnqp.NN_BLMVM)
    if what == "mixed":
        kw.update(precision=nnqp.NN_MIXED)
    return c.solve_nonneg(K, F, **kw)[0]


# what a solve adds to a matrix (copies, layout, transient values) is formed by
# whichever of the threads comes first and read by all
@pytest.mark.parametrize("what", ["galerkin", "blmvm", "one", "tron", "mixed", "step", "batch", "batch_mixed"])
def test_first_solves_of_a_matrix_on_several_threads(what):
    import torch
    from paper_1506_08435_amd import nnqp
    p = W.cube3d(14 if what == "one" else 20)
    home = nnqp.Context(0)
    streams = [torch.cuda.Stream(0) for _ in range(3)]
    ctxs = [nnqp.Context(0, stream=s) for s in streams]
    K, F, _ = home.assemble(p, with_mass=True)
    alone = _call(nnqp, what, home, K, F).cpu().numpy().copy()
    K.free()
    for _ in range(3):
        K, F, _ = home.assemble(p, with_mass=True)
        torch.cuda.synchronize()
        gate, got, errors = threading.Barrier(3), {}, []

        def work(i):
            try:
                with torch.cuda.stream(streams[i]):
                    gate.wait()
                    c = _call(nnqp, what, ctxs[i], K, F)
                    streams[i].synchronize()
                    got[i] = c.cpu().numpy().copy()
            except Exception as e:   # noqa: BLE001 (reported by the main thread)
                errors.append(e)

        threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        assert all(np.array_equal(got[i], alone) for i in range(3))
        K.free()
    for c in ctxs:
        c.close()
    home.close()


# a context on a stream of its own, tensors of the current stream with work
# still queued on them: the call starts behind that work
@pytest.mark.parametrize("what", ["warm start", "load", "product", "zeros", "assembly", "batch"])
def test_calls_start_behind_the_callers_stream(what):
    import torch
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0, stream=torch.cuda.Stream(0))
    p = W.cube3d(18)
    K, F, _ = c.assemble(p)
    rng = np.random.default_rng(3)
    host = torch.from_numpy(rng.uniform(0.0, 1e-3, K.n)).pin_memory()
    late = torch.empty(K.n, dtype=torch.float64, device=c.device)
    kw = dict(tol=1e-10)

    def call(x, wait):
        if what == "assembly":
            # F is made by the call on the block that `x` gives back
            if wait:
                torch.cuda.synchronize()
            del x
            A, G, _ = c.assemble(p)
            A.free()
            return G
        if wait:
            torch.cuda.synchronize()
        if what == "warm start":
            return c.solve_nonneg(K, F, c=x, c0_mode=1, **kw)[0]
        if what == "load":
            return c.solve_nonneg(K, x, **kw)[0]
        if what == "product":
            return c.matvec(K, x) * 2.0        # read on the current stream
        if what == "batch":
            return c.solve_batch([K], [x], **kw)[0][0]
        return c.solve_nonneg(K, F, **kw)[0]   # zeros made by the call

    out = []
    for wait in (True, False):
        late.fill_(0.5)
        torch.cuda.synchronize()
        torch.cuda._sleep(100_000_000)         # some 50 ms at 2 GHz
        late.copy_(host, non_blocking=True)
        x = late if what != "assembly" else torch.full((K.n,), 0.25, dtype=torch.float64, device=c.device)
        y = call(x, wait)
        out.append(y.cpu().numpy().copy())
        del x, y
    assert np.array_equal(*out)
    K.free()
    c.close()


def _entries(c, K):
    """Stored sliced-ELL entries of a matrix: slices of 64 rows as wide as their
    longest row."""
    n = np.diff(c.matrix_export(K)[0])
    return sum(64 * int(n[a:a + 64].max()) for a in range(0, K.n, 64))


# a solve in float64 adds the float64 copy (10 bytes an entry) and no other
@pytest.mark.parametrize("what", ["galerkin", "blmvm", "one", "tron"])
def test_float64_solves_make_no_float32_copy(what):
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0)
    K, F, _ = c.assemble(W.cube3d(14 if what == "one" else 20))
    c.solve_batch([K], [F], tol=1e-8, precision=nnqp.NN_MIXED)   # float32 values are there
    before = K.bytes()
    _call(nnqp, what, c, K, F)
    assert K.bytes() - before == 10 * _entries(c, K)
    K.free()
    c.close()


def test_one_workgroup_engine_copies_what_it_reads():
    """A small matrix without the diagonal layout (explicit zeros at random
    columns) is solved from its sliced-ELL arrays and takes no further memory;
    a multi-block solve adds the pairs, and the engine's result stays."""
    from paper_1506_08435_amd import nnqp
    from test_gpu_paths import _with_zeros
    c = nnqp.Context(0)
    K, F, _ = c.assemble(W.cube3d(12))
    rp, col, val, _ = c.matrix_export(K)
    rpz, colz, (valz,) = _with_zeros(rp, col, [val], 3, extra=3)
    Z = c.matrix_from_csr(rpz, colz, valz)
    before = Z.bytes()
    a = c.solve_nonneg(Z, F, tol=1e-10, engine=2)[0].cpu().numpy().copy()
    assert Z.bytes() == before
    c.solve_nonneg(Z, F, tol=1e-10, engine=1)
    assert Z.bytes() - before == 10 * _entries(c, Z)
    b = c.solve_nonneg(Z, F, tol=1e-10, engine=2)[0].cpu().numpy().copy()
    k = c.solve_nonneg(K, F, tol=1e-10, engine=2)[0].cpu().numpy().copy()
    assert np.array_equal(a, b) and np.array_equal(a, k)
    K.free()
    Z.free()
    c.close()


def test_float64_and_mixed_steps_of_one_matrix_at_the_same_time():
    """Steps at the same dt in both precisions: whichever precision comes second
    forms only what is missing while the first is reading."""
    import torch
    from paper_1506_08435_amd import nnqp
    p = W.cube3d(24)
    precs = [nnqp.NN_FP64, nnqp.NN_MIXED, nnqp.NN_FP64, nnqp.NN_MIXED]
    home = nnqp.Context(0)
    streams = [torch.cuda.Stream(0) for _ in precs]
    ctxs = [nnqp.Context(0, stream=s) for s in streams]

    def steps(c, K, F, prec, n):
        u = torch.zeros(K.n, dtype=torch.float64, device=c.device)
        for _ in range(n):
            c.step_transient(K, 1e-3, F, u, tol=1e-9, precision=prec)
        return u.cpu().numpy().copy()

    K, F, _ = home.assemble(p, with_mass=True)
    alone = {prec: steps(home, K, F, prec, 6) for prec in set(precs)}
    K.free()
    for _ in range(3):
        K, F, _ = home.assemble(p, with_mass=True)
        torch.cuda.synchronize()
        gate, got, errors = threading.Barrier(len(precs)), {}, []

        def work(i):
            try:
                with torch.cuda.stream(streams[i]):
                    gate.wait()
                    got[i] = steps(ctxs[i], K, F, precs[i], 6)
            except Exception as e:   # noqa: BLE001 (reported by the main thread)
                errors.append(e)

        threads = [threading.Thread(target=work, args=(i,)) for i in range(len(precs))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        assert all(np.array_equal(got[i], alone[precs[i]]) for i in range(len(precs)))
        K.free()
    for c in ctxs:
        c.close()
    home.close()


def test_transient_copies_of_several_time_steps():
    """Single, mixed and batched steps that change dt between them: every copy is
    formed anew for the dt it is read at (the bits of a fresh matrix)."""
    import torch
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0)
    p = W.cube3d(12)
    K, F, _ = c.assemble(p, with_mass=True)
    plan = [("fp64", 1e-3), ("mixed", 1e-3), ("fp64", 2e-3), ("mixed", 1e-3), ("batch", 4e-3), ("fp64", 4e-3),
            ("mixed", 4e-3), ("batch_mixed", 1e-3), ("blmvm", 1e-3), ("mixed", 2e-3), ("fp64", 2e-3)]

    def step(A, what, dt):
        u = torch.zeros(A.n, dtype=torch.float64, device=c.device)
        kw = dict(tol=1e-8, precision=nnqp.NN_MIXED if "mixed" in what else nnqp.NN_FP64, engine=1)
        if what == "blmvm":
            kw.update(method=nnqp.NN_BLMVM)
        if "batch" in what:
            c.step_transient_batch([A], dt, [F], [u], **kw)
        else:
            c.step_transient(A, dt, F, u, **kw)
        return u.cpu().numpy().copy()

    for what, dt in plan:
        fresh, _, _ = c.assemble(p, with_mass=True)
        assert np.array_equal(step(K, what, dt), step(fresh, what, dt)), (what, dt)
        fresh.free()
    K.free()
    c.close()


def test_memory_hooks_may_ask_for_the_matrix_size():
    """The hooks run while the library forms a copy: a hook that looks at the
    matrix's reported bytes (to account for them) gets an answer."""
    import torch
    from paper_1506_08435_amd import nnqp
    at, seen = [None], []

    def alloc(nbytes):
        if at[0] is not None:
            seen.append(at[0].bytes())
        return torch.cuda.caching_allocator_alloc(nbytes, 0, torch.cuda.current_stream(0))

    c = nnqp.Context(0, allocator=(alloc, torch.cuda.caching_allocator_delete))
    K, F, _ = c.assemble(W.cube3d(18))
    at[0] = K
    c.solve_nonneg(K, F, tol=1e-8)
    c.solve_batch([K], [F], tol=1e-8, precision=nnqp.NN_MIXED)
    c.solve_nonneg(K, F, tol=1e-8, precision=nnqp.NN_MIXED)
    at[0] = None
    assert seen and seen[-1] > seen[0]
    K.free()
    c.close()
