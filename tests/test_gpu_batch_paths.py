"""The batched solver's layouts and sizes of members, through the C ABI."""
import numpy as np
import pytest

from paper_1506_08435_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1506_08435_amd import nnqp
    c = nnqp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_without_room_to_look_for_the_layout(precision):
    """The scratch that the search for the diagonal layout asks for is refused:
    the batch runs in another layout, to the same bits, and the refusal leaves
    nothing behind."""
    import torch
    from paper_1506_08435_amd import nnqp
    refuse, seen = [0], []

    def alloc(nbytes):
        refuse[0] -= 1
        if refuse[0] == 0:
            seen.append(nbytes)
            return None
        return torch.cuda.caching_allocator_alloc(nbytes, 0, torch.cuda.current_stream(0))

    c = nnqp.Context(0, allocator=(alloc, torch.cuda.caching_allocator_delete))
    probs = [W.square2d(40), W.square2d(33), W.square2d(21)]
    kw = dict(tol=1e-10, precision=nnqp.NN_MIXED if precision == "mixed" else nnqp.NN_FP64)

    def solve(first):
        Ks, Fs = zip(*[c.assemble(p)[:2] for p in probs])
        out = []
        for k in range(2):
            # the call's first allocation behind the members' float32 values
            refuse[0] = 1 + (len(probs) if precision == "mixed" else 0) if first and k == 0 else 0
            cs, acts, _, rc = c.solve_batch(list(Ks), list(Fs), **kw)
            assert rc == 0 and c.last_error() == ""
            out.append([x.cpu().numpy().copy() for x in cs] + [x.cpu().numpy().copy() for x in acts])
        for K in Ks:
            K.free()
        return out

    want = solve(False)[0]
    assert not seen
    for got in solve(True):
        assert all(np.array_equal(u, w) for u, w in zip(got, want))
    assert len(seen) == 1
    c.close()


def _slices(K):
    return (K.n + 63) // 64


# members on both sides of the size from which a launch of its own sums their
# partials (3,584 slices): alone and side by side, the same bits; a bounded
# problem, a mixed one and two steps
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_large_members_alone_and_together(ctx, precision):
    import torch
    from paper_1506_08435_amd import nnqp
    probs = [W.square2d(300), W.cube3d(62), W.square2d(481), W.cube3d(65), W.square2d(23)]
    Ks, Fs = zip(*[ctx.assemble(p, with_mass=True)[:2] for p in probs])
    n = [_slices(K) for K in Ks]
    assert n[0] < n[1] < 3584 < n[2] < n[3] and n[4] < 64, n
    top = [float(ctx.solve_nonneg(K, F, tol=1e-8)[0].max()) for K, F in zip(Ks, Fs)]
    kw = dict(tol=1e-8, inner_rtol=0.3, precision=nnqp.NN_MIXED if precision == "mixed" else nnqp.NN_FP64)
    for extra in ({}, dict(upper=0.6 * max(top), delta0=1.0)):
        cs, acts, sts, rc = ctx.solve_batch(list(Ks), list(Fs), **kw, **extra)
        for K, F, c, a, s in zip(Ks, Fs, cs, acts, sts):
            c1, a1, s1, _ = ctx.solve_batch([K], [F], **kw, **extra)
            assert torch.equal(c, c1[0]) and torch.equal(a, a1[0])
            assert all(s[k] == s1[0][k] for k in ("kkt_rel", "cg_its", "outer_its", "spmvs", "min_c", "norm_f"))
            assert s["kkt_rel"] <= 1e-8
    steps = [[torch.zeros(K.n, dtype=torch.float64, device=ctx.device) for K in Ks] for _ in range(2)]
    for _ in range(2):
        ctx.step_transient_batch(list(Ks), 1e-3, list(Fs), steps[0], **kw)
        for K, F, c in zip(Ks, Fs, steps[1]):
            ctx.step_transient_batch([K], 1e-3, [F], [c], **kw)
    assert all(torch.equal(u, w) for u, w in zip(*steps))
    for K in Ks:
        K.free()


# the sums that the large members' transitions read have a closed form for a
# diagonal matrix, as in the single-problem solver (one slice past the line, a
# remainder of the sixteen loads in flight, and many times it)
@pytest.mark.parametrize("slices", [3584, 3585, 4097, 20000])
def test_large_diagonal_member(ctx, slices):
    import torch
    n = 64 * slices - 17
    rng = np.random.default_rng(slices)
    k, f = rng.uniform(0.5, 2.0, n), rng.uniform(-1.0, 1.0, n)
    K = ctx.matrix_from_csr(np.arange(n + 1), np.arange(n, dtype=np.int32), k)
    F = torch.from_numpy(f).to(ctx.device)
    cs, acts, sts, rc = ctx.solve_batch([K], [F], tol=1e-12)
    c, st = cs[0].cpu().numpy(), sts[0]
    eps = np.finfo(float).eps
    nf = float(np.sqrt(np.sum(f.astype(np.longdouble) ** 2)))
    assert rc == 0 and st["kkt_rel"] <= 1e-12
    assert abs(st["norm_f"] - nf) <= n * eps * nf
    # |c - ref| <= |g| / k, |g| <= tol |f|
    assert np.abs(c - np.maximum(f, 0.0) / k).max() <= 2.1e-12 * nf
    assert st["n_active"] == int((c == 0.0).sum()) == int((acts[0].cpu().numpy() == 1).sum())
    assert np.all(c[f <= 0.0] == 0.0) and st["min_c"] == c.min()
    K.free()


# new members are looked over together: more of them than get a wavefront per
# slice each, one matrix twice, and one without the layout among them (nobody
# has it then)
@pytest.mark.parametrize("what", ["many", "twice", "other"])
def test_new_members_are_looked_over_together(ctx, what):
    import torch
    small = W.square2d(17)
    probs = {"many": [small] * 1030 + [W.square2d(300)], "twice": [small, W.square2d(40)],
             "other": [small, W.square2d(9), W.square2d(40)]}[what]
    Ks, Fs = map(list, zip(*[ctx.assemble(p)[:2] for p in probs]))
    if what == "twice":
        Ks, Fs = Ks + Ks, Fs + [2.0 * F for F in Fs]
    kw = dict(tol=1e-9, inner_rtol=0.3)
    cs, _, sts, rc = ctx.solve_batch(Ks, Fs, **kw)
    again = ctx.solve_batch(Ks, Fs, **kw)[0]
    assert rc == 0 and all(torch.equal(u, w) for u, w in zip(cs, again))
    for k, K in enumerate(Ks):
        if what == "many" and 3 <= k < 1030:
            assert torch.equal(cs[k], cs[0])
            continue
        assert torch.equal(cs[k], ctx.solve_batch([K], [Fs[k]], **kw)[0][0])
    # a gradient pass reports the layout: 10 bytes an entry in pairs, fewer here
    st = ctx.solve_batch(Ks, Fs, tol=1e-15, max_outer=0, allow_fail=True)[2]
    per = [(s["bytes_moved"] - 4.0 * (K.n + 1) - 48.0 * K.n) / K.nnz for K, s in zip(Ks, st)]
    assert all(x == 10.0 if what == "other" else x < 9.0 for x in per), per
    for K in set(map(id, Ks)):
        next(k for k in Ks if id(k) == K).free()
