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
        if refuse[0] and nbytes == refuse[0]:
            refuse[0] = 0
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
            # 2 bytes per stored entry of the largest member (rows in slices of 64, 7 entries)
            refuse[0] = 2 * 7 * ((Ks[0].n + 63) // 64 * 64) if first and k == 0 else 0
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
