"""Dense adjoints under capture: after uncaptured calls of the same sizes, whichever
gradients those asked for, a capture takes any set of gradients; a replay gives the
uncaptured call's bits, also when a larger call has grown the scratch since."""
import pytest
import torch

import paper_1704_08907_amd as A

pytestmark = pytest.mark.gpu
ALL = ("xt", "xs", "w")


def make(nt, ns, d, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(nt + 7 * ns)
    xt, xs = (torch.rand((n, d), generator=g, device="cuda", dtype=dtype) for n in (nt, ns))
    w, gy = (torch.randn(n, generator=g, device="cuda", dtype=dtype) for n in (ns, nt))
    return xt, xs, w, 0.3, gy


# the adjoint's forms: two passes in one launch, and (from 2^25 pairs) each pair once, there
# with few targets and many sources, whose single passes take more scratch than it does
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("first,then", [([("w", "xs"), ("xt",)], ALL), ([ALL], ("w", "xs")), ([ALL], ("xt",)),
                                        ([ALL], ("w",)), ([ALL], ALL)])
@pytest.mark.parametrize("nt,ns,d", [(1000, 1500, 3), (300, 200000, 3), (371, 141726, 1), (6000, 6000, 2)])
def test_gradients_captured(nt, ns, d, first, then, dtype):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        c = A.Context(0, stream)
        args = make(nt, ns, d, dtype)
        for want in first:
            A.dense_sum_backward(c, *args, want=want)
        A.dense_sum(c, *args[:4])  # a forward of these sizes takes no more
        A.graph_capture_begin(c)
        got = A.dense_sum_backward(c, *args, want=then)
        y = A.dense_sum(c, *args[:4])
        g = A.graph_capture_end(c)
        # a larger call in between: the graph keeps its scratch
        A.dense_sum_backward(c, *make(3 * nt, 3 * ns, d, dtype))
        for _ in range(3):
            for t in got:
                if t is not None:
                    t.zero_()
            y.zero_()
            A.graph_launch(c, g)
            c.sync()
            ref = A.dense_sum_backward(c, *args, want=then)
            for a, b in zip(got, ref):
                if a is None:
                    assert b is None
                else:
                    # (another form of the adjoint where the scratch has grown: rounding of its sums)
                    tol = 1e-5 if dtype == torch.float32 else 1e-13
                    assert float((a - b).norm()) <= tol * float(b.norm())
            assert torch.equal(y, A.dense_sum(c, *args[:4]))
        g.close()
        c.close()
