"""Sums captured in a graph whose cell list is rebuilt with other boxes afterwards: a
replay follows the boxes of the latest build, also where these search deeper than the
ones it was captured with (same cell counts, reach 1 to 2)."""
import numpy as np
import pytest
import torch

import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import TOL_F32, TOL_F64, to_dev

pytestmark = pytest.mark.gpu


# a wave per row of 64 particles (5000), three waves (45000, in 2-d one row each), one (645000)
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d,n,L,ncell", [(3, 5000, 12.0, 6), (3, 45000, 24.0, 12), (2, 5000, 40.0, 20),
                                         (2, 45000, 100.0, 50), (2, 645000, 400.0, 200)])
def test_replay_after_a_deeper_rebuild(d, n, L, ncell, prec):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        c = A.Context(0, stream)
        rng = syn.SplitMix64(n + d)
        x = to_dev(syn.uniform_positions(rng, n, [0.0] * d, [L] * d, prec))
        gy = to_dev(rng.normal(n * d).reshape(n, d).astype(np.float32 if prec == "f32" else np.float64))

        def box(cutoff, reach):
            return A.BoxSpec(d, [0.0] * d, [L] * d, [1] * (d - 1) + [0], cutoff, [ncell] * d, reach)

        near, far = box(1.9, 1), box(3.9, 2)
        cells = A.build_cells(c, x, [near])
        out = [torch.empty((n, 1), dtype=x.dtype, device=x.device), torch.empty_like(x), torch.empty_like(x),
               torch.empty_like(x), torch.empty_like(x)]

        def sums():
            A.pair_sum(c, cells, "count", (), y=out[0])
            A.pair_sum(c, cells, "spring", (1.0,), y=out[1])
            A.pair_sum_backward(c, cells, "spring", (1.0,), gy, gx=out[2])
            A.pair_sum_and_backward(c, cells, "spring", (1.0,), gy, y=out[3], gx=out[4])

        sums()
        A.graph_capture_begin(c)
        sums()
        g = A.graph_capture_end(c)
        for b in (far, near, far):
            A.build_cells(c, x, [b], cells=cells)
            sums()
            want = [t.clone() for t in out]
            for t in out:
                t.zero_()
            A.graph_launch(c, g)
            c.sync()
            assert torch.equal(out[0], want[0])
            # the same pairs in another order
            tol = TOL_F32 if prec == "f32" else TOL_F64
            for got, ref in zip(out[1:], want[1:]):
                assert float((got - ref).norm()) <= tol * float(ref.norm())
        g.close()
        cells.close()
        c.close()
