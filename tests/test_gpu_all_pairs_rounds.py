"""All-pairs sums at the edges of their rounds of eight and two candidates, for every number
of lanes per particle, with inputs read in the caller's order (lists below 4096; of every
candidate in systems of up to 1024, else of the accepted ones) and gathered, against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import TOL_F32, TOL_F64, check_close, to_dev

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 13, 33, 64, 65, 257]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("sizes", [EDGES + [1024], EDGES + [1025], [1024], [1025], [320, 321], EDGES * 8, EDGES * 35,
                                   EDGES * 140], ids=["edges", "accepted", "1024", "1025", "five_each", "16", "4", "1"])
def test_rounds(sizes, d, prec):
    c = A.Context(0)
    rng = syn.SplitMix64(sum(sizes) + d)
    xs, boxes, off = [], [], [0]
    for n in sizes:
        L = max(syn.side_for_density(n, d, 12.0), 2.1)
        xs.append(syn.uniform_positions(rng, n, [0.0] * d, [L] * d, prec))
        boxes.append((L, A.BoxSpec(d, [0.0] * d, [L] * d, [1] * (d - 1) + [0], 1.0)))
        off.append(off[-1] + n)
    x = np.concatenate(xs)
    gy = rng.normal(len(x) * d).astype(x.dtype).reshape(-1, d)
    a = (0.4 + 0.1 * rng.uniform(len(x))).astype(x.dtype).reshape(-1, 1)
    cells = A.build_cells(c, to_dev(x), [b for _, b in boxes], off)
    assert "all particles" in A.variant_name(A.selected_variant(c, cells, "dem_spring"))
    y = A.pair_sum(c, cells, "dem_spring", (1.0,), to_dev(a)).cpu().numpy()
    gx, ga = (t.cpu().numpy() for t in A.pair_sum_backward(c, cells, "dem_spring", (1.0,), to_dev(gy), to_dev(a)))
    tol = TOL_F32 if prec == "f32" else TOL_F64
    for b in range(min(len(sizes), len(EDGES) + 1)):
        s = slice(off[b], off[b + 1])
        g = oracle.grid(d, [0.0] * d, [boxes[b][0]] * d, [1] * (d - 1) + [0], 1.0, prec)
        x64 = x[s].astype(np.float64)
        yo, so = oracle.pair_sum(g, "dem_spring", (1.0,), x64, a=a[s])
        check_close(y[s], yo, so, tol, "forward %d" % sizes[b], normwise=False)
        gxo, gao, sxo, sao = oracle.pair_sum_backward(g, "dem_spring", (1.0,), x64, gy[s], a=a[s])
        check_close(gx[s], gxo, sxo, tol, "adjoint %d" % sizes[b], normwise=False)
        check_close(ga[s], gao.reshape(-1, 1), sao, tol, "adjoint a %d" % sizes[b], normwise=False)
    # (the systems after the first of each size are not compared)
    assert np.isfinite(y).all() and np.isfinite(gx).all() and np.isfinite(ga).all()
    cells.close()
    c.close()
