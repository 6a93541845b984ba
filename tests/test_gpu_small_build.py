"""The one-workgroup build of small cell lists: counts around a wave's and the
workgroup's share, one cell more or less than a power of two, several systems,
and a domain error, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import box_of, cells_state, to_dev
from test_gpu_build import check_system
from test_gpu_build_rule import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d,n,L", [(1, 63, 20.0), (2, 64, 4.0), (2, 127, 16.5), (2, 128, 31.9), (3, 129, 8.1), (3, 1000, 6.5),
                                   (2, 1920, 30.5), (3, 2047, 9.9), (3, 2048, 10.05)])
def test_one_workgroup(d, n, L, prec):
    x = syn.uniform_positions(syn.SplitMix64(n), n, [0.0] * d, [L] * d, prec)
    check(x, L, d, prec)


def test_systems_and_domain_error():
    c = A.Context(0)
    w = syn.batch_cubes(nsys=5, nmin=200, nmax=500)
    x = np.concatenate([s.x for s in w.systems])
    assert len(x) <= 2048
    off = np.concatenate([[0], np.cumsum([s.n for s in w.systems])]).tolist()
    cells = A.build_cells(c, to_dev(x), [box_of(s) for s in w.systems], off)
    c.sync()
    state = cells_state(cells)
    base = 0
    for b, s in enumerate(w.systems):
        g = oracle.grid_of(s)
        check_system(g, s.x, *state, off[b], base)
        base += int(g.ncells)
    x[7, 1] = np.nan
    A.build_cells(c, to_dev(x), [box_of(s) for s in w.systems], off, cells=cells)
    with pytest.raises(A.AboriaError) as e:
        c.sync()
    assert e.value.status == "DOMAIN"
    cells.close()
    c.close()


@pytest.mark.parametrize("op,params", [("exp_force", (1.0,)), ("dem_spring", (1.0,)), ("soft_sphere", ())])
@pytest.mark.parametrize("n", [64, 4095, 4096])
def test_all_pairs_input_order(n, op, params):
    """The all-pairs sums read gradients and variables in the caller's order below 4096
    particles, gathered ones above; equal to the row search up to the order of the sums:
    m = 80 neighbours at most, summands below 40 (a jittered lattice: distances over 0.3,
    so a Jacobian's entries are below 5, times gradients below 8), so 2 m u m 40 = 6e-11."""
    c = A.Context(0)
    rng = np.random.default_rng(n)
    grid = np.stack(np.meshgrid(*[np.arange(16) * 0.5] * 3, indexing="ij"), -1).reshape(-1, 3)[rng.permutation(4096)[:n]]
    x = to_dev((grid + 0.25 + 0.1 * (2 * rng.random((n, 3)) - 1)).astype(np.float64))
    cells = A.build_cells(c, x, [A.BoxSpec(3, [0.0] * 3, [8.0] * 3, [1, 1, 1], 1.0)])
    a = to_dev(0.3 + 0.3 * rng.random((n, 1))) if op == "dem_spring" else None
    gy = to_dev(np.clip(rng.standard_normal((n, A.op_ny(op, 3))), -4, 4))
    got = []
    for name in ("over all particles of its system", "adjoint evaluated on every candidate"):
        c.set_variant(next(v for v in range(A.variant_count()) if name in A.variant_name(v)))
        y = A.pair_sum(c, cells, op, params, a)
        got.append((y, *A.pair_sum_backward(c, cells, op, params, gy, a)))
    for u, v in zip(*got):
        if u is not None:
            assert float((u - v).abs().max()) <= 6e-11
    cells.close()
    c.close()
