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
