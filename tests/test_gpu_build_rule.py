"""Cell lists under the built-in build rule, bit for bit against the oracle's
stable counting sort: one bucket and several, buckets of a few cells, every form
of the bucket pass (two to ten keys per thread, rows staged or gathered late),
and clustered positions whose buckets do not fit the room they are given."""
import numpy as np
import pytest

import oracle
import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import box_of, cells_state, to_dev
from test_gpu_build import check_system

pytestmark = pytest.mark.gpu


def check(x, L, d, prec, shape=(0, 0, 0)):
    c = A.Context(0)
    c.set_build_shape(*shape)
    s = syn.System(d, [0.0] * d, [L] * d, [1] * d, 1.0, x, prec)
    g = oracle.grid_of(s)
    cells = A.build_cells(c, to_dev(x), [box_of(s)])
    A.build_cells(c, to_dev(x), [box_of(s)], cells=cells)  # and again in place
    c.sync()
    check_system(g, x, *cells_state(cells))
    cells.close()
    c.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d,n,nbr", [(3, 1, 30.0), (2, 64, 5.0), (2, 2048, 9.0), (2, 2049, 9.0), (3, 2049, 60.0),
                                     (3, 4097, 30.0), (3, 30011, 30.0), (2, 70001, 20.0), (3, 140009, 40.0),
                                     (1, 50000, 4.0)])
def test_uniform(d, n, nbr, prec):
    L = max(syn.side_for_density(n, d, nbr), 3.0)
    x = syn.uniform_positions(syn.SplitMix64(17 * n + d), n, [0.0] * d, [L] * d, prec)
    print(d, n, prec, flush=True)
    check(x, L, d, prec)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [5000, 60001])
def test_clustered(n, prec):
    # half of the particles in one cell's corner, the rest uniform: buckets far over their room
    L = syn.side_for_density(n, 3, 30.0)
    rng = syn.SplitMix64(n)
    x = syn.uniform_positions(rng, n, [0.0] * 3, [L] * 3, prec)
    x[: n // 2] = syn.uniform_positions(rng, n // 2, [2.0] * 3, [2.4] * 3, prec)
    x = np.ascontiguousarray(x[np.argsort(rng.uniform(n))])
    check(x, L, 3, prec)


@pytest.mark.parametrize("low_bits", [9, 10])
def test_large_buckets_with_rows(low_bits):
    # 300000 particles, 7 a cell, rows carried: buckets of about 3700 and 7400 keys
    L = syn.side_for_density(300000, 3, 30.0)
    x = syn.uniform_positions(syn.SplitMix64(5), 300000, [0.0] * 3, [L] * 3, "f32")
    check(x, L, 3, "f32", (0, low_bits, 0))
