"""Neighbour lists recorded by several waves per 64 particles: sums over them equal the
box search's bit for bit, with rows of more neighbours than a wave keeps in LDS, lists
too short for some particles, a ragged last wave, and systems of uneven size."""
import pytest
import torch

import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import box_of, to_dev
from test_gpu_neighbours import inputs, replay_variant, run, same

pytestmark = pytest.mark.gpu


def equal_sums(c, cells, x, capacity):
    n, d = x.shape
    dtype = "float32" if x.dtype == torch.float32 else "float64"
    a, gy = inputs("exp_force", n, d, dtype)
    gy_d = to_dev(gy)
    want = run(c, cells, "exp_force", (1.0,), a, gy_d, 0)
    A.build_neighbours(c, cells, capacity)
    got = run(c, cells, "exp_force", (1.0,), a, gy_d, replay_variant())
    for u, v in zip(got, want):
        assert same(u, v)


# neighbours 5 to 60 (rows of the 2-d stencil hold a third of them: 20 at 60, and over 32
# at 160), capacities 0 (by density) and too small for many particles
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d,n,nbr,capacity", [(2, 4096, 20.0, 0), (2, 3001, 160.0, 0), (2, 3001, 160.0, 130), (3, 2049, 30.0, 0),
                                              (3, 5003, 160.0, 0), (3, 5003, 60.0, 50), (3, 41000, 30.0, 0),
                                              (3, 41000, 160.0, 0), (1, 3000, 12.0, 0)])
def test_recorded_by_several_waves(d, n, nbr, capacity, prec):
    c = A.Context(0)
    L = syn.side_for_density(n, d, nbr)
    x = to_dev(syn.uniform_positions(syn.SplitMix64(n), n, [0.0] * d, [L] * d, prec))
    cells = A.build_cells(c, x, [A.BoxSpec(d, [0.0] * d, [L] * d, [1] * d, 1.0)])
    equal_sums(c, cells, x, capacity)
    cells.close()
    c.close()


def test_recorded_systems():
    c = A.Context(0)
    w = syn.batch_cubes(nsys=7, nmin=300, nmax=4000)
    x = torch.cat([to_dev(s.x) for s in w.systems])
    off = [0]
    for s in w.systems:
        off.append(off[-1] + s.n)
    cells = A.build_cells(c, x, [box_of(s) for s in w.systems], off)
    equal_sums(c, cells, x, 0)
    cells.close()
    c.close()
