"""Recorded lists of clustered particles, whose neighbours are several times the mean the
capacity is made for: every replay equals the box search's bits, whether the recording is
shared by several waves or not, and a graph's replay also after the list was recorded
again with less room."""
import pytest
import torch

import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import to_dev
from test_gpu_list_split import equal_sums

pytestmark = pytest.mark.gpu


def settled(d, n, nbr, prec):
    """Uniform in the lowest quarter of the box (and a few above): four times the density."""
    L = syn.side_for_density(n, d, nbr)
    rng = syn.SplitMix64(n)
    x = syn.uniform_positions(rng, n, [0.0] * d, [L] * d, prec)
    x[: n - n // 50, d - 1] *= 0.25
    return L, to_dev(x)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d,n,nbr", [(3, 5000, 30.0), (3, 45000, 30.0), (3, 70000, 60.0), (2, 45000, 9.0),
                                     (2, 160000, 5.0)])
def test_settled(d, n, nbr, prec):
    c = A.Context(0)
    L, x = settled(d, n, nbr, prec)
    cells = A.build_cells(c, x, [A.BoxSpec(d, [0.0] * d, [L] * d, [0] * d, 1.0)])
    equal_sums(c, cells, x, 0)
    cells.close()
    c.close()


@pytest.mark.parametrize("n", [5000, 45000])
def test_replay_after_a_recording_with_less_room(n):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        c = A.Context(0, stream)
        L, x = settled(3, n, 30.0, "f32")
        cells = A.build_cells(c, x, [A.BoxSpec(3, [0.0] * 3, [L] * 3, [0] * 3, 1.0)])
        y = torch.empty_like(x)
        A.build_neighbours(c, cells, 160)
        A.pair_sum(c, cells, "spring", (1.0,), y=y)
        want = y.clone()
        A.graph_capture_begin(c)
        A.pair_sum(c, cells, "spring", (1.0,), y=y)
        g = A.graph_capture_end(c)
        for capacity in (160, 40, 100):
            A.build_neighbours(c, cells, capacity)
            y.zero_()
            A.graph_launch(c, g)
            c.sync()
            assert torch.equal(y, want)
        g.close()
        cells.close()
        c.close()
