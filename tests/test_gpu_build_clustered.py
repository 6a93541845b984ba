"""Cell lists of clustered particles, whose buckets are many times the room a uniform
system's would need: worked off in chunks, with several keys per thread, rows carried by the
sort or read by index, in every form of the bucket pass, bit for bit against the oracle's
stable counting sort."""
import numpy as np
import pytest

from paper_1704_08907_amd import synthetic as syn
from test_gpu_build_rule import check

pytestmark = pytest.mark.gpu


def clustered(rng, n, d, L, prec):
    """A quarter uniform, half in the lowest eighth, a quarter in one cell's corner; mixed."""
    x = syn.uniform_positions(rng, n, [0.0] * d, [L] * d, prec)
    x[n // 4: 3 * n // 4, d - 1] *= 0.125
    x[3 * n // 4:] = syn.uniform_positions(rng, n - 3 * n // 4, [2.0] * d, [2.4] * d, prec)
    return np.ascontiguousarray(x[np.argsort(rng.uniform(n))])


# bits of a bucket by the rule and forced, so that the mean bucket takes two, four, eight and
# ten keys a thread; positions below 2 MB (gathered by index) and above it (carried)
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d,n,nbr,low_bits", [(3, 20011, 30.0, 0), (2, 60001, 5.0, 0), (2, 60001, 9.0, 10), (3, 60001, 30.0, 8),
                                              (3, 60001, 30.0, 10), (3, 300007, 30.0, 8), (3, 300007, 8.0, 9),
                                              (2, 270001, 5.0, 0), (2, 550001, 5.0, 0)])
def test_clustered(d, n, nbr, low_bits, prec):
    L = syn.side_for_density(n, d, nbr)
    print(d, n, prec, flush=True)
    check(clustered(syn.SplitMix64(n + d), n, d, L, prec), L, d, prec, (0, low_bits, 0))


# the form of eight keys a thread on uniform particles: 8 bits of 7.6 particles a cell, a mean
# of about 1940 keys and room for 2330
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [60001, 300007])
def test_eight_keys_a_thread(n, prec):
    L = syn.side_for_density(n, 3, 30.0)
    x = syn.uniform_positions(syn.SplitMix64(n), n, [0.0] * 3, [L] * 3, prec)
    check(x, L, 3, prec, (0, 8, 0))
