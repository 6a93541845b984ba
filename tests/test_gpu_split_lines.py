"""Box-search sums on both sides of the sizes up to which waves share rows: by points in
a cell one cutoff wide (fewer than four, four to ten, more), also on grids whose cells are
a third of the cutoff in x.  Every kernel takes the same side, so all agree bit for bit."""
import numpy as np
import pytest

import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import to_dev
from test_gpu_split import agree, ctx  # noqa: F401  (ctx is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,nbr,m", [(3, 224000, 8.0, 3), (3, 224001, 8.0, 3), (3, 224001, 30.0, 3),
                                       (3, 268801, 30.0, 3), (2, 416000, 20.0, 3), (2, 416001, 20.0, 1)])
def test_lines(ctx, d, n, nbr, m):  # noqa: F811
    L = syn.side_for_density(n, d, nbr)
    rng = syn.SplitMix64(n + m)
    x = syn.uniform_positions(rng, n, [0.0] * d, [L] * d, "f32")
    print(d, n, nbr, m, flush=True)
    cells = A.build_cells(ctx, to_dev(x), [A.BoxSpec(d, [0.0] * d, [L] * d, [1] * d, 1.0, reach=[m] + [1] * (d - 1))])
    agree(ctx, cells, "soft_sphere", (), to_dev(rng.normal(n).astype(np.float32).reshape(n, 1)))
    agree(ctx, cells, "spring", (1.0,), to_dev(rng.normal(d * n).astype(np.float32).reshape(n, d)))
    cells.close()
