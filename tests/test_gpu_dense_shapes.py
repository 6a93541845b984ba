"""Dense sums and adjoints at the edges of their launch shapes: target counts
around one workgroup's block, source counts around the split granularity, the
unroll and the tile, one and two targets per lane, and the adjoint's single
launch against its outputs requested one at a time."""
import numpy as np
import pytest
import torch

import oracle
import paper_1704_08907_amd as A
from _parity import TOL_F32, TOL_F64, to_dev
from test_gpu_dense import close, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = A.Context(0)
    yield c
    c.close()


def coordinate_scales(kernel, prm, xt, xs, w, gy):
    """Per target and per source, the sum over its pairs of |gy_i w_j 2 phi'| times the
    magnitudes of the two points: what the rounding of the scaled coordinates, each
    2^-24 (2^-53) of its magnitude, is multiplied by in a position gradient.  A gradient
    of few, close pairs is small against it, so the summands' scale alone is no bound."""
    xt, xs = xt.astype(np.float64), xs.astype(np.float64)
    q = ((xt[:, None] - xs[None]) ** 2).sum(-1)
    slope = np.exp(-q / (2 * prm ** 2)) / prm ** 2 if kernel == "gaussian" else 1.0 / np.sqrt(q + prm ** 2)
    c = np.abs(gy.astype(np.float64)[:, None] * w.astype(np.float64)[None]) * slope
    c = c * (np.abs(xt).max(1)[:, None] + np.abs(xs).max(1)[None])
    return c.sum(1), c.sum(0)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("nt,ns", [(1, 1), (1, 65), (63, 3), (64, 64), (257, 63), (255, 129), (513, 256), (700, 257),
                                   (5, 4099), (4099, 5)])
def test_ragged_shapes(ctx, nt, ns, prec):
    d = 1 + (nt + ns) % 3
    xt, xs, w, gy = inputs(d, prec, nt, ns, 31 * nt + ns)
    tol = TOL_F32 if prec == "f32" else TOL_F64
    for kernel, prm in (("gaussian", 0.15), ("multiquadric", 0.2)):
        print(kernel, d, nt, ns, prec, flush=True)
        args = (ctx, to_dev(xt), to_dev(xs), to_dev(w), prm)
        yo, so = oracle.dense_sum(kernel, prm, xt, xs, w)
        close(A.dense_sum(*args, kernel=kernel).cpu().numpy(), yo, so, tol, "forward")
        ref = oracle.dense_backward(kernel, prm, xt, xs, w, gy)
        got = A.dense_sum_backward(*args, to_dev(gy), kernel=kernel)
        # 16 unit roundoffs of the coordinate scale, the allowance the neighbour sums' bound has
        slack = [16 * (2.0 ** -24 if prec == "f32" else 2.0 ** -53) / tol * c
                 for c in coordinate_scales(kernel, prm, xt, xs, w, gy)] + [0.0]
        for k, name in enumerate(("xt", "xs", "w")):
            close(got[k].cpu().numpy(), ref[k], ref[3 + k] + slack[k], tol, "g" + name)
            one = A.dense_sum_backward(*args, to_dev(gy), kernel=kernel, want=(name,))[k]
            torch.cuda.synchronize()
            assert torch.equal(one, got[k]), name


def test_two_targets_per_lane_past_the_rule(ctx):
    # 9001 x 32001 pairs take two targets per lane; a block's rows and the last one, all sources
    nt, ns = 9001, 32001
    xt, xs, w, gy = inputs(2, "f32", nt, ns, 8)
    y = A.dense_sum(ctx, to_dev(xt), to_dev(xs), to_dev(w), 0.15).cpu().numpy()
    rows = np.r_[0:3, 255:258, 511:514, nt - 2:nt]
    yo, so = oracle.dense_sum("gaussian", 0.15, np.ascontiguousarray(xt[rows]), xs, w)
    close(y[rows], yo, so, TOL_F32, "forward rows")
    gxt, gxs, gw = A.dense_sum_backward(ctx, to_dev(xt), to_dev(xs), to_dev(w), 0.15, to_dev(gy))
    ref = oracle.dense_backward("gaussian", 0.15, np.ascontiguousarray(xt[rows]), xs, w, gy[rows])
    close(gxt.cpu().numpy()[rows], ref[0], ref[3], TOL_F32, "gxt rows")
