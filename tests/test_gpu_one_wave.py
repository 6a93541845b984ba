"""The search kernels of large lists, which keep one wave per 64 particles and a running
sum: every operator and variant on grids narrower than their stencil, closed sides, rows of
more candidates than a record holds, both precisions. Batches repeat one of the parity
boxes until they are past the line, so that the oracle sums one system; single systems are
long and thin, or uniform just past the line of their type."""
import numpy as np
import pytest
import torch

import oracle
import paper_1704_08907_amd as A
from paper_1704_08907_amd import synthetic as syn
from _parity import check_close, to_dev
from test_gpu_parity import CASES, OPS, make_case, tol_of
from test_gpu_split import agree

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = A.Context(0)
    yield c
    c.set_variant(-1)
    c.close()


def inputs(n, d, dtype, op, seed):
    rng = syn.SplitMix64(seed)
    gy = rng.normal(n * A.op_ny(op, d)).astype(dtype).reshape(n, -1)
    a = (0.2 + 0.3 * rng.uniform(n)).astype(dtype).reshape(n, 1) if op == "dem_spring" else None
    return gy, a


def against_oracle(g, x, op, params, gy, a, got, tol, uniform):
    x64 = x.astype(np.float64)
    yo, so = oracle.pair_sum(g, op, params, x64, a=a)
    if op == "count":
        np.testing.assert_array_equal(got[0].cpu().numpy()[:, 0], yo[:, 0])
        assert torch.all(got[1] == 0)
        return
    check_close(got[0].cpu().numpy(), yo, so, tol, "forward " + op, normwise=uniform)
    gxo, gao, sxo, sao = oracle.pair_sum_backward(g, op, params, x64, gy, a=a)
    check_close(got[1].cpu().numpy(), gxo, sxo, tol, "adjoint " + op, normwise=uniform)
    if a is not None:
        check_close(got[2].cpu().numpy(), gao.reshape(-1, 1), sao, tol, "adjoint a", normwise=uniform)


def step_is_sum_and_integration(ctx, cells, x, y):
    v = 0.01 * torch.ones_like(y)
    x1, v1, x2, v2 = x.clone(), v.clone(), x.clone(), v.clone()
    ctx.set_variant(0)
    A.md_step(ctx, cells, "spring", (1.0,), 1e-3, x1, v1)
    A.integrate(ctx, cells, 1e-3, y, x2, v2)
    ctx.set_variant(-1)
    torch.cuda.synchronize()
    assert torch.equal(x1, x2) and torch.equal(v1, v2)


@pytest.mark.parametrize("case", [c for c in CASES if c[1] > 1], ids=[c[0] for c in CASES if c[1] > 1])
def test_repeated_parity_boxes(ctx, case):
    g, x, box, prec = make_case(case)
    n, d = x.shape
    copies = 64 * 3000 // n + 1  # past 3000 waves
    xd = to_dev(x).repeat(copies, 1)
    cells = A.build_cells(ctx, xd, [box] * copies, [n * i for i in range(copies + 1)])
    uniform = slice(0, n - n // 5)  # (the rest sit within ulps of cell faces)
    for op, params in OPS:
        print(case[0], op, flush=True)
        gy, a = inputs(n, d, x.dtype, op, 99)
        rep = [to_dev(t).repeat(copies, 1) if t is not None else None for t in (gy, a)]
        got = agree(ctx, cells, op, params, *rep)
        for t in got:
            assert torch.equal(t, t[:n].repeat(copies, 1))
        against_oracle(g, x, op, params, gy, a, [t[:n] for t in got], tol_of(prec), uniform)
        if op == "spring":
            step_is_sum_and_integration(ctx, cells, xd, got[0])
    cells.close()


# thin: two cells in x (and y) of a long box; at most four particles a cell, so that the line
# is at 224000 particles (float64 in 3-d at 102400)
@pytest.mark.parametrize("d,n,hi,periodic,prec", [
    (2, 224065, [2.1, 60000.0], [1, 0], "f32"), (2, 224065, [2.1, 60000.0], [0, 1], "f64"),
    (3, 224065, [2.2, 2.3, 20000.0], [1, 0, 1], "f32"), (3, 102465, [2.2, 2.3, 9000.0], [0, 1, 0], "f64"),
    (3, 102465, [24.0, 25.0, 26.0], [1, 0, 1], "f64"), (2, 224065, [300.0, 310.0], [0, 1], "f64"),
    (2, 224065, [300.0, 310.0], [1, 0], "f32"), (3, 224065, [48.0, 49.0, 50.0], [1, 1, 0], "f32"),
])
def test_single_systems(ctx, d, n, hi, periodic, prec):
    x = syn.uniform_positions(syn.SplitMix64(n + d), n, [0.0] * d, hi, prec)
    g = oracle.grid(d, [0.0] * d, hi, periodic, 1.0, prec)
    xd = to_dev(x)
    cells = A.build_cells(ctx, xd, [A.BoxSpec(d, [0.0] * d, hi, periodic, 1.0)])
    for op, params in OPS:
        print(d, hi, prec, op, flush=True)
        gy, a = inputs(n, d, x.dtype, op, 7)
        got = agree(ctx, cells, op, params, to_dev(gy), to_dev(a) if a is not None else None)
        if op in ("spring", "dem_spring"):
            # (in the thin boxes float32 coordinates are 2^-9 and more apart: points cluster within
            # a few of their ulps, which the normwise test does not cover)
            against_oracle(g, x, op, params, gy, a, got, tol_of(prec), slice(None) if max(hi) < 1000 else None)
        if op == "spring":
            step_is_sum_and_integration(ctx, cells, xd, got[0])
    cells.close()
