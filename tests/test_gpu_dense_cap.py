"""The dense adjoint either side of its scratch bound (256 MiB of partial sums), where it
goes from each pair once, in fewer and fewer splits, to two passes: rows of both sides'
gradients against float64."""
import pytest
import torch

import paper_1704_08907_amd as A

pytestmark = pytest.mark.gpu


# The bound of the sums that form each pair once: a summand's relative error below 16 u, a
# sum of 64-term blocks 200 u of its absolute value; blocks of 64 sources add up in up to
# 1400 steps per split, a running sum of which a random-sign rounding stays below 30 u more.
@pytest.mark.parametrize("dtype,u,sizes", [(torch.float32, 6e-8, (91000, 91600, 92100, 92600)),
                                           (torch.float64, 1.2e-16, (64000, 64500, 65200, 65300))])
def test_either_side_of_the_scratch_bound(dtype, u, sizes):
    c = A.Context(0)
    for n in sizes:
        print(n, flush=True)
        g = torch.Generator(device="cuda")
        g.manual_seed(n)
        xt, xs = (torch.rand((n, 3), generator=g, device="cuda", dtype=dtype) for _ in range(2))
        w, gy = (torch.randn(n, generator=g, device="cuda", dtype=dtype) for _ in range(2))
        gxt, gxs, gw = A.dense_sum_backward(c, xt, xs, w, 0.3, gy, "multiquadric")
        rows = torch.cat([torch.arange(0, 3), torch.arange(509, 515), torch.arange(n - 3, n)]).cuda()
        for a, b, wa, wb, got, gsum in ((xt, xs, gy, w, gxt, None), (xs, xt, w, gy, gxs, gw)):
            d = a[rows].double()[:, None] - b.double()[None]
            k = torch.sqrt((d * d).sum(-1) + 0.09)
            pair = (wa[rows].double()[:, None] * wb.double()[None] / k)[..., None] * d
            assert float(((got[rows].double() - pair.sum(1)).abs() / pair.abs().sum(1)).max()) <= 250 * u
            if gsum is not None:
                v = k * wb.double()[None]
                assert float(((gsum[rows].double() - v.sum(1)).abs() / v.abs().sum(1)).max()) <= 250 * u
    c.close()
