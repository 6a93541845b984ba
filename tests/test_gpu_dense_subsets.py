"""Gradients asked for one or two at a time where all three at once form each pair once
(2^25 pairs and more): the same sums in another order, so equal within their bound, and
untouched where not asked for."""
import pytest
import torch

import paper_1704_08907_amd as A
from test_gpu_dense_pairs import reference

pytestmark = pytest.mark.gpu


# the bound of the sums that form each pair once, 220 u of the sum of magnitudes
@pytest.mark.parametrize("dtype,u", [(torch.float32, 6e-8), (torch.float64, 1.2e-16)])
@pytest.mark.parametrize("kernel", ["gaussian", "multiquadric"])
@pytest.mark.parametrize("nt,ns,d", [(5793, 5793, 2), (511, 70001, 3), (70001, 513, 1)])
def test_subsets(kernel, dtype, u, nt, ns, d):
    g = torch.Generator(device="cuda")
    g.manual_seed(nt)
    xt, xs = (torch.rand((n, d), generator=g, device="cuda", dtype=dtype) for n in (nt, ns))
    w, gy = (torch.randn(n, generator=g, device="cuda", dtype=dtype) for n in (ns, nt))
    c = A.Context(0)
    want, mag = reference(kernel, 0.3, xt, xs, w, gy)
    for names in (("xt",), ("xs",), ("w",), ("xt", "xs"), ("xt", "w"), ("xs", "w"), ("xt", "xs", "w")):
        got = A.dense_sum_backward(c, xt, xs, w, 0.3, gy, kernel, want=names)
        for k, name in enumerate(("xt", "xs", "w")):
            if name not in names:
                assert got[k] is None
                continue
            assert float(((got[k].double() - want[k]).abs() / (mag[k] + 1e-30)).max()) <= 220 * u
    c.close()
