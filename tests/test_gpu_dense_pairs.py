"""The adjoint that forms each pair once (2^25 pairs and more): ragged counts on both
sides of its tiles of targets and of 64 sources, one and many target blocks, both kernels
and precisions, and the sizes either side of its rule, against the sums in float64."""
import pytest
import torch

import paper_1704_08907_amd as A

pytestmark = pytest.mark.gpu


def reference(kernel, prm, xt, xs, w, gy):
    """The three gradients and their absolute sums in float64, by blocks of targets."""
    xt, xs, w, gy = (v.double() for v in (xt, xs, w, gy))
    out = [torch.zeros_like(xt), torch.zeros_like(xs), torch.zeros_like(w)]
    mag = [torch.zeros_like(v) for v in out]
    for i in range(0, len(xt), 512):
        d = xt[i:i + 512, None, :] - xs[None, :, :]
        q = (d * d).sum(-1)
        if kernel == "gaussian":
            k = torch.exp(-q / (2 * prm * prm))
            g = -k / (prm * prm)
        else:
            k = torch.sqrt(q + prm * prm)
            g = 1.0 / k
        pair = (g * gy[i:i + 512, None] * w[None, :])[:, :, None] * d
        for s, a in ((out, lambda v: v), (mag, torch.abs)):
            s[0][i:i + 512] = a(pair).sum(1)
            s[1] += a(-pair).sum(0)
            s[2] += a(k * gy[i:i + 512, None]).sum(0)
    return out, mag


# A summand's relative error is below 16 u: the scaled coordinates' rounding moves q by
# (2 |x| |d| + d^2) u in units of the kernel's length, |x| <= 1, prm = 0.3: 13 u for the
# Gaussian where its summand is not negligible (q below 10), 5 u of arithmetic more; the
# sums, of 64-term blocks, add less than 200 u of their absolute value.
@pytest.mark.parametrize("kernel", ["gaussian", "multiquadric"])
@pytest.mark.parametrize("dtype,u", [(torch.float32, 6e-8), (torch.float64, 1.2e-16)])
@pytest.mark.parametrize("nt,ns,d", [(5793, 5793, 2), (5792, 5793, 3), (511, 70001, 3), (70001, 513, 1), (33000, 33001, 2)])
def test_pairs_once(kernel, dtype, u, nt, ns, d):
    if nt > 20000 and ns > 20000 and dtype == torch.float64:
        pytest.skip("the float32 rule's upper range")
    g = torch.Generator(device="cuda")
    g.manual_seed(nt + ns)
    xt, xs = (torch.rand((n, d), generator=g, device="cuda", dtype=dtype) for n in (nt, ns))
    w = torch.randn(ns, generator=g, device="cuda", dtype=dtype)
    gy = torch.randn(nt, generator=g, device="cuda", dtype=dtype)
    c = A.Context(0)
    got = A.dense_sum_backward(c, xt, xs, w, 0.3, gy, kernel)
    want, mag = reference(kernel, 0.3, xt, xs, w, gy)
    for a, b, m in zip(got, want, mag):
        assert float(((a.double() - b).abs() / (m + 1e-30)).max()) <= 220 * u
    c.close()
