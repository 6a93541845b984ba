"""Saved dense launch plans: the adjoint's two forms are tuned apart where both fall into
the same size buckets, and plans saved under the keys of earlier kernels are not used."""
import json

import pytest
import torch

import paper_1704_08907_amd as A

pytestmark = pytest.mark.gpu


def arrays(n, dtype=torch.float32):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.rand((n, 2), generator=g, device="cuda", dtype=dtype)
    return x, torch.randn(n, generator=g, device="cuda", dtype=dtype), torch.randn(n, generator=g, device="cuda", dtype=dtype)


def test_forms_of_the_adjoint_are_tuned_apart(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("ABORIA_TUNE_CACHE", str(path))
    c = A.Context(0)
    for n in (5000, 8000):  # below and above 2^25 pairs, in one size bucket
        x, w, gy = arrays(n)
        A.autotune_dense(c, x, x, w, 0.2, gy)
    c.sync()
    c.close()
    keys = [e["key"] for e in json.loads(path.read_text())["dense"]]
    assert len(keys) == len(set(keys)) == 2


def old_key(backward, kernel, dtype, d, bt, bs):
    k = int(backward)
    for base, v in ((4, kernel), (4, dtype), (4, d), (64, bt), (64, bs)):
        k = k * base + v
    return k


def test_plans_of_earlier_kernels_are_not_used(tmp_path, monkeypatch):
    x, w, gy = arrays(12000)
    plain = A.Context(0)
    want = [A.dense_sum(plain, x, x, w, 0.2), *A.dense_sum_backward(plain, x, x, w, 0.2, gy)]
    plan = next(p for p in range(20) if A.dense_plan_name(p).startswith("8 targets per lane, 1024"))
    plain.set_dense_plan(plan)
    other = A.dense_sum(plain, x, x, w, 0.2)
    assert not torch.equal(other, want[0])  # the plan shows in the bits
    path = tmp_path / "tune.json"
    monkeypatch.setenv("ABORIA_TUNE_CACHE", str(path))
    c = A.Context(0)
    A.autotune_dense(c, *[t[:100].contiguous() for t in (x, x, w)], 0.2)  # a file with this device's name
    c.close()
    doc = json.loads(path.read_text())
    line = '{"key": %d, "dense_plan": [8, 1024]}'
    text = path.read_text().replace('"dense": [\n', '"dense": [\n' + "".join(
        line % old_key(b, 0, 0, 2, 13, 13) + ",\n" for b in (0, 1)))
    path.write_text(text)
    assert len(json.loads(text)["dense"]) == len(doc["dense"]) + 2
    c = A.Context(0)
    got = [A.dense_sum(c, x, x, w, 0.2), *A.dense_sum_backward(c, x, x, w, 0.2, gy)]
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    c.close()
    plain.close()


@pytest.mark.parametrize("n", [3000, 6000])  # both forms of the adjoint
def test_float_only_plan_is_plan_0_in_float64(n):
    x, w, gy = arrays(n, torch.float64)
    names = [A.dense_plan_name(p) for p in range(9)]
    c = A.Context(0)
    got = []
    for plan in (0, names.index("8 targets per lane, 2048 workgroups")):
        c.set_dense_plan(plan)
        got.append([A.dense_sum(c, x, x, w, 0.2), *A.dense_sum_backward(c, x, x, w, 0.2, gy)])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*got))
    c.close()
