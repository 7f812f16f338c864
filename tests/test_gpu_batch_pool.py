"""A default batch whose shared arrays want more room than the pool has: those without a region are
left to the general kernel.  The arrays are overlapping views of one buffer at every alignment;
value and counts against the defining property of the k-th smallest, exactly, sums of the k
smallest within n 2^-53 of the sum of the absolute values (one rounding of a double sum per
element, on either side)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,n,count", [("float32", 1 << 24, 160), ("float64", 1 << 23, 600)])
def test_more_than_the_pool_holds(dtype, n, count):
    import paper_1104_2732_amd as cps
    g = torch.Generator(device="cuda")
    g.manual_seed(count)
    x = torch.randn(n + count, generator=g, device="cuda", dtype=getattr(torch, dtype))
    views = [x[i: i + n - 3 * i] for i in range(count)]
    ks = [int((0.02 + 0.96 * i / count) * v.numel()) for i, v in enumerate(views)]
    s = cps.Selector(0)
    try:
        print(f"case batch pool {dtype} n={n} count={count}", flush=True)
        res, ksum = s.select_kth_batched_ksum(views, ks)
        again = s.select_kth_batched(views, ks)
    finally:
        s.close()
    listed = res["passes"] > 1
    assert listed.any() and not listed.all()
    for f in ("value_bits", "less", "equal", "greater", "status"):  # (which ones are left is not fixed)
        assert np.array_equal(res[f], again[f]), f
    for i, (v, k) in enumerate(zip(views, ks)):
        r = res[i]
        t = torch.tensor(r["value"], dtype=v.dtype, device="cuda")
        less, eq = int((v < t).sum()), int((v == t).sum())
        assert r["status"] == 0 and less < k <= less + eq, (i, r)
        assert (r["less"], r["equal"], r["greater"]) == (less, eq, v.numel() - less - eq), (i, r)
        if i % 7 == 0 or listed[i]:
            d = v.to(torch.float64)
            low = torch.where(v < t, d, 0.0)
            want = float(low.sum()) + (k - less) * float(t)
            scale = float(low.abs().sum()) + (k - less) * abs(float(t))
            assert abs(ksum[i] - want) <= 2 * v.numel() * 2.0 ** -53 * scale, i
