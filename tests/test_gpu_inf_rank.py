"""Ranks among repeated infinities, at either end: the array is read once, as for any other repeated
value, and value and counts are exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def make(n, dtype, seed, low, high):
    r = np.random.default_rng([seed, n])
    x = r.standard_normal(n).astype(dtype)
    u = r.random(n)
    x[u < low] = -np.inf
    x[u >= 1.0 - high] = np.inf
    return x


def check(x, k, r):
    s = np.sort(x)
    v = s[k - 1]
    less, eq = int(np.searchsorted(s, v, "left")), int(np.searchsorted(s, v, "right"))
    assert r["status"] == 0 and r["value"] == float(v), (k, r)
    assert (r["less"], r["equal"], r["greater"]) == (less, eq - less, x.size - eq), (k, r)


SHARES = [(0.3, 0.4), (0.0, 0.7), (0.7, 0.0), (0.0, 1.0), (1.0, 0.0), (0.5, 0.5)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [70_001, 300_000, (1 << 24) + 3])
def test_single(dtype, n):
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    for low, high in SHARES:
        x = make(n, dtype, 1, low, high)
        d = torch.from_numpy(x).cuda()
        for q in (0.02, 0.1, 0.5, 0.9, 0.98):
            k = int(q * n)
            inside = q < low - 0.05 or q > 1.0 - high + 0.05
            print(f"case inf rank {x.dtype} n={n} shares {low} {high} q={q}", flush=True)
            r = s.select_kth(d, k)
            check(x, k, r)
            if inside:
                assert r["passes"] == 1, (low, high, q, r)
    s.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_batched(dtype):
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    arrays, ks, inside = [], [], []
    for n in (9000, 20_000, 70_001, 300_000, 1_000_001):
        for low, high in SHARES:
            for q in (0.02, 0.1, 0.5, 0.9, 0.98):
                arrays.append(make(n, dtype, 2, low, high))
                ks.append(int(q * n))
                inside.append(q < low - 0.05 or q > 1.0 - high + 0.05)
    dev = [torch.from_numpy(x).cuda() for x in arrays]
    print(f"case inf rank batch {np.dtype(dtype)}", flush=True)
    res = s.select_kth_batched(dev, ks)
    for i, (x, k) in enumerate(zip(arrays, ks)):
        check(x, k, res[i])
        if inside[i]:
            assert res[i]["passes"] == 1, (i, x.size, k, res[i])
    s.close()
