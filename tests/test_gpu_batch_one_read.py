"""The default batched selection at the sizes where a variant begins or ends (arrays held in
registers, one workgroup's interval, arrays cut into parts), on inputs whose ranks fall on
repeated ends, outside the interval, on infinities and NaN, at unaligned starts: value and counts
against the sorted array, exactly; sums of the k smallest within n 2^-53 of the sum of the
absolute values (one rounding of a double sum per element)."""
import numpy as np
import pytest

from tests.test_gpu_one_read import KINDS, make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [1, 2, 3, 64, 1000, 4095, 4096, 4097, 16383, 16384, 16385, 50_001, (1 << 16) - 1, 1 << 16,
         (1 << 17) - 1, 1 << 17, (1 << 17) + 1, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, 600_011,
         (1 << 20) + 3]


@pytest.fixture(scope="module")
def sel():
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    yield s
    s.close()


def check(arrays, ks, res, ksum=None):
    for i, (x, k) in enumerate(zip(arrays, ks)):
        if np.isnan(x).any():
            assert res[i]["status"] == 1, i
            continue
        s = np.sort(x)
        v = s[k - 1]
        less, eq = int(np.searchsorted(s, v, "left")), int(np.searchsorted(s, v, "right"))
        got = res[i]
        assert got["status"] == 0, (i, x.size, k, got)
        assert got["value"] == float(v), (i, x.size, k, got, v)
        assert (got["less"], got["equal"], got["greater"]) == (less, eq - less, x.size - eq), (i, got)
        if ksum is not None and np.isfinite(s[:k]).all():
            d = s[:k].astype(np.float64)
            assert abs(ksum[i] - d.sum()) <= 2 * x.size * 2.0 ** -53 * np.abs(d).sum(), (i, x.size, k)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", KINDS)
def test_edges(sel, kind, dtype):
    arrays, ks, dev = [], [], []
    for n in SIZES:
        for q in (0.0, 0.1, 0.5, 0.97, 1.0):
            off = len(arrays) % 4
            x = make(kind, n + off, dtype, len(arrays))
            dev.append(torch.from_numpy(x).cuda()[off:])
            arrays.append(x[off:])
            ks.append(min(n, max(1, int(round(q * n)))))
    print(f"case batch edges {kind} {np.dtype(dtype)} arrays={len(arrays)}", flush=True)
    check(arrays, ks, sel.select_kth_batched(dev, ks))
    print("with sums", flush=True)
    res, ksum = sel.select_kth_batched_ksum(dev, ks)
    check(arrays, ks, res, ksum)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_nan(sel, dtype):
    arrays, ks = [], []
    for n in (1, 500, 5000, 20_000, 140_000, 300_000, 900_000):
        for at in (0, n // 2, n - 1, None):
            x = make("normal", n, dtype, n)
            if at is not None:
                x[at] = np.nan
            arrays.append(x)
            ks.append((n + 1) // 2)
    dev = [torch.from_numpy(x).cuda() for x in arrays]
    print(f"case batch nan {np.dtype(dtype)}", flush=True)
    res, ksum = sel.select_kth_batched_ksum(dev, ks)
    check(arrays, ks, res, ksum)
    assert all(np.isnan(ksum[i]) == np.isnan(x).any() for i, x in enumerate(arrays))


def test_more_arrays_than_one_order_holds(sel):
    """4096 arrays are ordered together: one more, and a few thousand more."""
    r = np.random.default_rng(1)
    for count in (4097, 9001):
        sizes = r.integers(1, 300, count)
        flat = r.standard_normal(int(sizes.sum())).astype(np.float32)
        arrays = np.split(flat, np.cumsum(sizes)[:-1])
        d = torch.from_numpy(flat).cuda()
        dev = list(torch.split(d, sizes.tolist()))
        ks = [int(r.integers(1, n + 1)) for n in sizes]
        print(f"case batch count={count}", flush=True)
        check(arrays, ks, sel.select_kth_batched(dev, ks))
