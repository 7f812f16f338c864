"""The default selection's own kernels (arrays held in registers; one read against a likely
interval) at the sizes where a variant begins or ends, on inputs whose ranks fall on repeated
ends, into one crowded bin, outside the interval, at infinities and NaN: value and counts against
the oracle, exactly."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import assert_same_result

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sel():
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    yield s
    s.close()


def make(kind, n, dtype, seed):
    r = np.random.default_rng([seed, n])
    x = r.standard_normal(n).astype(dtype)
    h = n // 2
    if kind == "constant":
        x[:] = -3.25
    elif kind == "zeros":
        x = np.where(r.random(n) < 0.5, 0.0, -0.0).astype(dtype)
        x[:: max(1, n // 9)] = r.standard_normal(x[:: max(1, n // 9)].size)
    elif kind == "spike":  # most of the data one value, just off the rank's neighbours
        x[r.random(n) < 0.7] = 0.125
    elif kind == "ties":
        x = np.round(x * 8).astype(dtype)
    elif kind == "crowd":  # a bin with far more than the gather holds, of distinct keys
        x = (1.0 + r.integers(0, 1 << 20, n) * 2.0 ** -23).astype(dtype)
        x[: n // 64] = 1e30
        x[n // 64: n // 32] = -1e30
    elif kind == "hidden":  # what the runs at even distances see is not what the rest holds
        stride = n // (1024 if n >= (1 << 18) else 256) or 1
        x[(np.arange(n) % stride) < 16] = 7.0
    elif kind == "sorted":
        x.sort()
    elif kind == "inf":
        x[: h - h // 8] = np.inf
        x[n - h // 4:] = -np.inf
    elif kind == "denormal":
        x = (x * np.finfo(dtype).tiny / 64).astype(dtype)
    return x


KINDS = ["normal", "constant", "zeros", "spike", "ties", "crowd", "hidden", "sorted", "inf",
         "denormal"]
SIZES = [1, 2, 63, 64, 65, 255, 1024, 1025, 4096, 4097, 16384, 16385, 32767, 32768, 32769, 65536,
         65537, 200_003, (1 << 18) - 1, 1 << 18, 1_000_003]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", KINDS)
def test_edges(sel, oracle_mod, kind, dtype):
    for n in SIZES:
        x = make(kind, n, dtype, 5)
        d = torch.from_numpy(x).cuda()
        for k in sorted({1, 2, max(1, n // 1000), n // 4 + 1, (n + 1) // 2, n - n // 64, n}):
            if not 1 <= k <= n:
                continue
            print(f"case one read {kind} {x.dtype} n={n} k={k}", flush=True)
            assert_same_result(sel.select_kth(d, k), oracle_mod.select_kth(x, k),
                               f"{kind} n={n} k={k}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1 << 24, (1 << 25) + 5])
def test_copied(sel, oracle_mod, n, dtype):
    """Inputs whose interval is copied (2^26 bytes and more; one element less is read again), a few kinds and an unaligned start."""
    for kind in ("normal", "spike", "crowd", "hidden", "inf"):
        x = make(kind, n, dtype, 9)
        d = torch.from_numpy(x).cuda()
        for k, off in ((n // 3, 0), ((n - 1) // 2, 1)):
            print(f"case copied {kind} {x.dtype} n={n} k={k} off={off}", flush=True)
            want = np.partition(x[off:], k - 1)[k - 1]
            got = sel.select_kth(d[off:], k)
            assert got["status"] == 0 and got["value"] == float(want), (kind, got, want)
            v = x[off:]
            assert (got["less"], got["equal"], got["greater"]) == (
                int((v < want).sum()), int((v == want).sum()), int((v > want).sum()))
        del d


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_nan_and_repeats(sel, dtype):
    """A NaN anywhere is reported, and calls on one workspace do not see each other's bins."""
    import paper_1104_2732_amd as cps
    out = sel.new_results(1)
    for n in (1000, 5000, 65537, 300_001):
        x = make("normal", n, dtype, 3)
        want = sel.select_kth(torch.from_numpy(x).cuda(), n // 3)
        for at in (0, n // 2 + 37, n - 1):
            y = x.copy()
            y[at] = np.nan
            print(f"case nan n={n} at={at}", flush=True)
            sel.select_kth_async(torch.from_numpy(y).cuda(), n // 3, out)
            torch.cuda.synchronize()
            assert int(out.cpu().numpy().view(cps.RESULT_DTYPE)["status"][0]) == 1
            again = sel.select_kth(torch.from_numpy(x).cuda(), n // 3)
            assert again == want
