"""The form that is taken when the caller leaves it open, just below and from each rule's line on, at
the ends of the ranks: against the materialised form.  Values, counts and status exactly; sums and means
within the roundings of as many double additions."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sel():
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    yield s
    s.close()


@pytest.mark.parametrize("n", [8191, 8192, 8193, 12_345, 32_767])
def test_knn(sel, n):
    import paper_1104_2732_amd as cps
    r = np.random.default_rng(n)
    P = r.standard_normal((n, 3)).astype(np.float32)
    P[n // 2: n // 2 + 40] = P[0]  # repeated distances
    f = r.standard_normal(n).astype(np.float32)
    Q = np.concatenate([r.standard_normal((20, 3)), P[:1]]).astype(np.float32)
    t = [torch.from_numpy(a).cuda() for a in (P, f, Q)]
    for k in (1, 7, 300, n // 2, n - 1, n):
        print(f"case auto knn n={n} k={k}", flush=True)
        a, b = sel.knn_mean(*t, k), sel.knn_mean(*t, k, cps.LMS_MATERIALISED)
        for x in a.dtype.names:
            if x not in ("mean",):
                assert np.array_equal(a[x], b[x]), (x, k)
        assert np.all(np.abs(a["mean"] - b["mean"]) <= 4 * k * 2.0 ** -53 * np.abs(f).max())


@pytest.mark.parametrize("n", [16_383, 16_384, 16_385, 25_001, 32_767])
def test_lms_lts(sel, n):
    import paper_1104_2732_amd as cps
    X, y, _, betas = workloads.lms_problem(n, 4, 21, seed=n)
    t = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, y, betas)]
    print(f"case auto lms n={n}", flush=True)
    a, b = sel.lms_median_sq_residuals(*t), sel.lms_median_sq_residuals(*t, cps.LMS_MATERIALISED)
    for x in ("value_bits", "less", "equal", "greater", "status"):
        assert np.array_equal(a[x], b[x]), x
    for h in (1, (n + 1) // 2, n - 1, n):
        print(f"case auto lts n={n} h={h}", flush=True)
        a, b = sel.lts_trimmed_sq(*t, h), sel.lts_trimmed_sq(*t, h, cps.LMS_MATERIALISED)
        for x in ("m", "below", "a", "b", "status"):
            assert np.array_equal(a[x], b[x]), (x, h)
        assert np.all(np.abs(a["F"] - b["F"]) <= n * 2.0 ** -53 * b["F"])
