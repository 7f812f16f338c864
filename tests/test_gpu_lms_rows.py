"""The filtered form where its kernels' shapes begin or end: chunks of 64 candidates, ragged segments,
more segments than the select holds at once (rows past 4096 segments of 256 or of 128), rows that a
candidate fits exactly (repeated zero squares) and a NaN: medians and trimmed sums against the
materialised form.  Values, counts and status exactly; the sums within n * 2^-53 of themselves (the
same non-negative squares, added in double in another order)."""
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


@pytest.mark.parametrize("n,p,m,kind", [
    (1 << 15, 3, 64, "plain"), ((1 << 15) + 63, 3, 65, "plain"), (40_000, 12, 130, "plain"),
    (40_001, 4, 129, "fit"), (65_537, 2, 70, "nan"), (50_000, 1, 1, "zero"),
    ((1 << 19) + 300, 11, 3, "plain"), ((1 << 20) + 77, 2, 2, "plain")])
def test_shapes(sel, n, p, m, kind):
    import paper_1104_2732_amd as cps
    X, y, _, betas = workloads.lms_problem(n, p, m, seed=n % 1000 + p)
    X, y, betas = X.copy(), y.copy(), betas.copy()
    if kind == "fit":  # 40 % of the rows are the first candidate's own
        b = betas[0]
        for i in range(0, n, 5):
            for j in (i, i + 1):
                if j < n:
                    s = X[j, 0] * b[0]
                    for q in range(1, p):
                        s = s + X[j, q] * b[q]
                    y[j] = s
    elif kind == "nan":
        y[n // 2 + 5] = np.nan
    elif kind == "zero":
        X[:] = 0.0
        y[: n - 100] = 0.0
    t = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, y, betas)]
    print(f"case lms rows n={n} p={p} m={m} {kind}", flush=True)
    a = sel.lms_median_sq_residuals(*t, cps.LMS_FILTERED)
    b = sel.lms_median_sq_residuals(*t, cps.LMS_MATERIALISED)
    for f in ("less", "equal", "greater", "status"):
        assert np.array_equal(a[f], b[f]), f
    if kind == "nan":
        assert np.all(a["status"] == cps.STATUS_NAN)
        return
    assert np.array_equal(a["value_bits"], b["value_bits"])
    a = sel.lts_trimmed_sq(*t, None, cps.LMS_FILTERED)
    b = sel.lts_trimmed_sq(*t, None, cps.LMS_MATERIALISED)
    for f in ("m", "below", "a", "b", "status"):
        assert np.array_equal(a[f], b[f]), f
    assert np.all(np.abs(a["F"] - b["F"]) <= n * 2.0 ** -53 * b["F"])
