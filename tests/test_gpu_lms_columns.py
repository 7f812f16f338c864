"""The filter's instance for every number of columns: medians and trimmed sums of the filtered
form against the materialised form, at the smallest filtered size and one row past it.  Values,
counts and status exactly; the trimmed sum within n * 2^-53 of itself (both forms add the same
non-negative squares in double, in different orders)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sel():
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    yield s
    s.close()


@pytest.mark.parametrize("p", list(range(1, 17)))
def test_every_column_count(sel, p):
    import paper_1104_2732_amd as cps
    n, m = (1 << 15) + p % 2, 5 + p
    X, y, _, betas = workloads.lms_problem(n, p, m, seed=p)
    t = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, y, betas)]
    print(f"case lms columns p={p} n={n} m={m}", flush=True)
    a = sel.lms_median_sq_residuals(*t, cps.LMS_FILTERED)
    b = sel.lms_median_sq_residuals(*t, cps.LMS_MATERIALISED)
    for f in ("value_bits", "less", "equal", "greater", "status"):
        assert np.array_equal(a[f], b[f]), f
    a = sel.lts_trimmed_sq(*t, None, cps.LMS_FILTERED)
    b = sel.lts_trimmed_sq(*t, None, cps.LMS_MATERIALISED)
    for f in ("m", "below", "a", "b", "status"):
        assert np.array_equal(a[f], b[f]), f
    assert np.all(np.abs(a["F"] - b["F"]) <= n * 2.0 ** -53 * b["F"])
