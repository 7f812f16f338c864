"""Calls that leave the form open, below the filtered forms' sizes (2^15): they are the materialised
form's.  kNN means bit for bit (both in one fixed order), and the workspaces that such a call
leaves behind serve any smaller one under capture."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _knn(n, nq=40, dim=3):
    r = np.random.default_rng(n)
    P, f, Q = (r.standard_normal(s).astype(np.float32) for s in ((n, dim), n, (nq, dim)))
    f *= np.float32(10.0) ** r.uniform(-9, 9, n).astype(np.float32)  # (their sums round in double)
    return [torch.from_numpy(a).cuda() for a in (P, f, Q)]


def _lms(n, m=21):
    X, y, _, betas = workloads.lms_problem(n, 4, m, seed=n)
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, y, betas)]


@pytest.mark.parametrize("n", [8192, 12_345, 32_767])
def test_knn_means_are_the_materialised_ones(n):
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    t = _knn(n)
    for k in (5, 100, n // 3):
        print(f"case open knn n={n} k={k}", flush=True)
        a, b = s.knn_mean(*t, k), s.knn_mean(*t, k, cps.LMS_MATERIALISED)
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), k
    s.close()


def _captured(s, call, out):
    g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st), torch.cuda.graph(g, stream=st):
        call(out)
    torch.cuda.current_stream().wait_stream(st)
    for rep in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        yield out.cpu().numpy()
        _ = torch.arange(1000, device="cuda").sum().item()  # eager work between replays


def test_knn_smaller_call_under_capture():
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    s.knn_mean(*_knn(20_000), 7)
    t = _knn(6000)
    out = torch.zeros(t[2].shape[0] * cps.KNN_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    print("case open knn capture", flush=True)
    got = list(_captured(s, lambda o: s.knn_mean_async(*t, 7, o), out))
    want = s.knn_mean(*t, 7).view(np.uint8)
    assert all(np.array_equal(g, want) for g in got)
    s.close()


def test_lms_smaller_call_under_capture():
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    s.lms_median_sq_residuals(*_lms(20_000))
    t = _lms(9000)
    out = s.new_results(t[2].shape[0])
    print("case open lms capture", flush=True)
    got = list(_captured(s, lambda o: s.lms_median_sq_residuals_async(*t, o), out))
    want = s.lms_median_sq_residuals(*t).view(np.uint8)
    assert all(np.array_equal(g, want) for g in got)
    s.close()
