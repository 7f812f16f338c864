"""k nearest neighbours under capture on a handle whose workspace holds the plain filter but not the
screen's operands (its earlier call had few points, or a rank that the screen does not take):
the capture is accepted, and every replay gives the materialised form's distances and counts
exactly, its means within the roundings of k double additions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("warm_n,warm_k", [(1 << 15, 3), (1 << 19, 1 << 16)])
def test_capture_after_a_call_without_the_screen(warm_n, warm_k):
    import paper_1104_2732_amd as cps
    n, dim, nq, k = 1 << 19, 8, 4, 5
    r = np.random.default_rng(warm_n)
    P = torch.from_numpy(r.standard_normal((n, dim)).astype(np.float32)).cuda()
    f = torch.from_numpy(r.standard_normal(n).astype(np.float32)).cuda()
    Q = torch.from_numpy(r.standard_normal((nq, dim)).astype(np.float32)).cuda()
    ref = cps.Selector(0)
    want = ref.knn_mean(P, f, Q, k, cps.LMS_MATERIALISED)
    ref.close()
    s = cps.Selector(0)
    out = torch.zeros(nq * cps.KNN_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    print(f"case knn capture warm n={warm_n} k={warm_k}", flush=True)
    s.knn_mean(P[:warm_n], f[:warm_n], Q, warm_k)
    g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st), torch.cuda.graph(g, stream=st):
        s.knn_mean_async(P, f, Q, k, out)
    torch.cuda.current_stream().wait_stream(st)
    for rep in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(cps.KNN_DTYPE)
        for x in ("dk", "status", "below", "equal"):
            assert np.array_equal(got[x], want[x]), (x, rep)
        bound = 4 * k * 2.0 ** -53 * float(f.abs().max())
        assert np.all(np.abs(got["mean"] - want["mean"]) <= bound)
        _ = (P * 2).sum().item()  # eager work between replays
    s.close()
