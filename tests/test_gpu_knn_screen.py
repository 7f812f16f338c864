"""The kNN filter's matrix screen at the edges of its shapes: one point past a tile or a
segment, every number of matrix instructions per tile, one query up to several workgroups of
them, and data that the screen's margin has to stand: far from the origin, with a few huge
coordinates, clustered, on a grid (ties), with NaN and infinite points.

The filtered form (which takes the screen for these ranks) against the materialised form,
which forms every distance: the k-th distance bit for bit, the counts and the status exactly,
and the mean ordinate within k * 2^-53 of the mean absolute ordinate scale (both add the same
k float ordinates in double, in different orders)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sel():
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    yield s
    s.close()


def _points(kind, n, dim, nq, rng):
    P = rng.standard_normal((n, dim)).astype(np.float32)
    Q = rng.standard_normal((nq, dim)).astype(np.float32)
    if kind == "far":          # spread 1 around 4096: cancellation without the centre
        P, Q = P + np.float32(4096), Q + np.float32(4096)
    elif kind == "huge":       # a few coordinates whose squares leave the screened range
        P[rng.integers(0, n, 5), rng.integers(0, dim, 5)] = np.float32(3e18)
        P[rng.integers(0, n, 5), rng.integers(0, dim, 5)] = np.float32(-1e25)
        Q[0, 0] = np.float32(2e19)
    elif kind == "clusters":   # spread 1e-3 inside clusters 100 apart
        c = rng.integers(0, 5, n)
        P = (P * np.float32(1e-3) + c[:, None] * np.float32(100)).astype(np.float32)
        Q = (Q * np.float32(1e-3) + rng.integers(0, 5, nq)[:, None] * np.float32(100)).astype(np.float32)
    elif kind == "grid":
        P, Q = np.rint(P * 2).astype(np.float32), np.rint(Q * 2).astype(np.float32)
    elif kind == "inf":
        P[rng.integers(0, n, 3), rng.integers(0, dim, 3)] = np.inf
    return P, Q


CASES = [("normal", 1 << 15, 8, 1), ("normal", (1 << 15) + 1, 1, 33), ("normal", 65_535, 4, 64),
         ("normal", 40_001, 5, 65), ("normal", 33_000, 10, 129), ("normal", 33_000, 11, 257),
         ("normal", 50_021, 16, 513), ("far", 40_000, 8, 100), ("huge", 40_003, 3, 40),
         ("clusters", 40_000, 6, 70), ("grid", 45_000, 4, 130), ("inf", 33_333, 7, 36)]


@pytest.mark.parametrize("kind,n,dim,nq", CASES)
def test_screen_against_materialised(sel, kind, n, dim, nq):
    import paper_1104_2732_amd as cps
    rng = np.random.default_rng(n + dim + nq)
    P, Q = _points(kind, n, dim, nq, rng)
    f = rng.standard_normal(n).astype(np.float32)
    Pd, Qd, fd = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (P, Q, f))
    for k in (1, 17, n // 200):
        print(f"case knn screen {kind} n={n} dim={dim} nq={nq} k={k}", flush=True)
        a = sel.knn_mean(Pd, fd, Qd, k, cps.LMS_FILTERED)
        b = sel.knn_mean(Pd, fd, Qd, k, cps.LMS_MATERIALISED)
        for field in ("status", "below", "equal"):
            assert np.array_equal(a[field], b[field]), field
        assert np.array_equal(a["dk"].view(np.uint32), b["dk"].view(np.uint32))
        ok = b["status"] == 0
        bound = 2.0 * k * 2.0 ** -53 * np.abs(f).max()
        assert np.all(np.abs(a["mean"][ok] - b["mean"][ok]) <= bound)


def test_nan_point_reaches_every_query(sel):
    import paper_1104_2732_amd as cps
    n, dim, nq = 40_000, 8, 70
    rng = np.random.default_rng(1)
    P, Q = _points("normal", n, dim, nq, rng)
    P[n - 1, 3] = np.nan
    f = np.zeros(n, dtype=np.float32)
    print("case knn screen NaN point", flush=True)
    r = sel.knn_mean(*(torch.from_numpy(v).cuda() for v in (P, f, Q)), 5, cps.LMS_FILTERED)
    assert np.all(r["status"] == cps.STATUS_NAN)
