"""The margin of the kNN filter's matrix screen, emulated on the CPU: for points and queries of
many scales and offsets, a pair whose distance (float, fixed order) lies below b must never be
ruled out.  The emulation splits every value in two bfloat16 parts as the kernel does, forms
the screen's terms in double precision and then moves the sum up by the largest error the
matrix instruction's float additions may make (50 additions of 2^-22 of the terms' absolute
sum), the worst case for a pair that must pass."""
import numpy as np
import pytest


def bf16(x):
    """float32 rounded to bfloat16 (nearest, ties to even), widened again."""
    b = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)
    r = (b + np.uint32(0x7FFF) + ((b >> np.uint32(16)) & np.uint32(1))) & np.uint32(0xFFFF0000)
    return r.view(np.float32)


def split(x):
    hi = bf16(x)
    return hi.astype(np.float64), bf16(x - hi).astype(np.float64)


def exact_order(P, q):
    d = None
    for j in range(P.shape[1]):
        e = P[:, j] - q[j]
        d = e * e if d is None else d + e * e
    return d


@pytest.mark.parametrize("dim", [1, 2, 5, 8, 16])
@pytest.mark.parametrize("scale,offset", [(1.0, 0.0), (1e-3, 50.0), (1e6, 0.0), (1e-9, 0.0)])
def test_a_pair_below_b_always_passes(dim, scale, offset):
    rng = np.random.default_rng(dim)
    n, nq = 4000, 12
    P = (rng.standard_normal((n, dim)) * scale + offset).astype(np.float32)
    Q = (rng.standard_normal((nq, dim)) * scale + offset).astype(np.float32)
    Q[: nq // 2] = P[rng.integers(0, n, nq // 2)] * np.float32(1 + 1e-6)  # near a point
    centre = P[:64].astype(np.float64).mean(0).astype(np.float32)
    p = P - centre
    margin, u = 2.0 ** -14, 2.0 ** -24
    norm = np.zeros(n, dtype=np.float32)
    for j in range(dim):
        norm = norm + p[:, j] * p[:, j]
    nhi, nlo = split(norm * np.float32(1 - margin))
    phi, plo = split(p)
    for q in Q:
        d = exact_order(P, q)
        e = q - centre
        qhi, qlo = split(np.float32(-2) * e)
        terms = np.concatenate([phi * qhi, phi * qlo, plo * qhi, nhi[:, None], nlo[:, None]], axis=1)
        worst = terms.sum(1) + 50 * 2.0 ** -22 * np.abs(terms).sum(1)
        n2 = float(np.sum(e.astype(np.float64) ** 2))
        for b in np.sort(d)[[1, 5, 50, n // 2]]:
            v = float(b) * (1 + (dim + 8) * u) - n2 * (1 - margin) + 1e-36
            T = np.float32(v + abs(v) * 2.0 ** -23)
            assert np.all(worst[d < b] <= T)
