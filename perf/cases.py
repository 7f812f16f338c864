"""The calls this library is measured on, over the sizes its users call it with.

Each case is a dict of plain values; ``prepare`` makes what a program holds before the call
(inputs on the GPU, the handle, the descriptors and the output records), ``run`` makes the
call through the public entry points and returns the records' fields, ``work`` counts what
the call cannot do without, and ``exact`` computes the same outputs in 64 bits with torch.

A selection's record also says how often the input was read (``passes``).  That is an account
of the work done, not part of the answer, so ``run`` does not return it.
"""
import math

import numpy as np
import torch

import paper_1104_2732_amd as cps

DEVICE = 0
DISTS = ("uniform", "normal", "cauchy", "quantized", "lognormal")
DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # a short vector's median, as a control loop or a robust scale estimate calls it again
        # and again: the launch and the chain of steps count, not the bandwidth
        dict(name="select_1000_f32", kind="select", n=1000, dtype="f32", dist="normal",
             rank=0.5, offset=0),
        # the small configuration of the benchmark: 2^20 uniform values
        dict(name="select_1m_f32", kind="select", n=1 << 20, dtype="f32", dist="uniform",
             rank=0.5, offset=0),
        # a double column of no round size, cut out of a larger buffer (8-byte aligned only),
        # its 1 % quantile
        dict(name="select_3m_odd_f64", kind="select", n=3_000_017, dtype="f64", dist="normal",
             rank=0.01, offset=1),
        # the smaller size of the single-array sweep, heavy tails
        dict(name="select_16m_f32", kind="select", n=1 << 24, dtype="f32", dist="cauchy",
             rank=0.5, offset=0),
        # the larger size of the sweep, float: the headline call
        dict(name="select_268m_f32", kind="select", n=1 << 28, dtype="f32", dist="normal",
             rank=0.5, offset=0),
        # the same in double with 1024 distinct values (sensor or price data): ties everywhere
        dict(name="select_268m_f64_ties", kind="select", n=1 << 28, dtype="f64",
             dist="quantized", rank=0.5, offset=0),
        # many medians at once, sizes log-uniform between 10^3 and 10^6 (groups of a table)
        dict(name="batched_4096_f32", kind="batched", count=4096, lo=1000, hi=1_000_000,
             dtype="f32", dist="lognormal", rank=0.5, ksum=False),
        # few large arrays (channels of a recording)
        dict(name="batched_64_large_f32", kind="batched", count=64, lo=1 << 22, hi=1 << 22,
             dtype="f32", dist="lognormal", rank=0.5, ksum=False),
        # least median of squares: elemental-subset candidates of a contaminated regression
        dict(name="lms_1024x1m", kind="lms", n=1 << 20, p=8, m=1024),
        # least trimmed squares on a ragged problem of another width
        dict(name="lts_300x200k", kind="lts", n=200_003, p=5, m=300),
        # k nearest neighbour regression
        dict(name="knn_1024x1m", kind="knn", n=1 << 20, dim=8, nq=1024, k=64),
        # one minibatch of the proposal network's training: forward and backward
        dict(name="mlp_grad_256", kind="grad", batch=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("select", "select", "select", "batched", "batched", "lms", "lts", "knn",
                       "grad"))
    if kind == "select":
        return dict(kind=kind, n=_log_int(rng, 1000, 1 << 28), dtype=rng.choice(("f32", "f64")),
                    dist=rng.choice(DISTS), rank=rng.choice((0.0, 0.01, 0.25, 0.5, 0.9, 1.0)),
                    offset=rng.randrange(4))
    if kind == "batched":
        hi = _log_int(rng, 10_000, 1 << 22)
        count = max(4, min(4096, _log_int(rng, 16, 4096), (1 << 29) // hi))
        return dict(kind=kind, count=count, lo=max(1, hi // rng.choice((1, 30, 1000))), hi=hi,
                    dtype=rng.choice(("f32", "f64")), dist=rng.choice(DISTS),
                    rank=rng.choice((0.1, 0.5, 0.9)), ksum=rng.random() < 0.3)
    if kind in ("lms", "lts"):
        return dict(kind=kind, n=_log_int(rng, 1000, 1 << 20), p=rng.randint(2, 10),
                    m=_log_int(rng, 16, 800))
    if kind == "knn":
        return dict(kind=kind, n=_log_int(rng, 4000, 1 << 20), dim=rng.randint(2, 8),
                    nq=_log_int(rng, 32, 1024), k=rng.choice((1, 5, 16, 64, 100)))
    return dict(kind=kind, batch=_log_int(rng, 32, 1024))


# ---------------------------------------------------------------- inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _values(dist, n, dtype, g):
    if dist == "uniform":
        return torch.rand(n, generator=g, device="cuda", dtype=dtype)
    if dist == "cauchy":  # tan(pi (u - 1/2)): heavy tails, every value finite
        u = torch.rand(n, generator=g, device="cuda", dtype=dtype).clamp_(1e-9, 1 - 1e-7)
        return u.sub_(0.5).mul_(math.pi).tan_()
    x = torch.randn(n, generator=g, device="cuda", dtype=dtype)
    if dist == "normal":
        return x
    if dist == "lognormal":
        return x.exp_()
    if dist == "quantized":  # 1024 levels of N(0, 1)
        return x.add_(4.0).mul_(128.0).floor_().clamp_(0, 1023).add_(0.5).div_(128.0).sub_(4.0)
    raise ValueError(dist)


def _rank(fraction, n):
    """1-based rank: the median at 0.5 (the lower one), the extremes at 0 and 1."""
    if fraction == 0.5:
        return (n + 1) // 2
    return min(n, max(1, int(fraction * n)))


def _regression(n, p, m, seed):
    """X ~ N(0, 1), 30 % of the rows shifted by +10; candidates solve p-row subsets."""
    g = _generator(seed)
    f64 = torch.float64
    X = torch.randn((n, p), generator=g, device="cuda", dtype=f64)
    beta = torch.randn(p, generator=g, device="cuda", dtype=f64)
    y = (X * beta).sum(1) + 0.1 * torch.randn(n, generator=g, device="cuda", dtype=f64)
    y += 10.0 * (torch.rand(n, generator=g, device="cuda") < 0.3)
    rows = torch.randint(0, n, (m, p), generator=g, device="cuda")
    A, b = X[rows].cpu().numpy(), y[rows].cpu().numpy()
    A = A + 1e-9 * np.eye(p)  # (a row drawn twice)
    betas = np.linalg.solve(A, b[..., None])[..., 0]
    return X, y.contiguous(), torch.from_numpy(np.ascontiguousarray(betas)).cuda()


def _points(n, dim, nq, seed):
    g = _generator(seed)
    P = torch.randn((n, dim), generator=g, device="cuda")
    Q = torch.randn((nq, dim), generator=g, device="cuda")
    f = torch.sin(P.sum(1)) + 0.1 * torch.randn(n, generator=g, device="cuda")
    return P, f, Q


def _examples(batch, seed):
    """Feature rows as the sketch forms them: cumulative fractions, two extremes, the rank."""
    g = _generator(seed)
    c = torch.rand((batch, 64), generator=g, device="cuda").pow_(3).cumsum(1)
    ends = torch.rand((batch, 2), generator=g, device="cuda") * 2 - 1
    rank = torch.rand((batch, 1), generator=g, device="cuda")
    feat = torch.cat([c / c[:, -1:], ends, rank], dim=1).contiguous()
    ustar = 0.05 * torch.randn(batch, generator=g, device="cuda")
    return feat, ustar


def _selections(out, count):
    """The fields of `count` selection records, as views of the record buffer."""
    words = out.view(torch.int64).view(count, 6)
    return {"value": out.view(torch.float64).view(count, 6)[:, 1], "counts": words[:, 2:5],
            "status": out.view(torch.int32).view(count, 12)[:, 11]}


def _inputs(case, seed):
    kind = case["kind"]
    if kind == "select":
        dt = DTYPES[case["dtype"]]
        x = _values(case["dist"], case["n"] + case["offset"], dt, _generator(seed))
        return x[case["offset"]:]
    if kind == "batched":
        dt = DTYPES[case["dtype"]]
        r = np.random.default_rng(seed)
        u = r.random(case["count"])
        sizes = np.floor(case["lo"] * (case["hi"] / case["lo"]) ** u).astype(np.int64)
        flat = _values(case["dist"], int(sizes.sum()), dt, _generator(seed))
        return list(torch.split(flat, sizes.tolist()))
    if kind in ("lms", "lts"):
        return _regression(case["n"], case["p"], case["m"], seed)
    if kind == "knn":
        return _points(case["n"], case["dim"], case["nq"], seed)
    return _examples(case["batch"], seed)


def prepare(case, seed):
    kind = case["kind"]
    data = _inputs(case, seed)
    sel = cps.Selector(DEVICE)
    st = {"case": case, "sel": sel, "data": data}
    if kind == "select":
        sel.reserve(data.numel(), cps.CPS_F32 if case["dtype"] == "f32" else cps.CPS_F64)
        st["k"] = _rank(case["rank"], case["n"])
        st["out"] = sel.new_results(1)
        st["fields"] = _selections(st["out"], 1)
    elif kind == "batched":
        ks = [_rank(case["rank"], a.numel()) for a in data]
        st["desc"] = sel.batch_descriptors(data, ks)
        sel.reserve_batched(st["desc"][3])
        st["out"] = sel.new_results(len(data))
        st["fields"] = _selections(st["out"], len(data))
        if case["ksum"]:
            st["ksum"] = torch.empty(len(data), dtype=torch.float64, device="cuda")
            st["fields"]["ksum"] = st["ksum"]
    elif kind == "lms":
        st["out"] = sel.new_results(case["m"])
        st["fields"] = _selections(st["out"], case["m"])
    elif kind == "lts":
        m = case["m"]
        st["out"] = torch.empty(m * cps.TRIM_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
        w = st["out"].view(torch.float64).view(m, 6)
        st["fields"] = {"F": w[:, 0], "m": w[:, 1],
                        "counts": st["out"].view(torch.int64).view(m, 6)[:, 2:5],
                        "status": st["out"].view(torch.int32).view(m, 12)[:, 10]}
    elif kind == "knn":
        nq = case["nq"]
        st["out"] = torch.empty(nq * cps.KNN_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
        st["fields"] = {"mean": st["out"].view(torch.float64).view(nq, 4)[:, 0],
                        "dk": st["out"].view(torch.float32).view(nq, 8)[:, 2],
                        "counts": st["out"].view(torch.int64).view(nq, 4)[:, 2:4],
                        "status": st["out"].view(torch.int32).view(nq, 8)[:, 3]}
    else:
        st["params"] = sel.mlp_init(7)
    return st


def run(st):
    case, sel, data = st["case"], st["sel"], st["data"]
    kind = case["kind"]
    if kind == "select":
        sel.select_kth_async(data, st["k"], st["out"])
    elif kind == "batched":
        ptrs, sizes, ks, code = st["desc"]
        if case["ksum"]:
            sel.select_kth_batched_ksum_async(ptrs, sizes, ks, len(data), code, st["out"],
                                              st["ksum"])
        else:
            sel.select_kth_batched_async(ptrs, sizes, ks, len(data), code, st["out"])
    elif kind == "lms":
        sel.lms_median_sq_residuals_async(*data, st["out"])
    elif kind == "lts":
        sel.lts_trimmed_sq_async(*data, (case["n"] + 1) // 2, st["out"])
    elif kind == "knn":
        sel.knn_mean_async(*data, case["k"], st["out"])
    else:
        loss, grad = sel.mlp_loss_grad(st["params"], *data)
        return {"loss": loss, "grad": grad}
    return st["fields"]


def work(case):
    kind = case["kind"]
    if kind == "select":
        es = 4 if case["dtype"] == "f32" else 8
        return {"bytes": case["n"] * es + 48, "flops": case["n"]}
    if kind == "batched":
        es = 4 if case["dtype"] == "f32" else 8
        lo, hi = case["lo"], case["hi"]
        mean = lo if lo == hi else (hi - lo) / math.log(hi / lo)
        total = int(mean * case["count"])
        return {"bytes": total * es + case["count"] * (24 + 48), "flops": total}
    if kind in ("lms", "lts"):  # p products, p - 1 sums, a difference and a square per residual
        n, p, m = case["n"], case["p"], case["m"]
        return {"bytes": 8 * (n * (p + 1) + m * p) + 48 * m, "flops": n * m * (2 * p + 1)}
    if kind == "knn":  # dim differences, dim squares and dim - 1 sums per distance
        n, d, nq = case["n"], case["dim"], case["nq"]
        return {"bytes": 4 * (n * (d + 1) + nq * d) + 32 * nq, "flops": n * nq * (3 * d - 1)}
    b = case["batch"]  # two hidden layers and an output layer: forward, dX and dW
    macs = 67 * 64 + 64 * 64 + 64 * 2
    return {"bytes": 4 * (b * 68 + 2 * cps.MLP_PARAMS + 1),
            "flops": 2 * b * (2 * macs + 64 * 64 + 64 * 2)}


# ---------------------------------------------------------------- the same in 64 bits


def _kth(x, k):
    """(value, counts) of the k-th smallest of a 1-d tensor."""
    v = torch.sort(x).values[k - 1] if x.numel() > 1 else x[0]
    less, equal = (x < v).sum(), (x == v).sum()
    return v.to(torch.float64) + 0.0, torch.stack([less, equal, x.numel() - less - equal])


def _records(values, counts):
    return {"value": torch.stack(values), "counts": torch.stack(counts),
            "status": torch.zeros(len(values), dtype=torch.int32, device="cuda")}


def _exact_grad(case, seed):
    feat, ustar = _examples(case["batch"], seed)
    sel = cps.Selector(DEVICE)
    p = sel.mlp_init(7).to(torch.float64).requires_grad_(True)
    x, u = feat.to(torch.float64), ustar.to(torch.float64)
    at, parts = 0, []
    for shape in ((64, 67), (64,), (64, 64), (64,), (2, 64), (2,)):
        size = int(np.prod(shape))
        parts.append(p[at:at + size].view(shape))
        at += size
    W1, b1, W2, b2, W3, b3 = parts
    h = torch.relu(x @ W1.T + b1)
    h = torch.relu(h @ W2.T + b2)
    o = h @ W3.T + b3
    d, w = o[:, 0] - u, torch.exp(torch.clamp(o[:, 1], -20.0, 4.0))
    loss = (100.0 * d * d + torch.relu(d.abs() - w) + 0.02 * w).mean()
    (grad,) = torch.autograd.grad(loss, p)
    return {"loss": loss.detach().reshape(1), "grad": grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "grad":
        return _exact_grad(case, seed)
    data = _inputs(case, seed)
    if kind == "select":
        v, c = _kth(data, _rank(case["rank"], case["n"]))
        return _records([v], [c])
    if kind == "batched":
        values, counts, sums = [], [], []
        for a in data:
            k = _rank(case["rank"], a.numel())
            v, c = _kth(a, k)
            values.append(v)
            counts.append(c)
            if case["ksum"]:
                b = a.to(torch.float64)
                sums.append(torch.where(b < v, b, 0.0).sum() + (k - c[0]) * v)
        out = _records(values, counts)
        if case["ksum"]:
            out["ksum"] = torch.stack(sums)
        return out
    if kind in ("lms", "lts"):
        X, y, betas = data
        n, h = case["n"], (case["n"] + 1) // 2
        values, counts, sums = [], [], []
        for b in betas:
            s = X[:, 0] * b[0]
            for j in range(1, case["p"]):
                s = s + X[:, j] * b[j]
            r = (y - s) ** 2
            v, c = _kth(r, h)
            values.append(v)
            counts.append(c)
            sums.append(torch.where(r < v, r, 0.0).sum() + (h - c[0]) * v)
        out = _records(values, counts)
        if kind == "lms":
            return out
        c = out["counts"]
        return {"F": torch.stack(sums), "m": out["value"],
                "counts": torch.stack([c[:, 0], h - c[:, 0], c[:, 1]], dim=1),
                "status": out["status"]}
    P, f, Q = (t.to(torch.float64) for t in data)
    means, dks = [], []
    for q in Q:
        d = ((P - q) ** 2).sum(1)
        near = torch.topk(d, case["k"], largest=False)
        means.append(f[near.indices].mean())
        dks.append(near.values[-1])
    # (the tie counts are those of the distances rounded to float: no value in 64 bits)
    return {"mean": torch.stack(means), "dk": torch.stack(dks), "counts": None,
            "status": torch.zeros(case["nq"], dtype=torch.int32, device="cuda")}
