"""A default call leaves a workspace that serves any other call of its size under capture, with
options or with a trace, and so do a small call's megabyte those that need no more: of few
elements, or of many with options that need no split buffers.  Each replay gives the default
call's result."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def replays(s, x, k, want, **kw):
    import paper_1104_2732_amd as cps
    out = s.new_results(1)
    g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st), torch.cuda.graph(g, stream=st):
        s.select_kth_async(x, k, out, **kw)
    torch.cuda.current_stream().wait_stream(st)
    for rep in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(cps.RESULT_DTYPE)[0]
        for f in ("value_bits", "less", "equal", "greater", "status"):
            assert got[f] == want[f], (rep, f)
        _ = (x * 2).sum().item()  # eager work between replays


@pytest.mark.parametrize("n,kw", [(70_000, {}), (70_000, dict(count_first=0)),
                                  (1 << 22, dict(partition_fraction=0.0)),
                                  (1 << 22, dict(partition_fraction=0.0, hist_bits=0))])
def test_capture_after_a_small_call(n, kw):
    import paper_1104_2732_amd as cps
    x = torch.from_numpy(np.random.default_rng(n).standard_normal(n).astype(np.float32)).cuda()
    ref = cps.Selector(0)
    want = ref.select_kth(x, n // 3)
    ref.close()
    s = cps.Selector(0)
    s.select_kth(x[:1000], 500)
    print(f"case {kw} of {n} captured after a call of 1000", flush=True)
    replays(s, x, n // 3, want, options=cps.default_options(**kw))
    s.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1000, 30_000, 100_000])
def test_capture_after_a_default_call(n, dtype):
    import paper_1104_2732_amd as cps
    x = torch.from_numpy(np.random.default_rng(n).standard_normal(n).astype(dtype)).cuda()
    k = n // 3
    calls = {"options": dict(options=cps.default_options(hist_bits=0)),
             "trace": dict(stats=None), "default": dict()}
    for name, kw in calls.items():
        s = cps.Selector(0)
        want = s.select_kth(x, k)
        if "stats" in kw:
            kw["stats"] = s.new_stats()
        out = s.new_results(1)
        print(f"case {name} captured after a default call n={n}", flush=True)
        g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st), torch.cuda.graph(g, stream=st):
            s.select_kth_async(x, k, out, **kw)
        torch.cuda.current_stream().wait_stream(st)
        for rep in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            got = out.cpu().numpy().view(cps.RESULT_DTYPE)[0]
            for f in ("value_bits", "less", "equal", "greater", "status"):
                assert got[f] == want[f], (name, rep, f)
            _ = (x * 2).sum().item()  # eager work between replays
        s.close()
