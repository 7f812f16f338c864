"""The workspace that a gradient of one minibatch leaves behind serves every smaller one: a call
captured after a larger one is accepted, and each replay gives the eager call's bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("warm,count", [(4097, 4096), (8000, 3000), (4096, 31)])
def test_smaller_minibatch_under_capture(warm, count):
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    r = np.random.default_rng(warm)
    F = torch.from_numpy(r.uniform(0.0, 0.2, (warm, 67)).astype(np.float32)).cuda()
    u = torch.from_numpy(r.uniform(0.0, 1.0, warm).astype(np.float32)).cuda()
    P = s.mlp_init(3)
    print(f"case grad capture {warm} then {count}", flush=True)
    s.mlp_loss_grad(P, F, u)
    F, u = F[:count], u[:count]
    g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st), torch.cuda.graph(g, stream=st):
        loss, grad = s.mlp_loss_grad(P, F, u)
    torch.cuda.current_stream().wait_stream(st)
    got = []
    for _ in range(3):
        loss.zero_()
        grad.zero_()
        g.replay()
        torch.cuda.synchronize()
        got.append((loss.clone(), grad.clone()))
    want = s.mlp_loss_grad(P, F, u)
    for a, b in got:
        assert torch.equal(a, want[0]) and torch.equal(b, want[1])
    s.close()
