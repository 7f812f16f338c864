"""The minibatch gradient's kernels at the sizes where a workgroup is ragged or the rule's line
lies: loss within 1e-5 of itself and gradient within 1e-4 of its largest entry (the bounds of the
general test, 67 + 64 float additions and up to 2^12 examples), and the same bits again."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("B", [2, 3, 4, 5, 7, 255, 257, 4095, 4096, 4097])
def test_sizes(B):
    import paper_1104_2732_amd as cps
    from oracle import mlp
    sel = cps.Selector(0)
    rng = np.random.default_rng(B)
    theta = (rng.standard_normal(mlp.N_PARAMS) * 0.1).astype(np.float32)
    theta[-1] = np.float32(math.log(0.3))
    F = rng.uniform(0.0, 0.2, size=(B, mlp.N_IN)).astype(np.float32)
    u = rng.uniform(0.0, 1.0, size=B).astype(np.float32)
    dev = [torch.from_numpy(a).cuda() for a in (theta, F, u)]
    print(f"case grad few B={B}", flush=True)
    loss, grad = sel.mlp_loss_grad(*dev)
    L, g = mlp.loss_and_grad(theta.astype(np.float64), F.astype(np.float64), u.astype(np.float64))
    assert abs(float(loss.cpu().numpy()[0]) - L) <= 1e-5 * abs(L)
    got = grad.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - g) <= 1e-4 * np.max(np.abs(g)) + 1e-4 * np.abs(g))
    loss2, grad2 = sel.mlp_loss_grad(*dev)
    assert torch.equal(grad, grad2) and torch.equal(loss, loss2)
    sel.close()
