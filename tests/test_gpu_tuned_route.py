"""A batched call without options on a tuned handle runs the choice that the autotuner kept.

The tuning batch's sampled positions hold one value and the rest another distribution, so every
sampled bracket misses: the kept choice is one without the bracket, which on ordinary data reads
an array more than once.  The default selection, which an untuned handle runs, reads each
once; `passes` tells them apart."""
import numpy as np
import pytest

from tests.test_gpu_one_read import make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_tuned_choice_is_taken(oracle_mod):
    import paper_1104_2732_amd as cps
    # (whole 16-byte vectors between the runs, and too small for several workgroups an array)
    n, count = 1 << 16, 1024
    hidden = make("hidden", n, np.float32, 1)
    assert (hidden[(np.arange(n) % (n // 256)) < 16] == 7.0).all()
    data = torch.from_numpy(hidden).cuda()
    plain = [make("normal", n, np.float32, 2 + i) for i in range(8)]
    dev = [torch.from_numpy(x).cuda() for x in plain]
    ks = [(n + 1) // 2] * len(plain)
    s = cps.Selector(0)
    try:
        untuned = s.select_kth_batched(dev, ks)
        assert (untuned["passes"] == 1).all()
        ptrs, sizes, kk, code = s.batch_descriptors([data] * count, [n // 3] * count)
        out = s.new_results(count)
        print("case autotune where every sampled bracket misses", flush=True)
        best, _ = s.autotune_batched(ptrs, sizes, kk, count, code, out)
        assert best.proposal == 0, "the batch no longer rules the sampled bracket out"
        print("case tuned handle, ordinary data", flush=True)
        tuned, explicit = s.select_kth_batched(dev, ks), s.select_kth_batched(dev, ks, best)
        assert (explicit["passes"] > 1).all()
        assert np.array_equal(tuned["passes"], explicit["passes"])
        for r in (tuned, explicit):
            for f in ("value_bits", "less", "equal", "greater", "status"):
                assert np.array_equal(r[f], untuned[f]), f
    finally:
        s.close()
