"""What cps_reserve takes for a selection that one workgroup's registers hold, or that few
workgroups share: the split buffers (two of about n elements), and at most 4 MiB for
everything else (counters, partials, gather buffers; device memory comes in 2 MiB pieces)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def first_use():
    """The runtime takes memory of its own at a process's first allocation and fill."""
    import paper_1104_2732_amd as cps
    s = cps.Selector(0)
    s.reserve(1000, 0)
    torch.cuda.synchronize()
    s.close()


@pytest.mark.parametrize("n", [1000, 32_768, 65_537])
@pytest.mark.parametrize("dtype", [0, 1])
def test_reserve_takes_what_the_size_needs(n, dtype):
    import paper_1104_2732_amd as cps
    torch.cuda.synchronize()
    s = cps.Selector(0)
    before = torch.cuda.mem_get_info()[0]
    s.reserve(n, dtype)
    took = before - torch.cuda.mem_get_info()[0]
    print(f"case reserve n={n} dtype={dtype} took {took}", flush=True)
    assert took <= 2 * n * (4, 8)[dtype] + (4 << 20)
    s.close()
