"""A tree freed while a HIP graph is captured, on the stream that the tree was
built on or on another one: the capture goes on, the graph replays, and the
freed memory serves later calls."""
import numpy as np
import pytest

import oracle
from paper_2604_05885_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def jz():
    from paper_2604_05885_amd import api
    return api


@pytest.mark.parametrize("n", [1000, 20000])
@pytest.mark.parametrize("built_on", ["captured", "other", "default"])
@pytest.mark.parametrize("mode", ["global", "thread_local"])
def test_free_under_capture(jz, n, built_on, mode):
    side = torch.cuda.Stream()
    stream = {"captured": side, "other": torch.cuda.Stream(),
              "default": torch.cuda.default_stream()}[built_on]
    p = inputs.clustered(n, max(1, n // 900), 71)
    d = torch.from_numpy(p).cuda()
    torch.cuda.synchronize()
    t = jz.jz_build(d, stream=stream)
    t.knn_fof(8, inputs.linking_length(n, 0.2), stream=stream)
    x = torch.ones(1000, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side, capture_error_mode=mode):
        x.mul_(2)
        t.free()
        x.add_(1)
    want = 1.0
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        want = 2 * want + 1
        assert torch.equal(x, torch.full_like(x, want))
        x.mul_(0.5)
        want *= 0.5
        torch.cuda.synchronize()
    with jz.jz_build(d) as t:
        i, _ = t.knn(8)
        assert np.array_equal(i.cpu().numpy(), oracle.knn_bf(p, 8)[0])
