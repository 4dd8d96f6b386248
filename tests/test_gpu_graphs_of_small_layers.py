"""HIP graphs of the fp32 tiles, the router launch and the two-wave decode kernel: captured once, replayed with new inputs in
the same buffers and eager work in between, every replay equal to the eager result (needs an MI355X)."""
import numpy as np
import pytest

import workloads
from helpers import DeviceLayer, HostLayer, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over,T,kw", [
    ("c1_tiny", dict(), 16, dict(unique=True)),                                                     # fp32, one tile
    ("c4_qwen3", dict(d=256, F=96, dtype="f32"), 40, dict(unique=True, rho=1)),                     # fp32, router launch, several tiles
    ("c4_qwen3", dict(d=256, F=256), 8, dict(unique=True)),                                         # router launch, two-wave decode
    ("c4_qwen3", dict(d=256, F=256), 40, dict(beta=1.5)),                                           # routing, substitution and grouping apart
    ("c5_deepseek", dict(d=256, F=1408), 12, dict(rho=1)),                                          # two-wave decode, width of 128s
    ("c4_qwen3", dict(d=256, F=2048, E=16, K=4, n_resident=8), 12, dict()),                         # its split down projection
])
def test_replays_equal_eager(name, over, T, kw):
    import torch
    spec = workloads.scaled(name, **over)
    print("graph", name, over, T, kw, flush=True)
    hosts = [HostLayer(spec, T, stream=s) for s in (0, 1, 2)]
    dev = DeviceLayer(hosts[0], **kw)
    eager = []
    for h in hosts:
        dev.x.copy_(to_device(h.x))
        eager.append(dev.forward(debug=False)["y"].copy())
    assert not np.array_equal(eager[0], eager[1])

    def call():
        dev.bm.bm_moe_forward(dev.desc, dev.x, dev.weights, dev.bitmap, dev.table, dev.y, dev.workspace, None)

    side = torch.cuda.Stream()                                  # default priority
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rep in range(3):
        for i in (2, 0, 1):
            dev.x.copy_(to_device(hosts[i].x))
            dev.y.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(dev.y.float().cpu().numpy(), eager[i], err_msg=f"replay {rep} input {i}")
