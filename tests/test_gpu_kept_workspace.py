"""One workspace, sized for the largest batch of a loop, over falling and rising batch sizes (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import DeviceLayer, HostLayer, err_metric

pytestmark = pytest.mark.gpu


# widths that are no multiple of 256: 11 to 16 tokens stream where the workspace has room and are tiled in one kept for
# 17 to 25; widths that are: the decode path throughout
@pytest.mark.parametrize("name,over", [("c5_deepseek", dict(d=256, F=1408)), ("c5_deepseek", dict(d=1024, F=384)),
                                       ("c4_qwen3", dict(d=256, F=256))])
@pytest.mark.parametrize("most", [17, 25, 64])
def test_one_workspace_for_all_batches(name, over, most):
    spec = workloads.scaled(name, **over)
    base, kept = None, None
    for T in (most, 16, 11, 3, 1, 16):
        print("kept workspace", name, over, most, T, flush=True)
        host = HostLayer(spec, T, only_resident=True, poison=True, base=base)
        dev = DeviceLayer(host)
        if kept is None:
            base, kept = host, dev.workspace
            kept.fill_(0xA5)
        dev.workspace = kept
        ref, out = host.oracle_forward(oracle), dev.forward()
        np.testing.assert_array_equal(out["ids_remapped"], ref["ids_remapped"])
        assert err_metric(out["y"], ref["y"]) <= 2e-2          # bf16 rounding of h, o and y: the suite's bound
