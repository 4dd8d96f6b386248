"""The router product in a launch of its own: widths, expert counts and token counts around its tiles and its rule
(needs an MI355X)."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import DeviceLayer, HostLayer, err_metric

pytestmark = pytest.mark.gpu

TOL = {"bf16": 2e-2, "f32": 1e-5}          # the suite's bounds

# hidden widths of less than, exactly and more than one batch of the eight waves, and with a partial last batch; expert
# counts around 16-expert tiles and the rule's edge; token counts around 16-token tiles and past the rule
CASES = [
    ("c4_qwen3", dict(d=256, F=256, E=65, n_resident=30), 1),
    ("c4_qwen3", dict(d=2048, F=128, E=80, n_resident=40), 17),
    ("c4_qwen3", dict(d=2336, F=64, E=129, n_resident=60), 33),
    ("c4_qwen3", dict(d=288, F=64, E=256, n_resident=100), 64),
    ("c4_qwen3", dict(d=288, F=64, E=128), 65),
    ("c4_qwen3", dict(d=256, F=64, E=64, n_resident=30), 16),
    ("c4_qwen3", dict(d=288, F=64, E=33, n_resident=16, dtype="f32"), 19),
    ("c4_qwen3", dict(d=64, F=96, E=200, n_resident=90, dtype="f32"), 40),
    ("c4_qwen3", dict(d=32, F=4, E=128, K=2, dtype="f32"), 16),       # no room for the logits: product in the front kernel
]


@pytest.mark.parametrize("name,over,T", CASES)
@pytest.mark.parametrize("unique", [False, True])
def test_router_launch_matches_oracle(name, over, T, unique):
    spec = workloads.scaled(name, **over)
    print("router launch", name, over, T, unique, flush=True)
    host = HostLayer(spec, T, only_resident=True, poison=True)
    ref = host.oracle_forward(oracle, unique=unique)
    dev = DeviceLayer(host, unique=unique)
    dev.workspace.fill_(0xA5)
    out = dev.forward()
    for k in ("ids", "ids_remapped"):
        np.testing.assert_array_equal(out[k], ref[k])
    np.testing.assert_allclose(out["w"], ref["w"], rtol=2e-5, atol=1e-7)
    e = err_metric(out["y"], ref["y"])
    print("   err", e, flush=True)
    assert e <= TOL[spec.dtype], e
