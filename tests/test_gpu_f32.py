"""fp32 layers: the grouped fp32 tiles and the fp32 front kernel at the edges of their tiles (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import DeviceLayer, HostLayer, err_metric

pytestmark = pytest.mark.gpu

# fp32 sums over at most 512 values: measured errors are below 1e-6, the bound is the suite's (test_gpu_f32_chains.py
# has the long reductions, with one close to the measured error)
TOL = 1e-5

# (overrides, tokens): group sizes around 16, 32 and 64 rows, more than one 64-row tile of a group (the table lists a live
# group once, whatever the layer's average), expert counts of every front kernel, widths that are no multiple of 64, 4 (outputs) or
# 32 (reductions: the row-by-row kernel and the front kernel's checked loads), shared experts
CASES = [
    (dict(E=4, K=1, n_resident=1, R=3, H=3), 1),
    (dict(E=4, K=1, n_resident=1, R=3, H=3), 16),
    (dict(E=4, K=1, n_resident=1, R=3, H=3), 17),
    (dict(E=4, K=2, n_resident=2, R=3, H=3), 33),
    (dict(E=4, K=2, n_resident=2, R=3, H=3), 65),
    (dict(E=4, K=2, n_resident=4, R=3, H=3), 300),
    (dict(E=2, K=1, n_resident=2, R=1, H=1), 257),
    (dict(d=288, E=20, F=352, K=4, n_resident=10), 50),
    (dict(d=96, E=40, F=96, K=6, n_resident=20, n_shared=2), 37),
    (dict(d=512, E=100, F=64, K=8, n_resident=50), 129),
    (dict(d=64, E=200, F=32, K=8, n_resident=100), 70),
    (dict(d=66, E=8, F=96, K=2, n_resident=4), 20),
    (dict(d=32, E=8, F=70, K=2, n_resident=4), 40),
    (dict(d=77, E=130, F=33, K=3, n_resident=60, n_shared=1), 18),
    # a histogram that takes the one-workgroup scan, groups from one to a few hundred rows in no order of size
    (dict(d=32, E=256, F=32, K=1, R=8, H=8, n_resident=100, zipf_s=1.0, resident="alternate"), 2200),
]


@pytest.mark.parametrize("over,T", CASES)
@pytest.mark.parametrize("unique", [False, True])
def test_f32_layer_matches_oracle(over, T, unique):
    spec = workloads.scaled("c1_tiny", **over)
    print("f32 layer", over, T, unique, flush=True)
    host = HostLayer(spec, T, only_resident=True, poison=True)      # weights of absent experts are NaN
    ref = host.oracle_forward(oracle, unique=unique)
    dev = DeviceLayer(host, unique=unique)
    dev.workspace.fill_(0xA5)
    out = dev.forward()
    for k in ("ids", "ids_remapped"):
        np.testing.assert_array_equal(out[k], ref[k])
    for k, want in zip(("offsets", "perm", "inv_perm"), oracle.permute(ref["ids_remapped"], spec.E)):
        np.testing.assert_array_equal(out[k], want)
    e = err_metric(out["y"], ref["y"])
    print("   err", e, flush=True)
    assert e <= TOL, e
