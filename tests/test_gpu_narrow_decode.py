"""The two-wave streaming decode kernel at the edges of its range (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import DeviceLayer, HostLayer, err_metric

pytestmark = pytest.mark.gpu

# bf16 rounding of h, o and y: the suite's bound for bf16 layers
TOL = 2e-2

# groups of one row, of 16 and 17, of 32, of more than 32 (a second pass; a token may hold a substitute twice); reductions
# of one chunk of 128, an odd number of them, chunks of 256; weight rows that are no multiple of the block of 32; shared
# experts; the last token count of each rule and the first one past it
CASES = [
    ("c4_qwen3", dict(d=256, F=256), 16),
    ("c4_qwen3", dict(d=384, F=128), 32),
    ("c4_qwen3", dict(d=256, F=640, E=16, K=4, n_resident=1), 32),
    ("c4_qwen3", dict(d=256, F=640, E=16, K=4, n_resident=2), 33),
    ("c5_deepseek", dict(d=256, F=1408), 5),
    ("c5_deepseek", dict(d=256, F=1408), 16),
    ("c5_deepseek", dict(d=256, F=1408), 17),
    ("c5_deepseek", dict(d=640, F=384, E=8, K=2, n_resident=1), 16),
    ("c4_qwen3", dict(d=512, F=768), 9),
]


@pytest.mark.parametrize("name,over,T", CASES)
@pytest.mark.parametrize("pack", [False, True])
def test_narrow_decode_matches_oracle(name, over, T, pack):
    spec = workloads.scaled(name, **over)
    print("narrow decode", name, over, T, pack, flush=True)
    host = HostLayer(spec, T, only_resident=True, poison=True)
    ref = host.oracle_forward(oracle)
    dev = DeviceLayer(host, pack=pack)
    dev.workspace.fill_(0xA5)
    out = dev.forward()
    np.testing.assert_array_equal(out["ids_remapped"], ref["ids_remapped"])
    assert np.isfinite(out["y"]).all()
    e = err_metric(out["y"], ref["y"])
    print("   err", e, flush=True)
    assert e <= TOL, e
