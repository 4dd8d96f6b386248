"""A token's output bits in batches of other tokens (needs an MI355X).  fp32 layers and the streaming bf16 kernels start a
row's sums at a place that follows from the expert and the output columns alone, so which other tokens (and experts) a call
holds must not show; fp32 layers give the same bits in batches of another size too."""
import numpy as np
import pytest

import workloads
from helpers import DeviceLayer, HostLayer

pytestmark = pytest.mark.gpu

# fp32: short and long reductions (chains of one and of two); bf16: two-wave and four-wave streaming kernels of 8 chunks.
# (overrides, tokens of the two batches, tokens that they share: many in bf16, where rounding hides most differences)
CASES = [
    ("c1_tiny", dict(d=512, F=448, E=40, K=4, n_resident=20, R=8, H=8), 100, 37, 7),
    ("c1_tiny", dict(d=1024, F=1056, E=12, K=2, n_resident=9, R=8, H=8, n_shared=1), 150, 24, 7),
    ("c4_qwen3", dict(d=2048, F=768, E=24, K=4, n_resident=12), 16, 16, 10),
    ("c4_qwen3", dict(d=2048, F=768, E=24, K=4, n_resident=12, n_shared=1), 40, 40, 30),
    ("c2_mixtral_decode", dict(d=2048, F=1536, n_resident=5), 72, 72, 50),
]


@pytest.mark.parametrize("config,over,T,T2,n", CASES)
def test_rows_do_not_depend_on_the_rest_of_their_batch(config, over, T, T2, n):
    spec = workloads.scaled(config, **over)
    print("batch independence", config, over, T, T2, flush=True)
    host = HostLayer(spec, T, only_resident=True)
    other = HostLayer(spec, T2, stream=1, base=host)
    other.x[5:5 + n] = host.x[:n]
    dev = DeviceLayer(host, y_f32=True)
    a, b = dev.forward(), DeviceLayer(other, y_f32=True, base=dev).forward()
    np.testing.assert_array_equal(a["ids_remapped"][:n], b["ids_remapped"][5:5 + n])
    assert np.array_equal(a["y"][:n], b["y"][5:5 + n]), np.abs(a["y"][:n] - b["y"][5:5 + n]).max()
