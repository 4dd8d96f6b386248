"""The tiled bf16 projections at the edges of their tiles and of the pieces that tiles are cut into (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import DeviceLayer, HostLayer, err_metric

pytestmark = pytest.mark.gpu

# (overrides, tokens): reductions of 4 to 11 k-steps (an item's first loads, its look-up and its hand-over fall together
# in the shortest), widths that end inside a column tile, groups of a few rows to a few 256-row tiles with rests on both sides of
# 128, many groups, shared experts; then reductions of 64 and more k-steps, whose tiles are cut: both heights
# (below 128 routed rows an expert on average) and 256 rows only, one to sixteen column tiles, pieces of unequal length; up
# to 65 k-steps 3 and 4 pieces, then 6 and 7 of 256- and 128-row tiles, 7 of 256-row tiles alone, 8 of both heights, 8 of unequal
# length of 128-row tiles alone
CASES = [
    (dict(d=256, F=256, E=4, K=2, n_resident=4), 150),
    (dict(d=320, F=448, E=4, K=2, n_resident=2), 257),
    (dict(d=384, F=320, E=6, K=3, n_resident=5, n_shared=1), 129),
    (dict(d=512, F=704, E=40, K=4, n_resident=20), 385),
    (dict(d=640, F=576, E=100, K=8, n_resident=50), 640),
    (dict(d=1024, F=256, E=3, K=1, n_resident=1, R=2, H=2), 400),
    (dict(d=256, F=4096, E=8, K=2, n_resident=4), 200),
    (dict(d=256, F=4160, E=4, K=1, n_resident=3, R=3, H=3, n_shared=1), 300),
    (dict(d=1024, F=4096, E=8, K=2, n_resident=5), 500),
    (dict(d=1024, F=4160, E=8, K=2, n_resident=5), 530),
    (dict(d=4096, F=4096, E=8, K=2, n_resident=5), 150),
    (dict(d=256, F=4096, E=4, K=2, n_resident=4), 700),
    (dict(d=512, F=8192, E=8, K=2, n_resident=5), 300),
    (dict(d=512, F=8256, E=4, K=2, n_resident=4), 300),
    (dict(d=256, F=16384, E=16, K=2, n_resident=12), 300),
    (dict(d=256, F=16448, E=8, K=2, n_resident=5), 120),
]


@pytest.mark.parametrize("over,T", CASES)
def test_tiled_layer_matches_oracle(over, T):
    spec = workloads.scaled("c4_qwen3", **over)
    print("tiled edges", over, T, flush=True)
    host = HostLayer(spec, T, only_resident=True, poison=True)      # weights of absent experts are NaN
    ref = host.oracle_forward(oracle)
    dev = DeviceLayer(host)
    for fill in (0xA5, 0xFF):                                        # scratch holds nothing of use, and NaN
        dev.workspace.fill_(fill)
        out = dev.forward()
        np.testing.assert_array_equal(out["ids_remapped"], ref["ids_remapped"])
        e = err_metric(out["y"], ref["y"])
        print("   err", e, flush=True)
        assert e <= 2e-2, e                                          # bf16 rounding of h, o and y: the suite's bound


# launches of fewer tiles than units: every tile in as many column tiles as give each unit one, of 16 (32) columns up and of
# unequal widths, 256-row tiles in halves; tiles of at most half the width run on the narrow loop, from 6 k-steps on
FEW = [
    (dict(d=256, F=256, E=3, K=1, n_resident=3, R=2, H=2), 300),
    (dict(d=384, F=384, E=3, K=1, n_resident=2, R=2, H=2), 300),
    (dict(d=448, F=1344, E=4, K=2, n_resident=2, R=3, H=3), 260),
    (dict(d=1792, F=256, E=6, K=1, n_resident=5), 495),
    (dict(d=576, F=704, E=10, K=2, n_resident=6, n_shared=2), 131),
    (dict(d=2048, F=1408, E=16, K=4, n_resident=10, n_shared=1), 70),
]


@pytest.mark.parametrize("over,T", FEW)
def test_launches_of_few_tiles_match_oracle(over, T):
    test_tiled_layer_matches_oracle(over, T)
