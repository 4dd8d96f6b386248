"""fp32 projections of long reductions against the 64-bit result, with a bound close to what their summation tree gives (needs
an MI355X): both forms of the chain (below 1024 values and from 1024 on), folds that end inside and on an eighth k-step,
row tiles of 16, 32 and 64 rows and their neighbours."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import DeviceLayer, HostLayer, err_metric

pytestmark = pytest.mark.gpu

# One rounding is 2^-24 = 6e-8.  A value passes some 15 of them in a row (chains of one or two, pairs, eight k-steps, the folds,
# the two halves), falling at random, in each of two projections: about 3e-7, the largest of some 10^5 values three to four
# times that (measured: 5e-7 to 9.5e-7).  One chain over the whole reduction, as a plain loop has it, gives 3.9e-6 at 1024
# and 5.5e-6 at 2048 values, so losing the tree fails.
TOL = 2e-6


# K = 1 and one resident expert: the group is as large as the batch
@pytest.mark.parametrize("d,F", [(992, 1056), (1024, 1024), (1056, 992), (2048, 2048), (2048, 96)])
@pytest.mark.parametrize("T", [1, 16, 17, 32, 33, 64, 65])
def test_long_fp32_reductions(d, F, T):
    spec = workloads.scaled("c1_tiny", d=d, F=F, E=4, K=1, n_resident=1, R=3, H=3)
    print("fp32 chains", d, F, T, flush=True)
    host = HostLayer(spec, T, only_resident=True, poison=True)
    ref = host.oracle_forward(oracle)
    out = DeviceLayer(host).forward()
    np.testing.assert_array_equal(out["ids_remapped"], ref["ids_remapped"])
    e = err_metric(out["y"], ref["y"])
    print("   err", e, flush=True)
    assert e <= TOL, e


# Live groups whose weights outgrow the 256 MB memory-side cache (csrc/bm_dispatch_rules.h): groups of at most 64 rows, one row tile,
# load them non-temporally, by copies of the tiles of their own, larger groups do not.  One group of 270 MB with chains of two,
# two of 178 MB (a shared expert, which takes every token as well) with chains of one in either projection.  The bound is the one
# above: a reduction of 15968 values has three more levels of folds than one of 2048 (measured: up to 1.2e-6).
@pytest.mark.parametrize("d,F,n_shared", [(2048, 11008, 0), (928, 15968, 1), (15968, 928, 1)])
def test_fp32_weights_past_the_memory_side_cache(d, F, n_shared):
    assert (1 + n_shared) * 12 * d * F > 256 << 20
    spec = workloads.scaled("c1_tiny", d=d, F=F, E=4, K=1, n_resident=1, R=3, H=3, n_shared=n_shared)
    host = dev = None
    for T in (1, 16, 17, 32, 33, 64, 65, 130):
        print("fp32 past the cache", d, F, T, flush=True)
        host = HostLayer(spec, T, only_resident=True, poison=True, base=host)
        rows = np.unique([0, T // 2, T - 1])                         # tokens are independent: the oracle takes three
        ref = host.oracle_forward(oracle, rows=rows)
        dev = DeviceLayer(host, base=dev)
        out = dev.forward()
        np.testing.assert_array_equal(out["ids_remapped"][rows], ref["ids_remapped"])
        e = err_metric(out["y"][rows], ref["y"])
        print("   err", e, flush=True)
        assert e <= TOL, e
