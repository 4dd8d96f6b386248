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


# F = 2048 past 32 rows: two slices of the down projection's reduction, one where the workspace has no room for them;
# gate/up on two waves (8 experts) and on four (16); reductions of 1024 with few and with more groups, and their row limit
@pytest.mark.parametrize("over,T", [(dict(d=256, F=2048, E=8, K=4, n_resident=4), 9), (dict(d=256, F=2048, E=16, K=4, n_resident=8), 20),
                                    (dict(d=256, F=2048, E=16, K=4, n_resident=16), 8), (dict(d=1024, F=1024, E=8, K=2, n_resident=4), 2),
                                    (dict(d=1024, F=1024, E=8, K=2, n_resident=4), 3), (dict(d=1024, F=1024, E=4, K=1, n_resident=3, R=3, H=3), 32),
                                    (dict(d=1024, F=1024, E=4, K=2, n_resident=4, R=3, H=3), 17), (dict(d=384, F=1024, E=8, K=2, n_resident=4), 5)])
@pytest.mark.parametrize("pack", [False, True])
def test_whole_and_split_reductions(over, T, pack):
    import paper_2511_10054_amd as bm
    spec = workloads.scaled("c4_qwen3", **over)
    print("whole and split reductions", over, T, pack, flush=True)
    host = HostLayer(spec, T, only_resident=True, poison=True)
    ref = host.oracle_forward(oracle)
    dev = DeviceLayer(host, pack=pack)
    sizes = [dev.workspace.numel()]
    if spec.F == 2048 and T * spec.K > 32:
        sizes.append(sizes[0] - T * spec.K * spec.d * 4)
    for n in sizes:
        dev.workspace = dev.workspace[:n]
        dev.workspace.fill_(0xA5)
        out = dev.forward()
        np.testing.assert_array_equal(out["ids_remapped"], ref["ids_remapped"])
        assert err_metric(out["y"], ref["y"]) <= 2e-2
    with pytest.raises(bm.BuddyMoEError):
        dev.workspace = dev.workspace[:sizes[-1] - 256]
        dev.forward()
