"""Arrays of 4-byte values that do not start on a 16-byte boundary (a view into a larger array): the kernels that fetch 16
bytes at a time leave them to 4-byte accesses (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import DeviceLayer, HostLayer, err_metric, to_device

pytestmark = pytest.mark.gpu


def _shifted(t, by):
    """The same tensor `by` elements past a 16-byte boundary, with poison around it."""
    import torch
    if t is None:
        return None
    room = torch.full((t.numel() + 8,), -77 if t.dtype == torch.int32 else float("nan"), dtype=t.dtype, device=t.device)
    view = room[by:by + t.numel()].view(t.shape)
    view.copy_(t)
    assert view.data_ptr() % 16 == 4 * by
    return view


@pytest.mark.parametrize("by", [1, 2, 3])
@pytest.mark.parametrize("T,E,K", [(1, 8, 1), (1, 40, 2), (2, 200, 3), (257, 128, 3), (300, 64, 8)])
def test_distribution_gate_reads_ids_at_any_offset(T, E, K, by):
    import torch
    import paper_2511_10054_amd as bm
    print("unaligned ids", T, E, K, by, flush=True)
    g = np.random.default_rng(T + E)
    ids = np.stack([g.permutation(E)[:K] for _ in range(T)]).astype(np.int32)
    res = g.random(E) < 0.5
    table = np.stack([np.delete(g.permutation(E), 0)[:4] for _ in range(E)]).astype(np.int32)
    table[table == np.arange(E)[:, None]] = -1
    ref, _, st = oracle.buddy_remap_gated(ids, res, table, np.ones((T, K), np.float32), H=4, unique=True, beta=1.5)
    desc = bm.LayerDesc(T=T, d=32, E=E, F=0, K=K, n_shared=0, R=4, H=4, dtype=bm.BM_BF16, flags=bm.BM_REMAP_UNIQUE | bm.BM_GATE_DIST,
                        dist_beta=1.5)
    out, stats = torch.full((T, K), -9, dtype=torch.int32, device="cuda"), torch.full((6,), -9, dtype=torch.int32, device="cuda")
    bm.bm_buddy_remap(desc, to_device(workloads.pack_bitmap(res)), to_device(table), _shifted(to_device(ids), by), out, None, stats)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), ref)
    assert stats.cpu().tolist() == [st["n_miss"], st["n_substituted"], st["n_dropped"], st["n_requested"], st["n_requested_offloaded"], 0]


# the input, the router matrix, the expert matrices; with the router product in its own launch (40 experts) and without
@pytest.mark.parametrize("which", ["x", "router", "experts", "all"])
@pytest.mark.parametrize("over", [dict(d=64, E=8, F=96), dict(d=96, E=40, F=64, K=4, n_resident=20, n_shared=1)])
def test_fp32_layer_takes_arrays_at_any_offset(which, over):
    from paper_2511_10054_amd.binding import make_weights
    spec = workloads.scaled("c1_tiny", **over)
    print("unaligned fp32", which, over, flush=True)
    host = HostLayer(spec, 19)
    ref = host.oracle_forward(oracle)
    dev = DeviceLayer(host)
    if which in ("x", "all"):
        dev.x = _shifted(dev.x, 1)
    if which in ("router", "all"):
        dev.w_router = _shifted(dev.w_router, 3)
    if which in ("experts", "all"):
        dev.wg, dev.wu, dev.wd, dev.sg, dev.su, dev.sd = (_shifted(t, 1 + i % 3) for i, t in enumerate((dev.wg, dev.wu, dev.wd, dev.sg, dev.su, dev.sd)))
    dev.weights = make_weights(dev.w_router, dev.bias, dev.wg, dev.wu, dev.wd, dev.sg, dev.su, dev.sd)
    out = dev.forward()
    np.testing.assert_array_equal(out["ids_remapped"], ref["ids_remapped"])
    assert err_metric(out["y"], ref["y"]) <= 1e-5
