"""A token's routing is the same bits whatever call, batch or gate it comes through (needs an MI355X): the router
product adds the hidden dimension in one order for every number of tokens, in the launch of its own as well as inside the
front kernels, so an engine that prefetches by bm_route_topk loads the experts that bm_moe_forward then asks for."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MOST = 8200                    # past the batch from which the bf16 front kernel takes 32-token tiles


# expert counts of every form of the product (up to 16, 32, 64, 128 and 256 experts); hidden widths with and without a
# partial last batch of the waves, and one that gives some waves nothing
@pytest.mark.parametrize("dtype,E,d", [("bf16", 8, 288), ("bf16", 24, 1024), ("bf16", 64, 2080), ("bf16", 65, 288), ("bf16", 128, 2336),
                                       ("bf16", 128, 64), ("bf16", 200, 1056), ("f32", 8, 288), ("f32", 33, 96), ("f32", 64, 1056),
                                       ("f32", 128, 288), ("f32", 200, 1056), ("f32", 40, 50)])
def test_every_call_routes_alike(dtype, E, d):
    import torch
    import paper_2511_10054_amd as bm
    from paper_2511_10054_amd.binding import make_weights
    print("routing bits", dtype, E, d, flush=True)
    K, F = min(8, E), 64
    g = torch.Generator(device="cuda")
    g.manual_seed(E * 10007 + d)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32

    def rand(*shape, scale=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * scale).to(td)

    x, wr, bias = rand(MOST, d), rand(E, d, scale=d ** -0.5), torch.randn(E, generator=g, device="cuda")
    weights = make_weights(wr, bias, rand(E, F, d, scale=d ** -0.5), rand(E, F, d, scale=d ** -0.5), rand(E, d, F, scale=0.1))
    words = np.zeros((E + 63) // 64, np.uint64)
    for e in range(E):
        words[e // 64] |= np.uint64(1) << np.uint64(e % 64)
    bitmap = torch.from_numpy(words.view(np.int64)).cuda()                  # all resident: nothing is replaced or dropped
    table = torch.full((E, 1), -1, dtype=torch.int32, device="cuda")

    def desc(T, flags=0):
        return bm.LayerDesc(T=T, d=d, E=E, F=F, K=K, n_shared=0, R=1, H=1, dtype=bm.BM_BF16 if dtype == "bf16" else bm.BM_F32,
                            flags=bm.BM_RENORM_TOPK | flags, dist_beta=2.0)

    def outputs(T):
        return (torch.full((T, K), -7, dtype=torch.int32, device="cuda"), torch.full((T, K), -7.0, device="cuda"))

    ids_all, w_all = outputs(MOST)
    bm.bm_route_topk(desc(MOST), x, wr, bias, ids_all, w_all)
    for T in (1, 16, 17, 32, 33, 64, 65, 300, 1024, 1025, MOST):
        want_ids, want_w = ids_all[:T], w_all[:T].view(torch.int32)
        xs = x[:T]
        ids, w = outputs(T)
        bm.bm_route_topk(desc(T), xs, wr, bias, ids, w)
        assert torch.equal(ids, want_ids) and torch.equal(w.view(torch.int32), want_w), ("route_topk", T)
        for flags in (0, bm.BM_GATE_DIST):                                  # the gate: one workgroup up to 32 tokens, routing apart beyond
            ids, w = outputs(T)
            ws = torch.full((bm.bm_workspace_bytes(desc(T, flags)),), 0xA5, dtype=torch.uint8, device="cuda")
            y = torch.empty((T, d), dtype=td, device="cuda")
            bm.bm_moe_forward(desc(T, flags), xs, weights, bitmap, table, y, ws, dict(ids=ids, w=w))
            torch.cuda.synchronize()
            assert torch.equal(ids, want_ids) and torch.equal(w.view(torch.int32), want_w), ("forward", T, flags)
