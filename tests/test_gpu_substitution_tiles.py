"""Substitution and grouping at the edges of their tiles: 64 tokens a tile, eight slots a batch, 64 assignments a word
of an assignment set (needs an MI355X).  Whole numbers, bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import safe_threshold, tae_margin, to_device

pytestmark = pytest.mark.gpu


def _problem(seed, T, E, K, R, n_res):
    g = np.random.default_rng(seed)
    ids = np.stack([g.permutation(E)[:K] for _ in range(T)]).astype(np.int32)
    ids[g.random((T, K)) < 0.03] = -1
    res = np.zeros(E, bool)
    res[g.permutation(E)[:n_res]] = True
    # few favourites head every row: a token's misses compete for the same candidates
    fav = g.permutation(E)[: max(2, R)]
    table = np.stack([g.permutation(np.concatenate([fav, g.permutation(E)]))[:R] for _ in range(E)]).astype(np.int32)
    table[table == np.arange(E)[:, None]] = -1
    return ids, res, table


# one token, one tile, its neighbours, batches of one and of several workgroups, 1 to 4 words of experts, K past 8 and 16
@pytest.mark.parametrize("T,E,K,R,n_res", [(1, 5, 5, 3, 2), (63, 64, 8, 8, 40), (64, 65, 9, 8, 30), (65, 128, 16, 9, 60),
                                           (256, 129, 8, 8, 64), (257, 200, 17, 32, 90), (5000, 128, 8, 8, 64)])
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("dist", [False, True])
def test_substitution_tiles(T, E, K, R, n_res, in_place, dist):
    import torch
    import paper_2511_10054_amd as bm
    print("substitution tiles", T, E, K, R, n_res, in_place, dist, flush=True)
    ids, res, table = _problem(T + E, T, E, K, R, n_res)
    ref, _, st = oracle.buddy_remap(ids, res, table, H=R, unique=True, w=np.ones((T, K), np.float32))
    flags = bm.BM_REMAP_UNIQUE | (bm.BM_GATE_DIST if dist else 0)
    desc = bm.LayerDesc(T=T, d=32, E=E, F=0, K=K, n_shared=0, R=R, H=R, dtype=bm.BM_BF16, flags=flags, dist_beta=1.5)
    d_in = to_device(ids)
    d_out = d_in if in_place else torch.full((T, K), -9, dtype=torch.int32, device="cuda")
    stats = torch.full((6,), -9, dtype=torch.int32, device="cuda")
    bm.bm_buddy_remap(desc, to_device(workloads.pack_bitmap(res)), to_device(table), d_in, d_out, None, stats)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(d_out.cpu().numpy(), ref)
    req = np.unique(ids[ids >= 0])
    extra = [len(req), int((~res[req]).sum()), 0] if dist else [0, 0, 0]
    assert stats.cpu().tolist() == [st["n_miss"], st["n_substituted"], st["n_dropped"]] + extra


# K of the eight-lane form (up to 8) and of the walk (9, 17), budgets from none to more than enough, gates that close
# about half of the tokens (thresholds in a gap of the tokens' values), with and without U_t
@pytest.mark.parametrize("T,E,K,R,n_res", [(1, 8, 2, 3, 3), (65, 64, 6, 8, 30), (300, 128, 8, 8, 60), (64, 130, 9, 8, 60), (70, 200, 17, 8, 90)])
@pytest.mark.parametrize("unique", [False, True])
@pytest.mark.parametrize("rho", [None, 0, 1, 3, 32])
def test_gates_and_budget_in_substitution_tiles(T, E, K, R, n_res, unique, rho):
    import torch
    import paper_2511_10054_amd as bm
    print("gated substitution tiles", T, E, K, R, n_res, unique, rho, flush=True)
    ids, res, table = _problem(7 * T + E, T, E, K, R, n_res)
    w = np.random.default_rng(T).dirichlet(np.full(K, 0.7), size=T).astype(np.float32) + np.float32(1e-4)
    tae, margin = tae_margin(w.astype(np.float64))
    gates = [dict(), dict(tau=safe_threshold(tae, 0.5)), dict(gamma=safe_threshold(margin, 0.5))]
    for gate in gates:
        if rho is None and not gate:
            continue
        ref, w_ref, st = oracle.buddy_remap_gated(ids, res, table, w=w, H=R, unique=unique, rho=rho, **gate)
        flags = (bm.BM_REMAP_UNIQUE if unique else 0) | (bm.BM_REPLACE_BUDGET if rho is not None else 0)
        flags |= (bm.BM_GATE_TAE if "tau" in gate else 0) | (bm.BM_GATE_MARGIN if "gamma" in gate else 0)
        desc = bm.LayerDesc(T=T, d=32, E=E, F=0, K=K, n_shared=0, R=R, H=R, dtype=bm.BM_BF16, flags=flags, rho=rho or 0,
                            tae_tau=gate.get("tau", 0.0), margin_gamma=gate.get("gamma", 0.0))
        d_w, out = to_device(w), torch.full((T, K), -9, dtype=torch.int32, device="cuda")
        stats = torch.full((6,), -9, dtype=torch.int32, device="cuda")
        bm.bm_buddy_remap(desc, to_device(workloads.pack_bitmap(res)), to_device(table), to_device(ids), out, d_w, stats)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), ref)
        np.testing.assert_array_equal(d_w.cpu().numpy(), np.asarray(w_ref, np.float32))
        assert stats.cpu().tolist()[:3] == [st["n_miss"], st["n_substituted"], st["n_dropped"]]


# one slot a token, which has a form of its own: rows that head the expert itself (U_t holds it), every gate, batches of one
# and several workgroups, 1 to 4 words of experts
@pytest.mark.parametrize("T,E", [(1, 3), (64, 64), (97, 65), (300, 128), (257, 200)])
@pytest.mark.parametrize("unique", [False, True])
@pytest.mark.parametrize("gate", [dict(), dict(rho=0), dict(rho=1), dict(tau=0.5), dict(gamma=0.5), dict(gamma=1.5), dict(beta=1.5)])
def test_one_slot_per_token(T, E, unique, gate):
    import torch
    import paper_2511_10054_amd as bm
    print("one slot per token", T, E, unique, gate, flush=True)
    ids, res, table = _problem(T + E, T, E, 1, 3, (E + 1) // 2)
    table[:, 0] = np.where(np.arange(E) % 2 == 0, np.arange(E), table[:, 0])
    w = np.random.default_rng(E).uniform(0.1, 1.0, size=(T, 1)).astype(np.float32)
    ref, w_ref, st = oracle.buddy_remap_gated(ids, res, table, w=w, H=3, unique=unique, **gate)
    flags = bm.BM_REMAP_UNIQUE if unique else 0
    for name, bit in (("rho", bm.BM_REPLACE_BUDGET), ("tau", bm.BM_GATE_TAE), ("gamma", bm.BM_GATE_MARGIN), ("beta", bm.BM_GATE_DIST)):
        flags |= bit if name in gate else 0
    desc = bm.LayerDesc(T=T, d=32, E=E, F=0, K=1, n_shared=0, R=3, H=3, dtype=bm.BM_BF16, flags=flags, rho=gate.get("rho", 0),
                        tae_tau=gate.get("tau", 0.0), margin_gamma=gate.get("gamma", 0.0), dist_beta=gate.get("beta", 0.0))
    d_w, out = to_device(w), torch.full((T, 1), -9, dtype=torch.int32, device="cuda")
    stats = torch.full((6,), -9, dtype=torch.int32, device="cuda")
    bm.bm_buddy_remap(desc, to_device(workloads.pack_bitmap(res)), to_device(table), to_device(ids), out, d_w, stats)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), ref)
    np.testing.assert_array_equal(d_w.cpu().numpy(), np.asarray(w_ref, np.float32))
    assert stats.cpu().tolist()[:3] == [st["n_miss"], st["n_substituted"], st["n_dropped"]]


# the last batch that a single workgroup takes and the first that it does not, without ties, with U_t and for walks
@pytest.mark.parametrize("T,E,K", [(128, 24, 3), (129, 24, 3), (96, 24, 8), (97, 24, 8), (64, 40, 9), (65, 40, 9)])
@pytest.mark.parametrize("unique", [False, True])
def test_substitution_around_one_workgroup(T, E, K, unique):
    import torch
    import paper_2511_10054_amd as bm
    print("substitution around one workgroup", T, E, K, unique, flush=True)
    ids, res, table = _problem(T + K, T, E, K, 6, E // 2)
    ref, _, st = oracle.buddy_remap(ids, res, table, H=6, unique=unique, w=np.ones((T, K), np.float32))
    desc = bm.LayerDesc(T=T, d=32, E=E, F=0, K=K, n_shared=0, R=6, H=6, dtype=bm.BM_BF16, flags=bm.BM_REMAP_UNIQUE if unique else 0)
    out, stats = torch.full((T, K), -9, dtype=torch.int32, device="cuda"), torch.full((6,), -9, dtype=torch.int32, device="cuda")
    bm.bm_buddy_remap(desc, to_device(workloads.pack_bitmap(res)), to_device(table), to_device(ids), out, None, stats)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), ref)
    assert stats.cpu().tolist() == [st["n_miss"], st["n_substituted"], st["n_dropped"], 0, 0, 0]


# assignments around one and several words, one workgroup and a workgroup per tile, the largest batch and sets of both
@pytest.mark.parametrize("T,E,K", [(1, 1, 1), (21, 7, 3), (32, 256, 2), (65, 8, 1), (128, 32, 8), (129, 32, 8), (1024, 32, 1),
                                   (31, 256, 32), (32, 256, 32), (33, 256, 32), (128, 128, 8), (1024, 16, 2), (1024, 17, 2), (683, 15, 3), (3001, 128, 8), (9000, 200, 4)])
def test_grouping_sets(T, E, K):
    import torch
    import paper_2511_10054_amd as bm
    print("grouping sets", T, E, K, flush=True)
    ids = _problem(T * K, T, E, K, 1, 1)[0]
    ids[:, 0] = np.where(np.arange(T) % 3 == 0, E - 1, ids[:, 0])        # a large group
    desc = bm.LayerDesc(T=T, d=0, E=E, F=0, K=K, n_shared=0, R=0, H=0, dtype=bm.BM_BF16, flags=0)
    i32 = dict(dtype=torch.int32, device="cuda")
    off, perm, inv = torch.full((E + 1,), -9, **i32), torch.full((T * K,), -9, **i32), torch.full((T * K,), -9, **i32)
    ws = torch.full((bm.bm_workspace_bytes(desc),), 0xA5, dtype=torch.uint8, device="cuda")
    bm.bm_permute_by_expert(desc, to_device(ids), off, perm, inv, ws)
    torch.cuda.synchronize()
    for got, want in zip((off, perm, inv), oracle.permute(ids, E)):
        np.testing.assert_array_equal(got.cpu().numpy(), want)
