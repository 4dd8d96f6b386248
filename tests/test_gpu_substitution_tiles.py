"""Substitution and grouping at the edges of their tiles: 64 tokens a tile, eight slots a batch, 64 assignments a word
of an assignment set (needs an MI355X).  Whole numbers, bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import to_device

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


# assignments around one and several words, one workgroup and a workgroup per tile, the largest batch and sets of both
@pytest.mark.parametrize("T,E,K", [(1, 1, 1), (21, 7, 3), (32, 256, 2), (65, 8, 1), (128, 32, 8), (129, 32, 8), (1024, 32, 1),
                                   (31, 256, 32), (33, 256, 32), (3001, 128, 8), (9000, 200, 4)])
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
