"""Which batches stream and which are tiled, seen through the workspaces that the layer takes (no GPU)."""
import ctypes

import pytest

import paper_2511_10054_amd as bm
from paper_2511_10054_amd.binding import DebugOut, LayerDesc, Weights


def _desc(T, **shape):
    a = dict(T=T, d=2048, E=128, F=768, K=8, n_shared=0, R=4, H=4, dtype=bm.BM_BF16, flags=0, tae_tau=0.0, rho=0, dist_beta=0.0)
    a.update(shape)
    return LayerDesc(**a)


def _accepts(desc, nbytes):
    """bm_moe_forward takes a workspace of so many bytes (it then stops, before any launch, at the half-filled events)."""
    one = ctypes.c_void_p(256)
    w = Weights(*([256] * 8 + [0] * 5))
    dbg = DebugOut()
    dbg.stage_events[0] = 1
    rc = bm.load_library().bm_moe_forward(ctypes.byref(desc), one, ctypes.byref(w), one, one, one, one, nbytes, ctypes.byref(dbg), None)
    assert rc in (-1, -4), rc
    return rc == -1


# up to 256 rows, or 16 rows an expert on average, a batch streams and its down-projection output is held in fp32;
# beyond, it is tiled (bf16 output): the sizes say which
@pytest.mark.parametrize("shape,T,n", [(dict(), 208, 16243712), (dict(), 220, 17181696), (dict(), 256, 19991552), (dict(), 300, 13601024),
                                       (dict(d=4096, E=8, F=14336, K=2), 112, 13770752), (dict(d=4096, E=8, F=14336, K=2), 128, 15736832),
                                       (dict(d=4096, E=8, F=14336, K=2), 512, 104887552)])
def test_batches_that_stream_keep_their_fp32_output(shape, T, n):
    assert bm.bm_workspace_bytes(_desc(T, **shape)) == n
    assert _accepts(_desc(T, **shape), n)
