"""Co-activation counts at the edges of the chunks of tokens that a workgroup counts, and of the rule on their length (needs an MI355X)."""
import numpy as np
import pytest

import oracle
from test_gpu_profiling import _device_counts

pytestmark = pytest.mark.gpu


# 512 or 1024 tokens (coact_short_chunks) and 4 pivots a workgroup; a chunk each, but for 12000 tokens of 250 experts (12 chunks, 8
# workgroups along the tokens) and 140001 of 16 (137 chunks, 128 workgroups), the last chunk ragged
@pytest.mark.parametrize("T,E,K", [(511, 5, 2), (512, 4, 4), (513, 250, 3), (2048, 33, 5), (2049, 33, 5), (8192, 18, 8), (8193, 18, 8),
                                   (2049, 16, 1), (20000, 16, 3), (12000, 250, 9), (16384, 16, 3), (16385, 16, 3), (4096, 128, 8), (4097, 128, 8),
                                   (140001, 16, 2)])
def test_counts_of_short_and_long_chunks(T, E, K):
    print("coactivation chunks", T, E, K, flush=True)
    g = np.random.default_rng(T + E)
    ids = np.argsort(g.random((T, E)), axis=1)[:, :K].astype(np.int32)
    ids[::7, 0] = -1                                    # requests nothing
    A_ref, M_ref = oracle.coactivation(ids, E)
    A, M = _device_counts([ids], E, K)
    np.testing.assert_array_equal(A.cpu().numpy(), A_ref)
    np.testing.assert_array_equal(M.cpu().numpy(), M_ref)
