"""Co-activation counts at the edges of the short chunks and of the rule that takes them (needs an MI355X)."""
import numpy as np
import pytest

import oracle
from test_gpu_profiling import _device_counts

pytestmark = pytest.mark.gpu


# 512 tokens and 4 pivots a workgroup: up to 2048 tokens, or up to 16 experts, or eight and more slots up to 8192 tokens;
# 12000 tokens of 250 experts walk several chunks of 1024, 20000 of 16 several of 512
@pytest.mark.parametrize("T,E,K", [(511, 5, 2), (512, 4, 4), (513, 250, 3), (2048, 33, 5), (2049, 33, 5), (8192, 18, 8), (8193, 18, 8),
                                   (2049, 16, 1), (20000, 16, 3), (12000, 250, 9)])
def test_counts_of_short_and_long_chunks(T, E, K):
    print("coactivation chunks", T, E, K, flush=True)
    g = np.random.default_rng(T + E)
    ids = np.argsort(g.random((T, E)), axis=1)[:, :K].astype(np.int32)
    ids[::7, 0] = -1                                    # requests nothing
    A_ref, M_ref = oracle.coactivation(ids, E)
    A, M = _device_counts([ids], E, K)
    np.testing.assert_array_equal(A.cpu().numpy(), A_ref)
    np.testing.assert_array_equal(M.cpu().numpy(), M_ref)
