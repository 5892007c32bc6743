"""The selection launch of large populations (eight individuals per block, the
counts in LDS, classes in chunks) against the oracle: a whole run by the
per-generation kernels, its best tree and final population bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2311_06952_amd import synth

pytestmark = pytest.mark.gpu


# the last block full, with one individual and with seven; one class, and more
# classes than a chunk holds at depth 5 (33) and 4 (68)
@pytest.mark.parametrize("D,P,K,n,M,n_min", [
    (1, 256, 1, 900, 0.5, 1), (2, 257, 3, 1200, -1.0, 4), (3, 263, 2, 2000, 0.5, 1),
    (4, 512, 69, 3000, 0.5, 2), (5, 256, 33, 2500, -1.0, 1), (5, 300, 34, 2500, 0.5, 3),
    (5, 257, 255, 2600, 0.5, 1)])
def test_large_population_selection(monkeypatch, D, P, K, n, M, n_min):
    import paper_2311_06952_amd as mh
    from paper_2311_06952_amd import capi
    monkeypatch.setenv("MHDEOCT_PERSIST", "0")
    X, y = synth.random_small(D * 100 + P, n, 4, K)
    prm = (P, 4, M, 0.6, 21, n_min, 0.25)
    want = oracle.deoct(oracle.dataset_from_X(X, y, K), D, oracle.de_params(*prm), with_pop=True)
    ctx = capi.Context(0)
    got = mh.subtree_solve(mh.dataset(X, y, K, ctx=ctx), D, mh.de_params(*prm), ctx=ctx,
                           with_pop=True)
    ctx.close()
    for key in ("feat", "tau", "label", "pop", "pop_cost"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"] and got["cost"] == want["cost"]
