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


@pytest.mark.parametrize("D,D_MH,P", [(5, 4, 9), (5, 5, 64), (6, 4, 130)])
def test_selection_of_several_problems(monkeypatch, D, D_MH, P):
    """From depth 4 on the two launches also serve small populations, and the
    levels of a batched horizon run all their problems in one grid."""
    import paper_2311_06952_amd as mh
    from paper_2311_06952_amd import capi
    monkeypatch.setenv("MHDEOCT_PERSIST", "0")
    X, y = synth.random_small(D * 10 + P, 1500, 5, 4)
    prm = (P, 3, -1.0, 0.6, 5, 2, 0.5)
    want = oracle.mh_train(oracle.dataset_from_X(X, y, 4), D, D_MH, oracle.de_params(*prm))
    ctx = capi.Context(0)
    got = mh.mh_train(mh.dataset(X, y, 4, ctx=ctx), D, D_MH, mh.de_params(*prm), batched=True,
                      ctx=ctx)
    ctx.close()
    for key in ("feat", "tau", "label"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"] and got["cost"] == want["cost"]
