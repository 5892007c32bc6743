"""GPU parity of the whole-run kernel with resident tiles (one block, several
blocks, the class counts in chunks, every depth and group count) against the
oracle: best tree, counts, cost and the final population bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2311_06952_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mh():
    import paper_2311_06952_amd as m
    return m


@pytest.mark.parametrize("blocks", [0, 1, 2, 7])
@pytest.mark.parametrize("D,P,K,n,F,M,alpha,n_min", [
    (1, 3, 2, 5, 1, 0.5, 0.0, 1),        # fewer samples than a tile, the smallest population
    (2, 32, 2, 1000, 4, 0.5, 0.0, 1),
    (3, 64, 5, 900, 3, -1.0, 2.0, 7),    # one wave of individuals, 16 groups
    (3, 129, 3, 640, 6, 0.5, 0.0, 1),    # a padded wave
    (4, 100, 4, 1500, 5, -1.0, 0.5, 3),
    (4, 300, 2, 300, 4, 0.5, 0.0, 1),    # two groups per block
    (5, 65, 3, 1200, 7, 0.5, 0.0, 2),
    (5, 100, 23, 2000, 4, -1.0, 1.0, 4),  # more classes than counters: chunks
    (5, 256, 2, 400, 2, 0.5, 0.0, 1),    # the widest population at depth 5
    (4, 64, 255, 700, 3, 0.5, 0.0, 1),
])
def test_resident_run_matches_oracle(mh, monkeypatch, blocks, D, P, K, n, F, M, alpha, n_min):
    from paper_2311_06952_amd import capi
    X, y = synth.random_small(D * 1000 + P, n, F, K, levels=50 if K == 5 else None)
    prm = (P, 12, M, 0.7, 77 + D, n_min, alpha)
    want, pop, cost = _oracle(X, y, K, D, prm)
    monkeypatch.setenv("MHDEOCT_RESIDENT_BLOCKS", str(blocks))
    ctx = capi.Context(0)
    got = mh.subtree_solve(mh.dataset(X, y, K, ctx=ctx), D, mh.de_params(*prm), ctx=ctx,
                           with_pop=True)
    ctx.close()
    for key in ("feat", "tau", "label"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"] and got["cost"] == want["cost"]
    np.testing.assert_array_equal(got["pop"], pop)
    np.testing.assert_array_equal(got["pop_cost"], cost)


def _oracle(X, y, K, D, prm):
    r = oracle.deoct(oracle.dataset_from_X(X, y, K), D, oracle.de_params(*prm), with_pop=True)
    return r, r["pop"], r["pop_cost"]


# the kernel each shape runs in: one resident block only where its searches cost
# less than the other form's exchange, several from depth 3 on and up to 128
# individuals, or at depth 1 where few classes and many tiles meet
@pytest.mark.parametrize("D,P,K,n,F,kernel", [
    (2, 32, 2, 1000, 4, "k_deoct_resident<2,1>: 1 runs, grid 1,"),
    (2, 512, 2, 300, 4, "k_deoct_persist<2,"),
    (3, 262, 2, 2000, 3, "k_deoct_persist<3,"),
    (3, 100, 2, 2000, 4, "k_deoct_resident<3,2>: 1 runs, grid "),
    (1, 64, 5, 4000, 10, "k_deoct_persist<1,"),
    (1, 64, 2, 30_000, 4, "k_deoct_resident<1,1>: 1 runs, grid "),
    (1, 300, 2, 30_000, 4, "k_deoct_persist<1,"),
    (2, 100, 3, 8000, 20, "k_deoct_persist<2,"),
])
def test_whole_run_form_by_shape(mh, monkeypatch, capfd, D, P, K, n, F, kernel):
    from paper_2311_06952_amd import capi
    X, y = synth.random_small(D * 1000 + P, n, F, K)
    prm = (P, 5, 0.5, 0.7, 7, 1, 0.0)
    want, pop, cost = _oracle(X, y, K, D, prm)
    monkeypatch.setenv("MHDEOCT_DEBUG", "1")
    ctx = capi.Context(0)
    capfd.readouterr()
    got = mh.subtree_solve(mh.dataset(X, y, K, ctx=ctx), D, mh.de_params(*prm), ctx=ctx,
                           with_pop=True)
    err = capfd.readouterr().err
    ctx.close()
    assert kernel in err
    if "grid 1," not in kernel:
        assert "grid 1," not in err
    for key in ("feat", "tau", "label"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"] and got["cost"] == want["cost"]
    np.testing.assert_array_equal(got["pop"], pop)
    np.testing.assert_array_equal(got["pop_cost"], cost)
