"""Costs that overflow: with a huge alpha two splits cost infinity, with an
infinite one every split does and a tree without a split costs NaN.  The best
individual is then still the one the oracle's scan ends with, in every launch
form (populations that leave lanes of a wave without an individual, whose place
in the search must never win)."""
import numpy as np
import pytest

import oracle
from paper_2311_06952_amd import synth

pytestmark = pytest.mark.gpu

FORMS = [
    # D, P, n, environment
    (2, 32, 900, {}),                                        # one resident block
    (3, 65, 900, {"MHDEOCT_RESIDENT_BLOCKS": "4"}),          # resident, several blocks
    (5, 100, 1500, {"MHDEOCT_RESIDENT_BLOCKS": "9"}),        # its shared-out costs
    (3, 100, 3000, {"MHDEOCT_PERSIST_RESIDENT": "0"}),       # staged whole run
    (2, 300, 900, {"MHDEOCT_PERSIST_RESIDENT": "0"}),        # several waves of individuals
    (3, 40, 700, {"MHDEOCT_PERSIST": "0"}),                  # one-block DE step
    (4, 70, 700, {"MHDEOCT_PERSIST": "0"}),                  # selection and mutation launches
    (3, 300, 700, {"MHDEOCT_PERSIST": "0"}),
    (3, 64, 700, {"MHDEOCT_PERSIST": "0", "MHDEOCT_FUSE_DE": "1"}),
    (6, 37, 500, {}),                                        # the walk path's DE launch
]


def _env(monkeypatch, env):
    for k, v in env.items():
        monkeypatch.setenv(k, v)


@pytest.mark.parametrize("alpha", [1e308, float("inf")])
@pytest.mark.parametrize("D,P,n,env", FORMS)
def test_infinite_costs(monkeypatch, D, P, n, env, alpha):
    import paper_2311_06952_amd as mh
    from paper_2311_06952_amd import capi
    _env(monkeypatch, env)
    X, y = synth.random_small(D * 100 + P, n, 5, 3)
    prm = (P, 6, 0.5, 0.6, 31, 2, alpha)
    want = oracle.deoct(oracle.dataset_from_X(X, y, 3), D, oracle.de_params(*prm), with_pop=True)
    assert D == 2 or not np.isfinite(want["pop_cost"]).any()
    ctx = capi.Context(0)
    got = mh.subtree_solve(mh.dataset(X, y, 3, ctx=ctx), D, mh.de_params(*prm), ctx=ctx,
                           with_pop=True)
    ctx.close()
    for key in ("feat", "tau", "label", "pop", "pop_cost", "cost"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"]


@pytest.mark.parametrize("env", [{}, {"MHDEOCT_PERSIST_RESIDENT": "0"}, {"MHDEOCT_PERSIST": "0"}])
@pytest.mark.parametrize("D_MH", [3, 4])
def test_infinite_costs_batched_horizon(monkeypatch, D_MH, env):
    import paper_2311_06952_amd as mh
    from paper_2311_06952_amd import capi
    _env(monkeypatch, env)
    X, y = synth.random_small(7, 1500, 5, 3)
    prm = (50, 4, 0.5, 0.6, 31, 2, 1e308)
    want = oracle.mh_train(oracle.dataset_from_X(X, y, 3), 5, D_MH, oracle.de_params(*prm))
    ctx = capi.Context(0)
    got = mh.mh_train(mh.dataset(X, y, 3, ctx=ctx), 5, D_MH, mh.de_params(*prm), batched=True,
                      ctx=ctx)
    ctx.close()
    for key in ("feat", "tau", "label", "cost"):
        np.testing.assert_array_equal(got[key], want[key])


@pytest.mark.parametrize("solo", ["0", "512"])
def test_infinite_costs_served(monkeypatch, solo):
    import torch

    import paper_2311_06952_amd as mh
    from paper_2311_06952_amd import capi
    monkeypatch.setenv("MHDEOCT_SERVE_SOLO_TILES", solo)  # stepped; run whole in a group
    ctx = capi.Context(0)
    srv = mh.Server(1 << 28, 4, ctx=ctx)
    reqs = [(900, 5, 3, 3, 40), (1500, 4, 2, 5, 100), (700, 6, 3, 2, 20)]
    for i, (n, F, K, D, P) in enumerate(reqs):
        X, y = synth.random_small(50 + i, n, F, K)
        srv.submit(i, torch.as_tensor(X).cuda(), torch.as_tensor(y).cuda(), K, D,
                   mh.de_params(P, 5, 0.5, 0.6, i, 1, 1e308))
    res = {r["req_id"]: r for r in srv.drain()}
    srv.close()
    ctx.close()
    for i, (n, F, K, D, P) in enumerate(reqs):
        X, y = synth.random_small(50 + i, n, F, K)
        want = oracle.deoct(oracle.dataset_from_X(X, y, K), D,
                            oracle.de_params(P, 5, 0.5, 0.6, i, 1, 1e308))
        assert res[i]["status"] == 0
        for key in ("feat", "tau", "label", "cost"):
            np.testing.assert_array_equal(res[i]["tree"][key], want[key])


@pytest.mark.parametrize("cost", [[np.inf, np.inf, np.inf], [np.inf, 3.0, np.nan, 3.0],
                                  [np.nan, 1.0, 2.0], [np.nan, np.nan, np.nan, np.inf]])
@pytest.mark.parametrize("D", [2, 6])
def test_infinite_costs_de_step(cost, D):
    import torch

    import paper_2311_06952_amd as mh
    P, F = len(cost), 4
    pop = oracle.de_init(P, D, F, 9, 2)
    c = np.array(cost)
    want = oracle.de_trial(pop, D, F, 0.7, 0.5, 9, 2, 1, oracle.argmin(c))
    best, trial = mh.de_step(mh.de_params(P, 3, 0.7, 0.5, 9), D, F, 2, 1,
                             torch.as_tensor(pop).cuda(), torch.as_tensor(c).cuda())
    assert int(best.cpu()[0]) == oracle.argmin(c)
    np.testing.assert_array_equal(trial.cpu().numpy(), want)
