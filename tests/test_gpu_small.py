"""GPU parity of the one-launch preparation of small data sets (ranks, tile
plan, initial population) at the sizes where its kernels change course, and of
a burst of small served requests that needs more blocks than the device has
CUs."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev, np_, random_trees, u32
from paper_2311_06952_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mh():
    import paper_2311_06952_amd as m
    return m


@pytest.mark.parametrize("n", [1, 2, 63, 64, 1023, 1024, 1025, 2049, 4096, 4097, 8192, 8193, 14336,
                               14337, 22528, 22529])
@pytest.mark.parametrize("levels", [None, 9])
def test_ranks_and_tiles_at_round_edges(mh, n, levels):
    """Ranks equal to the oracle's, and the layout's counts on all samples and
    on a subset (repeated and reversed indices)."""
    X, y = synth.random_small(n, n, 3, 4, levels)
    X[: n // 2, 0] *= -1.0  # both signs, -0 beside +0
    ods, ds = oracle.dataset_from_X(X, y, 4), mh.dataset(X, y, 4)
    np.testing.assert_array_equal(u32(ds.ranks)[:, :n], ods.ranks)
    np.testing.assert_array_equal(u32(ds.n_unique), ods.n_unique)
    rng = np.random.default_rng(n)
    feat, tau = random_trees(rng, 5, 3, 3, ods.n_unique)
    idx = np.concatenate([np.arange(n)[::-1], np.arange(n)[: n // 3]]).astype(np.uint32)
    for sub in (None, idx):
        counts, correct, label, cost = mh.fitness_eval(ds, dev(feat), dev(tau), 3,
                                                       idx=None if sub is None else dev(sub))
        want = oracle.fitness(ods, feat, tau, 3, idx=sub)
        for got, w in zip((counts, correct, label, cost), want):
            np.testing.assert_array_equal(np_(got).astype(np.asarray(w).dtype), w)


def test_small_nan_is_reported(mh):
    from paper_2311_06952_amd import capi
    X, y = synth.random_small(3, 3000, 5, 2)
    X[2999, 4] = np.nan
    with pytest.raises(mh.MhError) as ei:
        mh.dataset(X, y, 2)
    assert ei.value.code == capi.MH_EINVAL


def test_burst_larger_than_the_device(mh):
    """Requests of every depth whose runs need several rounds of the CUs, each
    equal to the oracle's DEOCT."""
    import torch
    from paper_2311_06952_amd import capi
    rng = np.random.default_rng(11)
    ctx = capi.Context(0)
    srv = mh.Server(2 << 30, 64, ctx=ctx)
    reqs = []
    for j in range(30):
        n, F = int(rng.integers(1, 3000)) if j % 3 else 22_528 - j, int(rng.integers(1, 33))
        K, D, P = int(rng.integers(2, 11)), 1 + j % 5, int(rng.choice([3, 64, 65, 128]))
        X, y = synth.random_small(900 + j, n, F, K, 30 if j % 2 else None)
        prm = (P, 3, -1.0 if j % 4 == 0 else 0.5, 0.8, 40 + j, 1 + j % 3, 0.5 * (j % 2))
        srv.submit(j, torch.as_tensor(X).cuda(), torch.as_tensor(y).cuda(), K, D,
                   mh.de_params(*prm))
        reqs.append((X, y, K, D, prm))
    res = {r["req_id"]: r for r in srv.drain()}
    srv.close()
    ctx.close()
    for j, (X, y, K, D, prm) in enumerate(reqs):
        assert res[j]["status"] == 0
        want = oracle.deoct(oracle.dataset_from_X(X, y, K), D, oracle.de_params(*prm))
        got = res[j]["tree"]
        for key in ("feat", "tau", "label"):
            np.testing.assert_array_equal(got[key], want[key])
        assert got["correct"] == want["correct"] and got["cost"] == want["cost"]
